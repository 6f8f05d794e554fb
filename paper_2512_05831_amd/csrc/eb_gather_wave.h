// Wave gather: a whole wave per bag, or up to 16 waves (one workgroup) for one
// long bag.  Selection by shape in choose_route (eb_gather.h), instantiated in
// eb_gather_wave.hip and eb_gather_wave_weighted.hip.
//
// What bounds the gather when rows come from the caches is vector issue and
// the L1 path, not HBM, so this kernel keeps both short:
//   * the bag is wave-uniform: its bounds come by scalar loads and its loops
//     branch on scalars;
//   * rows are read with structured buffer loads: the hardware multiplies the
//     staged row number by the row pitch and adds the lane's offset, so a
//     load needs no address arithmetic, and a row number past the table's
//     last reads zeros, so a bag's last pass needs no predication (the window
//     is padded with kInvalidRow).  The product is taken modulo 2^32, so only
//     launches whose tables all hold less than 4 GB of gatherable rows come
//     here;
//   * 16-byte loads for any row of 16 bytes or more, whatever its size: the
//     last lane of a ragged row reads the row's last 16 bytes, overlapping its
//     neighbour's, so nothing past the row is touched.  gfx950 serves buffer
//     and global accesses at any byte alignment (rows at multiples of 4 bytes
//     at the aligned rate, rows at odd multiples of 2 bytes about a third
//     slower from the L2s).
// (v_fma_mix_f32 in place of a conversion and an addition per fp16 element
// was slower: 64 ids of 512 B each, 16 x 4096 bags, 229 against 174 us.)
#pragma once

#include "eb_gather.h"
#include "eb_internal.h"

namespace eb_gather {

using eb_detail::scalar_load;

typedef int i32x4 __attribute__((ext_vector_type(4)));

// buffer_load_dwordx4 with an index and an offset per lane.
__device__ u32x4 struct_load_x4(i32x4 rsrc, int index, int offset, int soffset, int aux)
    __asm("llvm.amdgcn.struct.buffer.load.v4i32");
constexpr int kAuxNt = 2; // non-temporal

// A table as n records of `pitch` bytes (pitch below 2^14).
__device__ __forceinline__ i32x4 table_rsrc(const char *p, uint32_t pitch, uint32_t n)
{
    const uint64_t a = (uint64_t)p;
    i32x4 r;
    r[0] = (int)(uint32_t)a;
    r[1] = (int)(((uint32_t)(a >> 32) & 0xFFFFu) | (pitch << 16));
    r[2] = (int)n;
    r[3] = 0x00020000;
    return r;
}

template <int DT, bool kW>
__device__ __forceinline__ void pool16(float *acc, u32x4 v, float w)
{
    if constexpr (kW) {
        Elem<DT>::fma(acc, make_uint4(v[0], v[1], v[2], v[3]), w);
    } else {
        Elem<DT>::add(acc, make_uint4(v[0], v[1], v[2], v[3]));
    }
}

// One pass: U rows per lane group, the group's staged entries P apart.
template <int DT, int P, int C, int U, bool kW, bool kStream>
__device__ __forceinline__ void wave_pass(float *acc, i32x4 rsrc, const int *coff, const uint32_t *rows,
                                          const float *weights)
{
    constexpr int kEpc = 16 / (DT == EB_F32 ? 4 : 2);
    int row[U];
    float w[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        row[u] = (int)rows[u * P];
        w[u] = kW ? weights[u * P] : 1.f;
    }
    u32x4 v[U][C];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int c = 0; c < C; ++c) v[u][c] = struct_load_x4(rsrc, row[u], coff[c], 0, kStream ? kAuxNt : 0);
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int c = 0; c < C; ++c) pool16<DT, kW>(acc + c * kEpc, v[u][c], w[u]);
}

__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Rows in flight per lane group, U * C KB per wave: 4 for rows of 65 to 512
// bytes, less for narrower ones (a pass stays within a window of 64), 5 to 8
// for wider ones; registers for 8 waves per SIMD up to 512-B rows and for 5 and
// more up to 2 KB (2 instead of 4 for 128-B rows: 15% slower; 8 instead of 4 for
// 512-B rows: within 1%; 4 instead of 8 for 768-B rows in bags of 64: 4%
// slower).
constexpr int wave_unroll(int R, int C)
{
    return C > 1 ? (C >= 5 ? 1 : C >= 3 ? 2 : 4) : R == 64 ? 8 : R >= 8 ? 4 : R >= 2 ? 2 : 1;
}

// R lanes of 16-byte chunks per row, C chunks per lane; P = 64 / R rows at a
// time.  Launched with grid.y = tables.  a.split == 1: workgroups of 4 waves,
// a bag each.  a.split > 1: workgroups of a.split waves, which take a bag's
// windows of 64 ids in turn; their partial sums meet in LDS
// (a.split * chunks * 16 bytes' worth of floats, dynamic).
template <typename IT, int DT, int R, int C, bool kW, bool kStream>
__global__ __launch_bounds__(kWave *wave_block(C, DT)) void eb_gather_wave(const GatherArgs a)
{
    constexpr int P = kWave / R;
    constexpr int U = wave_unroll(R, C);
    constexpr int kEs = DT == EB_F32 ? 4 : 2;
    constexpr int kEpc = 16 / kEs;
    static_assert(U * P <= kWave, "a pass stays within the window");
    constexpr int kWaves = wave_block(C, DT);
    __shared__ uint32_t stage[kWaves][kWave];
    __shared__ float wstage[kW ? kWaves : 1][kWave];
    __shared__ int wave_hits[kWaves];
    extern __shared__ float partial[];

    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const int g = lane / R, rl = lane % R;
    int t = blockIdx.y, block = blockIdx.x;
    if (a.xcd_runs) { // workgroups go to the XCDs in turn: each takes a run of them
        const int n = gridDim.x * gridDim.y, i = t * gridDim.x + block, x = i % kXcds;
        const int lb = x * (n / kXcds) + min(x, n % kXcds) + i / kXcds;
        t = lb / (int)gridDim.x;
        block = lb - t * (int)gridDim.x;
    }
    const int split = a.split;
    const int64_t b = a.bag_begin + (split > 1 ? (int64_t)block : (int64_t)block * kWavesPerBlock + wave);
    if (b >= a.B) return; // never a part of a split bag's workgroup

    const IT *o = (const IT *)a.offsets + (int64_t)t * a.B + b;
    int64_t s = scalar_load(o), e = scalar_load(o + 1);
    clamp_bag(s, e, a.nnz);
    const uint64_t nlocal = a.nlocal[t];
    const uint64_t shard_lo = (uint64_t)a.shard_lo;
    const i32x4 rsrc = table_rsrc(a.base[t], (uint32_t)a.row_bytes, (uint32_t)nlocal);
    int coff[C];
#pragma unroll
    for (int c = 0; c < C; ++c) coff[c] = min(16 * (c * R + rl), a.row_bytes - 16);
    uint32_t *rows = stage[wave];
    float *weights = wstage[kW ? wave : 0];

    float acc[C * kEpc];
#pragma unroll
    for (int j = 0; j < C * kEpc; ++j) acc[j] = 0.f;
    int count = 0;

    const IT *ids = (const IT *)a.indices;
    int64_t w0 = s + (split > 1 ? (int64_t)wave * kWave : 0);
    IT id = 0;
    float w = 0.f;
    auto load_window = [&](int64_t at) {
        const int64_t k = at + min(lane, (int)min<int64_t>(e - at, kWave) - 1);
        id = __builtin_nontemporal_load(ids + k);
        if constexpr (kW) w = __builtin_nontemporal_load(a.weights + k);
    };
    if (w0 < e) load_window(w0);
    while (w0 < e) {
        // The window's gathered ids to its front as local rows, in position
        // order; the rest of it reads as zeros.
        const uint64_t r = (uint64_t)(int64_t)id - shard_lo;
        const bool ok = lane < (int)min<int64_t>(e - w0, kWave) && r < nlocal;
        const uint64_t m = __ballot(ok);
        const int nv = (int)__popcll(m);
        rows[lane] = kInvalidRow;
        if constexpr (kW) weights[lane] = 0.f;
        if (ok) {
            const int at = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
            rows[at] = (uint32_t)r;
            if constexpr (kW) weights[at] = w;
        }
        count += nv;
        wave_lds_sync();
        w0 += (int64_t)split * kWave;
        if (w0 < e) load_window(w0); // in flight while this window's rows are
        // Full passes, then a half or a quarter one for what is left.
        int k = 0;
        for (; nv - k > U * P / 2; k += U * P)
            wave_pass<DT, P, C, U, kW, kStream>(acc, rsrc, coff, rows + k + g, weights + k + g);
        if (U >= 4 && nv - k > U * P / 4)
            wave_pass<DT, P, C, (U + 1) / 2, kW, kStream>(acc, rsrc, coff, rows + k + g, weights + k + g);
        else if (nv - k > 0)
            wave_pass<DT, P, C, (U >= 4 ? U / 4 : (U + 1) / 2), kW, kStream>(acc, rsrc, coff, rows + k + g, weights + k + g);
        wave_lds_sync();
    }
    team_reduce<R, P>(acc);

    const int64_t L = e - s;
    float *dst = a.out + b * a.ldo + a.col[t];
    // The first wave has all of a bag of one window, and ends it alone.
    if (split > 1 && L <= kWave && wave > 0) return;
    if (split > 1 && L > kWave) {
        // Chunk by chunk, as loaded: the last one holds the row's last kEpc elements.
        const int width = a.chunks * kEpc;
        if (g == 0) {
#pragma unroll
            for (int c = 0; c < C; ++c) {
                if (c * R + rl >= a.chunks) break;
#pragma unroll
                for (int j = 0; j < kEpc; ++j) partial[wave * width + (c * R + rl) * kEpc + j] = acc[c * kEpc + j];
            }
        }
        if (lane == 0) wave_hits[wave] = count;
        __syncthreads();
        for (int c = threadIdx.x; c < a.D; c += blockDim.x) {
            const int at = c < width - kEpc ? c : c + width - a.D;
            float x = 0.f;
            for (int v = 0; v < split; ++v) x += partial[v * width + at];
            if (a.mean) x = L > 0 ? x / (float)L : 0.f;
            __builtin_nontemporal_store(x, dst + c);
        }
        if (a.hits && threadIdx.x == 0) {
            int h = 0;
            for (int v = 0; v < split; ++v) h += wave_hits[v];
            a.hits[b * a.ldh + t] = h;
        }
        return;
    }
    if (g == 0) {
        if (a.mean) {
            const float fl = (float)L;
#pragma unroll
            for (int j = 0; j < C * kEpc; ++j) acc[j] = L > 0 ? acc[j] / fl : 0.f;
        }
        // Stores at any multiple of 4 bytes; where the last chunk overlaps its
        // neighbour both store the same sums.
        typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
#pragma unroll
        for (int c = 0; c < C; ++c) {
            if (c * R + rl >= a.chunks) break;
#pragma unroll
            for (int h = 0; h < kEpc / 4; ++h) {
                const float *x = acc + c * kEpc + 4 * h;
                const f32x4_any v = {x[0], x[1], x[2], x[3]};
                __builtin_nontemporal_store(v, (f32x4_any *)(dst + coff[c] / kEs + 4 * h));
            }
        }
        if (a.hits && rl == 0) a.hits[b * a.ldh + t] = count;
    }
}

// The wave kernel for R lanes and C chunks per lane (C > 1 with R = 64 only).
template <typename IT, int DT, bool kW, bool kStream>
KernelFn pick_wave_kernel(int R, int C)
{
    switch (R) {
    case 1: return eb_gather_wave<IT, DT, 1, 1, kW, kStream>;
    case 2: return eb_gather_wave<IT, DT, 2, 1, kW, kStream>;
    case 4: return eb_gather_wave<IT, DT, 4, 1, kW, kStream>;
    case 8: return eb_gather_wave<IT, DT, 8, 1, kW, kStream>;
    case 16: return eb_gather_wave<IT, DT, 16, 1, kW, kStream>;
    case 32: return eb_gather_wave<IT, DT, 32, 1, kW, kStream>;
    }
    switch (C) {
    case 1: return eb_gather_wave<IT, DT, 64, 1, kW, kStream>;
    case 2: return eb_gather_wave<IT, DT, 64, 2, kW, kStream>;
    case 3: return eb_gather_wave<IT, DT, 64, 3, kW, kStream>;
    case 4: return eb_gather_wave<IT, DT, 64, 4, kW, kStream>;
    case 5: return eb_gather_wave<IT, DT, 64, 5, kW, kStream>;
    case 6: return eb_gather_wave<IT, DT, 64, 6, kW, kStream>;
    case 7: return eb_gather_wave<IT, DT, 64, 7, kW, kStream>;
    case 8: return eb_gather_wave<IT, DT, 64, 8, kW, kStream>;
    }
    return nullptr;
}

template <typename IT, bool kW>
KernelFn pick_wave_kernel(int dtype, int R, int C, bool stream)
{
    switch (dtype) {
    case EB_F32: return stream ? pick_wave_kernel<IT, EB_F32, kW, true>(R, C) : pick_wave_kernel<IT, EB_F32, kW, false>(R, C);
    case EB_F16: return stream ? pick_wave_kernel<IT, EB_F16, kW, true>(R, C) : pick_wave_kernel<IT, EB_F16, kW, false>(R, C);
    default: return stream ? pick_wave_kernel<IT, EB_BF16, kW, true>(R, C) : pick_wave_kernel<IT, EB_BF16, kW, false>(R, C);
    }
}

} // namespace eb_gather
