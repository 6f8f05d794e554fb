// Gather kernels of the pooled lookup and their selection by shape (shared by
// the translation units that instantiate them: eb.hip for unweighted bags,
// eb_gather_weighted.hip for per-sample weights).  The kernel design is
// described at the top of eb.hip.
#pragma once

#include <hip/hip_runtime.h>

#include <stdint.h>

#include "../../include/eb.h"
#include "../../include/eb_route.h"

namespace eb_gather {


typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kWave = 64;
constexpr int kWavesPerBlock = 4;
constexpr int kBlock = kWave * kWavesPerBlock;
constexpr int kXcds = 8;
constexpr int kMaxTablesPerLaunch = 64;
constexpr int kStagePerWave = 256;                // LDS index window, entries per wave
constexpr int kMaxSplit = 16;                     // waves per bag of the wave kernel
constexpr uint32_t kInvalidRow = 0xFFFFFFFFu;     // never a staged row: local rows stay below it
constexpr uint64_t kMaxLocalRows = 0xFFFFFFFEull; // local rows must fit below the marker

// Per-launch arguments.  The table arrays are read with a block-uniform
// index, so they stay in the kernel-argument segment (scalar loads).
struct GatherArgs {
    const char *base[kMaxTablesPerLaunch]; // stored table (local row 0 = global row shard_lo)
    uint64_t nlocal[kMaxTablesPerLaunch];  // gatherable local rows of each table
    int64_t col[kMaxTablesPerLaunch];      // output column of each table's first element
    const void *indices;    // int64 or int32 (the kernel's index type)
    const void *offsets;    // bag (t, b) of this launch at offsets[t*B + b]
    const float *weights;   // per-sample weights [nnz] (weighted kernels only)
    float *out;             // element (b, t, c) at out[b*ldo + col[t] + c]
    int32_t *hits;          // hits[b*ldh + t], or null
    int64_t nnz;
    int64_t B;
    int64_t bag_begin;      // first bag (within each table) of this launch
    int64_t shard_lo;
    int64_t ldo;
    int64_t ldh;
    int32_t D;
    int32_t row_bytes;      // D * element bytes
    int32_t chunks;         // chunks per row (the wave kernel's last one may overlap its neighbour)
    int32_t blocks_per_table;
    int32_t nblocks;        // logical blocks; the grid is padded to a multiple of 8
    int32_t mean;
    int32_t xcd_runs;       // give each XCD a contiguous run of logical blocks
    int32_t split;          // waves per bag (wave kernel)
};

// ---------------------------------------------------------------------------- device helpers

// Block id -> logical block such that XCD x (which receives hardware blocks
// x, x+8, x+16, ...) works on logical blocks [x*per, (x+1)*per).
__device__ __forceinline__ int xcd_contiguous_block(int bid, int padded)
{
    const int per = padded / kXcds;
    return (bid % kXcds) * per + bid / kXcds;
}

// v + (v of lane ^ m), for the lane-group sizes the teams use.
template <int M>
__device__ __forceinline__ float add_xor(float v)
{
    static_assert(M == 1 || M == 2 || M == 4 || M == 8 || M == 16 || M == 32, "lane mask");
    if constexpr (M == 1) {   // DPP quad_perm [1,0,3,2]
        return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xF, 0xF, false));
    } else if constexpr (M == 2) { // DPP quad_perm [2,3,0,1]
        return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x4E, 0xF, 0xF, false));
    } else if constexpr (M == 8) { // DPP row_ror:8 == xor 8 inside a 16-lane row
        return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x128, 0xF, 0xF, false));
    } else if constexpr (M == 32) { // swap the two 32-lane halves
        auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        return __uint_as_float(r[0]) + __uint_as_float(r[1]);
    } else { // ds_swizzle bit mode: and 0x1f, xor M (within 32 lanes)
        return v + __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(v), (M << 10) | 0x1F));
    }
}

// Sum over the P lane groups of a team (groups are R lanes apart).
template <int R, int P, int N>
__device__ __forceinline__ void team_reduce(float (&acc)[N])
{
    if constexpr (P > 1) {
#pragma unroll
        for (int j = 0; j < N; ++j) acc[j] = add_xor<R>(acc[j]);
        if constexpr (P > 2) team_reduce<R * 2, P / 2, N>(acc);
    }
}

// Elements per 16-byte chunk and their widening to fp32.
template <int DT> struct Elem;
template <> struct Elem<EB_F32> {
    static constexpr int kPerChunk = 4;
    __device__ static __forceinline__ void add(float *acc, uint4 v)
    {
        acc[0] += __uint_as_float(v.x);
        acc[1] += __uint_as_float(v.y);
        acc[2] += __uint_as_float(v.z);
        acc[3] += __uint_as_float(v.w);
    }
    __device__ static __forceinline__ void fma(float *acc, uint4 v, float w)
    {
        acc[0] = fmaf(w, __uint_as_float(v.x), acc[0]);
        acc[1] = fmaf(w, __uint_as_float(v.y), acc[1]);
        acc[2] = fmaf(w, __uint_as_float(v.z), acc[2]);
        acc[3] = fmaf(w, __uint_as_float(v.w), acc[3]);
    }
    __device__ static __forceinline__ void add(float *acc, uint2 v)
    {
        acc[0] += __uint_as_float(v.x);
        acc[1] += __uint_as_float(v.y);
    }
    __device__ static __forceinline__ void fma(float *acc, uint2 v, float w)
    {
        acc[0] = fmaf(w, __uint_as_float(v.x), acc[0]);
        acc[1] = fmaf(w, __uint_as_float(v.y), acc[1]);
    }
    __device__ static __forceinline__ void add(float *acc, uint32_t v) { acc[0] += __uint_as_float(v); }
    __device__ static __forceinline__ void fma(float *acc, uint32_t v, float w) { acc[0] = fmaf(w, __uint_as_float(v), acc[0]); }
    __device__ static __forceinline__ float load1(const char *p) { return *(const float *)p; }
};
template <> struct Elem<EB_F16> {
    static constexpr int kPerChunk = 8;
    __device__ static __forceinline__ float lo(uint32_t w) { return (float)__builtin_bit_cast(_Float16, (uint16_t)(w & 0xFFFFu)); }
    __device__ static __forceinline__ float hi(uint32_t w) { return (float)__builtin_bit_cast(_Float16, (uint16_t)(w >> 16)); }
    __device__ static __forceinline__ void add(float *acc, uint4 v)
    {
        acc[0] += lo(v.x); acc[1] += hi(v.x);
        acc[2] += lo(v.y); acc[3] += hi(v.y);
        acc[4] += lo(v.z); acc[5] += hi(v.z);
        acc[6] += lo(v.w); acc[7] += hi(v.w);
    }
    __device__ static __forceinline__ void fma(float *acc, uint4 v, float w)
    {
        acc[0] = fmaf(w, lo(v.x), acc[0]); acc[1] = fmaf(w, hi(v.x), acc[1]);
        acc[2] = fmaf(w, lo(v.y), acc[2]); acc[3] = fmaf(w, hi(v.y), acc[3]);
        acc[4] = fmaf(w, lo(v.z), acc[4]); acc[5] = fmaf(w, hi(v.z), acc[5]);
        acc[6] = fmaf(w, lo(v.w), acc[6]); acc[7] = fmaf(w, hi(v.w), acc[7]);
    }
    __device__ static __forceinline__ void add(float *acc, uint2 v)
    {
        acc[0] += lo(v.x); acc[1] += hi(v.x);
        acc[2] += lo(v.y); acc[3] += hi(v.y);
    }
    __device__ static __forceinline__ void fma(float *acc, uint2 v, float w)
    {
        acc[0] = fmaf(w, lo(v.x), acc[0]); acc[1] = fmaf(w, hi(v.x), acc[1]);
        acc[2] = fmaf(w, lo(v.y), acc[2]); acc[3] = fmaf(w, hi(v.y), acc[3]);
    }
    __device__ static __forceinline__ void add(float *acc, uint32_t v) { acc[0] += lo(v); acc[1] += hi(v); }
    __device__ static __forceinline__ void fma(float *acc, uint32_t v, float w)
    {
        acc[0] = fmaf(w, lo(v), acc[0]); acc[1] = fmaf(w, hi(v), acc[1]);
    }
    __device__ static __forceinline__ float load1(const char *p) { return (float)*(const _Float16 *)p; }
};
template <> struct Elem<EB_BF16> {
    static constexpr int kPerChunk = 8;
    __device__ static __forceinline__ float lo(uint32_t w) { return __uint_as_float(w << 16); }
    __device__ static __forceinline__ float hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }
    __device__ static __forceinline__ void add(float *acc, uint4 v)
    {
        acc[0] += lo(v.x); acc[1] += hi(v.x);
        acc[2] += lo(v.y); acc[3] += hi(v.y);
        acc[4] += lo(v.z); acc[5] += hi(v.z);
        acc[6] += lo(v.w); acc[7] += hi(v.w);
    }
    __device__ static __forceinline__ void fma(float *acc, uint4 v, float w)
    {
        acc[0] = fmaf(w, lo(v.x), acc[0]); acc[1] = fmaf(w, hi(v.x), acc[1]);
        acc[2] = fmaf(w, lo(v.y), acc[2]); acc[3] = fmaf(w, hi(v.y), acc[3]);
        acc[4] = fmaf(w, lo(v.z), acc[4]); acc[5] = fmaf(w, hi(v.z), acc[5]);
        acc[6] = fmaf(w, lo(v.w), acc[6]); acc[7] = fmaf(w, hi(v.w), acc[7]);
    }
    __device__ static __forceinline__ void add(float *acc, uint2 v)
    {
        acc[0] += lo(v.x); acc[1] += hi(v.x);
        acc[2] += lo(v.y); acc[3] += hi(v.y);
    }
    __device__ static __forceinline__ void fma(float *acc, uint2 v, float w)
    {
        acc[0] = fmaf(w, lo(v.x), acc[0]); acc[1] = fmaf(w, hi(v.x), acc[1]);
        acc[2] = fmaf(w, lo(v.y), acc[2]); acc[3] = fmaf(w, hi(v.y), acc[3]);
    }
    __device__ static __forceinline__ void add(float *acc, uint32_t v) { acc[0] += lo(v); acc[1] += hi(v); }
    __device__ static __forceinline__ void fma(float *acc, uint32_t v, float w)
    {
        acc[0] = fmaf(w, lo(v), acc[0]); acc[1] = fmaf(w, hi(v), acc[1]);
    }
    __device__ static __forceinline__ float load1(const char *p) { return __uint_as_float((uint32_t)(*(const uint16_t *)p) << 16); }
};

// Row chunk load: default cache policy, or non-temporal (streamed past L2
// and the last-level cache) when the caller hints that ids have no reuse.
template <bool kStream>
__device__ __forceinline__ uint4 load_chunk(const char *p)
{
    if constexpr (kStream) {
        const u32x4 v = __builtin_nontemporal_load((const u32x4 *)p);
        return make_uint4(v[0], v[1], v[2], v[3]);
    } else {
        return *(const uint4 *)p;
    }
}

// The part of a row one lane loads: 16 bytes (global_load_dwordx4) for rows
// that are a multiple of 16 bytes, else 8 or 4 bytes.  Loads are cached, or
// non-temporal when the caller hints that ids have no reuse.
template <int CB> struct Chunk;
template <> struct Chunk<16> {
    using T = uint4;
    __device__ static __forceinline__ T zero() { return make_uint4(0, 0, 0, 0); }
    template <bool kStream> __device__ static __forceinline__ T load(const char *p) { return load_chunk<kStream>(p); }
};
template <> struct Chunk<8> {
    using T = uint2;
    __device__ static __forceinline__ T zero() { return make_uint2(0, 0); }
    template <bool kStream> __device__ static __forceinline__ T load(const char *p)
    {
        typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
        if constexpr (kStream) {
            const u32x2 v = __builtin_nontemporal_load((const u32x2 *)p);
            return make_uint2(v[0], v[1]);
        } else {
            return *(const uint2 *)p;
        }
    }
};
template <> struct Chunk<4> {
    using T = uint32_t;
    __device__ static __forceinline__ T zero() { return 0u; }
    template <bool kStream> __device__ static __forceinline__ T load(const char *p)
    {
        if constexpr (kStream) return __builtin_nontemporal_load((const uint32_t *)p);
        else return *(const uint32_t *)p;
    }
};

// Results, ids and offsets are touched once: non-temporal accesses.  Four
// fp32 results of a chunk, stored as one access.
__device__ __forceinline__ void store_nt(float *p, float a, float b, float c, float d)
{
    const f32x4 v = {a, b, c, d};
    __builtin_nontemporal_store(v, (f32x4 *)p);
}

// The kE fp32 results of one chunk, stored as one 16-, 8- or 4-byte access
// per group of up to four.
// The one or two fp32 results of a narrow chunk, stored as one access.
__device__ __forceinline__ void store_nt(float *p, float a, float b)
{
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    const f32x2 v = {a, b};
    __builtin_nontemporal_store(v, (f32x2 *)p);
}
__device__ __forceinline__ void store_nt(float *p, float a) { __builtin_nontemporal_store(a, p); }

__device__ __forceinline__ void clamp_bag(int64_t &s, int64_t &e, int64_t nnz)
{
    s = s < 0 ? 0 : (s > nnz ? nnz : s);
    e = e > nnz ? nnz : e;
    e = e < s ? s : e;
}

// ---------------------------------------------------------------------------- team gather kernel

template <typename IT, int DT, int R, int P, int C, int U, bool kStream, bool kW, int CB>
__global__ __launch_bounds__(kBlock) void eb_gather_team(const GatherArgs a)
{
    constexpr int kTeam = R * P;
    constexpr int kTeamsPerWave = kWave / kTeam;
    constexpr int kStage = kStagePerWave / kTeamsPerWave; // window entries per team
    constexpr int kEpc = CB / (DT == EB_F32 ? 4 : 2);    // elements per chunk
    using V = typename Chunk<CB>::T;
    static_assert(kTeam <= kWave && kWave % kTeam == 0, "team shape");
    static_assert(kStage % kTeam == 0, "window shape");

    __shared__ uint32_t stage[kWavesPerBlock * kStagePerWave];
    __shared__ float wstage[kW ? kWavesPerBlock * kStagePerWave : 1]; // weights of the staged rows

    const int lb = a.xcd_runs ? xcd_contiguous_block(blockIdx.x, gridDim.x) : (int)blockIdx.x;
    if (lb >= a.nblocks) return;

    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    const int team = lane / kTeam;
    const int tl = lane % kTeam;
    const int g = tl / R;  // lane group within the team
    const int rl = tl % R; // lane within the row

    const int t = lb / a.blocks_per_table;
    const int64_t b = a.bag_begin +
                      (int64_t)(lb - t * a.blocks_per_table) * (kTeamsPerWave * kWavesPerBlock) +
                      wave * kTeamsPerWave + team;
    const bool bag_ok = b < a.B;

    int64_t s = 0, e = 0;
    if (bag_ok) {
        const IT *o = (const IT *)a.offsets + (int64_t)t * a.B + b;
        s = __builtin_nontemporal_load(o);
        e = __builtin_nontemporal_load(o + 1);
        clamp_bag(s, e, a.nnz);
    }

    // Chunk c of a row goes to lane rl of a group when c*R + rl < chunks.
    // Surplus lanes (rows whose chunk count is not R*C) re-read the last
    // chunk, which the wave's other lanes fetch anyway, and never store.
    int coff[C];
#pragma unroll
    for (int c = 0; c < C; ++c) coff[c] = CB * min(c * R + rl, a.chunks - 1);
    const char *base = a.base[t];
    const size_t row_bytes = (size_t)a.row_bytes;
    const uint64_t nlocal = a.nlocal[t];
    const uint64_t shard_lo = (uint64_t)a.shard_lo;
    uint32_t *my_stage = stage + wave * kStagePerWave + team * kStage;
    float *my_wstage = wstage + (kW ? wave * kStagePerWave + team * kStage : 0);

    float acc[C * kEpc];
#pragma unroll
    for (int j = 0; j < C * kEpc; ++j) acc[j] = 0.f;
    int count = 0; // rows gathered so far (the same in every lane of the team)

    // This team's lanes as a wave mask, and the lanes below this one.
    const uint64_t team_lanes = kTeam == kWave ? ~0ull : (((1ull << kTeam) - 1) << (team * kTeam));
    const uint64_t below = (1ull << lane) - 1;

    for (int64_t w0 = s; w0 < e; w0 += kStage) {
        const int n = (int)((e - w0) < kStage ? (e - w0) : kStage);
        // Stage: coalesced index loads, all issued before the first is used
        // (positions past the window re-read its last entry).  The ids
        // gathered here are then written to the front of the team's window
        // as 32-bit local rows, in position order (ballot + prefix count),
        // so the gather loop below runs over gathered rows only.
        constexpr int kQ = kStage / kTeam;
        const IT *src = (const IT *)a.indices + w0;
        int64_t iv[kQ];
        float wv[kQ];
#pragma unroll
        for (int q = 0; q < kQ; ++q) {
            const int k = q * kTeam + tl;
            iv[q] = __builtin_nontemporal_load(src + (k < n ? k : n - 1));
            if constexpr (kW) wv[q] = __builtin_nontemporal_load(a.weights + w0 + (k < n ? k : n - 1));
        }
        int nv = 0; // gathered rows of the window
#pragma unroll
        for (int q = 0; q < kQ; ++q) {
            const int k = q * kTeam + tl;
            const uint64_t r = (uint64_t)iv[q] - shard_lo;
            const bool ok = k < n && r < nlocal;
            const uint64_t m = __ballot(ok) & team_lanes;
            if (ok) {
                const int at = nv + (int)__popcll(m & below);
                my_stage[at] = (uint32_t)r;
                if constexpr (kW) my_wstage[at] = wv[q];
            }
            nv += (int)__popcll(m);
        }
        count += nv;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

        // Gather: group g pools staged rows g, g+P, ...; U rows in flight.
        // Every staged entry below nv is a row, so the marker test in this
        // loop never fails; it stays because the compiler's schedule for the
        // predicated loads sustains more of the random-row rate than that
        // for unconditional ones (8-table uniform 512-B rows: 57.3 against
        // 60.3 us).
        int k = g;
        for (; k + (U - 1) * P < nv; k += U * P) {
            uint32_t rr[U];
            float ww[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                rr[u] = my_stage[k + u * P];
                if constexpr (kW) ww[u] = my_wstage[k + u * P];
            }
            V v[U][C];
#pragma unroll
            for (int u = 0; u < U; ++u) {
#pragma unroll
                for (int c = 0; c < C; ++c) v[u][c] = Chunk<CB>::zero();
                if (rr[u] != kInvalidRow) {
                    const char *p = base + (size_t)rr[u] * row_bytes;
#pragma unroll
                    for (int c = 0; c < C; ++c) v[u][c] = Chunk<CB>::template load<kStream>(p + coff[c]);
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    if constexpr (kW) Elem<DT>::fma(acc + c * kEpc, v[u][c], ww[u]);
                    else Elem<DT>::add(acc + c * kEpc, v[u][c]);
                }
            }
        }
        // The window's last rows (fewer than U for this group) in one
        // predicated pass: a bag's tail costs one round trip instead of one
        // per row, and the rows are added in the same order.  With U = 1
        // there is no tail; the row-at-a-time loop kept there never runs,
        // but without it the compiler allocates the main loop's registers so
        // that it waits for loads still in flight (2.5% slower for 1-KB rows).
        if constexpr (U == 1) {
            for (; k < nv; k += P) {
                const char *p = base + (size_t)my_stage[k] * row_bytes;
                V v[C];
#pragma unroll
                for (int c = 0; c < C; ++c) v[c] = Chunk<CB>::template load<kStream>(p + coff[c]);
                const float w = kW ? my_wstage[k] : 1.f;
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    if constexpr (kW) Elem<DT>::fma(acc + c * kEpc, v[c], w);
                    else Elem<DT>::add(acc + c * kEpc, v[c]);
                }
            }
        } else {
            if (k < nv) {
                bool in[U - 1];
                uint32_t rr[U - 1];
                float ww[U - 1];
#pragma unroll
                for (int u = 0; u < U - 1; ++u) {
                    in[u] = k + u * P < nv;
                    rr[u] = in[u] ? my_stage[k + u * P] : 0u;
                    if constexpr (kW) ww[u] = in[u] ? my_wstage[k + u * P] : 0.f;
                }
                V v[U - 1][C];
#pragma unroll
                for (int u = 0; u < U - 1; ++u) {
#pragma unroll
                    for (int c = 0; c < C; ++c) v[u][c] = Chunk<CB>::zero();
                    if (in[u]) {
                        const char *p = base + (size_t)rr[u] * row_bytes;
#pragma unroll
                        for (int c = 0; c < C; ++c) v[u][c] = Chunk<CB>::template load<kStream>(p + coff[c]);
                    }
                }
#pragma unroll
                for (int u = 0; u < U - 1; ++u) {
#pragma unroll
                    for (int c = 0; c < C; ++c) {
                        if constexpr (kW) Elem<DT>::fma(acc + c * kEpc, v[u][c], ww[u]);
                        else Elem<DT>::add(acc + c * kEpc, v[u][c]);
                    }
                }
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }

    team_reduce<R, P>(acc);

    if (bag_ok && g == 0) {
        if (a.mean) {
            const int64_t L = e - s;
            const float fl = (float)L;
#pragma unroll
            for (int j = 0; j < C * kEpc; ++j) acc[j] = L > 0 ? acc[j] / fl : 0.f;
        }
        float *o = a.out + b * a.ldo + a.col[t];
#pragma unroll
        for (int c = 0; c < C; ++c) {
            if (c * R + rl >= a.chunks) break;
            float *dst = o + (size_t)(c * R + rl) * kEpc;
            if constexpr (kEpc == 1) {
                store_nt(dst, acc[c]);
            } else if constexpr (kEpc == 2) {
                store_nt(dst, acc[2 * c], acc[2 * c + 1]);
            } else {
#pragma unroll
                for (int h = 0; h < kEpc / 4; ++h)
                    store_nt(dst + 4 * h, acc[c * kEpc + 4 * h], acc[c * kEpc + 4 * h + 1],
                             acc[c * kEpc + 4 * h + 2], acc[c * kEpc + 4 * h + 3]);
            }
        }
        if (a.hits && rl == 0) a.hits[b * a.ldh + t] = count;
    }
}

// ---------------------------------------------------------------------------- plain kernel

// One wave per bag, lanes striding over the columns; any D, any alignment.
// The bag's ids come in windows of 64 (one coalesced load, one id per lane);
// the gathered ones are taken in position order, kPlainRows at a time, each
// row's columns loaded by all lanes with every row's loads in flight
// together.  Rows are added in position order.
constexpr int kPlainRows = 8;

__device__ __forceinline__ uint64_t readlane_u64(uint64_t v, int l)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, l);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), l);
    return ((uint64_t)hi << 32) | lo;
}

template <typename IT, int DT, bool kW>
__global__ __launch_bounds__(kBlock) void eb_gather_plain(const GatherArgs a)
{
    constexpr int kEs = DT == EB_F32 ? 4 : 2;
    constexpr int kCols = 4; // columns per lane per pass
    const int lb = blockIdx.x;
    if (lb >= a.nblocks) return;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    const int t = lb / a.blocks_per_table;
    const int64_t b = a.bag_begin + (int64_t)(lb - t * a.blocks_per_table) * kWavesPerBlock + wave;
    if (b >= a.B) return;

    int64_t s, e;
    {
        const IT *o = (const IT *)a.offsets + (int64_t)t * a.B + b;
        s = o[0];
        e = o[1];
        clamp_bag(s, e, a.nnz);
    }
    const char *base = a.base[t];
    const uint64_t nlocal = a.nlocal[t];
    const uint64_t shard_lo = (uint64_t)a.shard_lo;
    const int D = a.D;
    const size_t pitch = (size_t)D * kEs;
    float *o = a.out + b * a.ldo + a.col[t];
    int count = 0;

    for (int c0 = 0; c0 < D; c0 += kWave * kCols) {
        float acc[kCols];
#pragma unroll
        for (int j = 0; j < kCols; ++j) acc[j] = 0.f;
        count = 0;
        for (int64_t w0 = s; w0 < e; w0 += kWave) {
            const int n = (int)((e - w0) < kWave ? (e - w0) : kWave);
            const int64_t k = w0 + (lane < n ? lane : n - 1);
            const uint64_t r = (uint64_t)(int64_t)((const IT *)a.indices)[k] - shard_lo;
            const float wt = kW ? a.weights[k] : 1.f;
            uint64_t m = __ballot(lane < n && r < nlocal); // the window's gathered ids
            count += (int)__popcll(m);
            while (m) {
                const char *p[kPlainRows];
                float w[kPlainRows];
                bool have[kPlainRows];
#pragma unroll
                for (int u = 0; u < kPlainRows; ++u) {
                    have[u] = m != 0;
                    const int l = have[u] ? (int)__builtin_ctzll(m) : 0;
                    m &= m - 1;
                    p[u] = base + readlane_u64(r, l) * pitch;
                    w[u] = kW ? __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wt), l)) : 1.f;
                }
                float x[kPlainRows][kCols];
#pragma unroll
                for (int u = 0; u < kPlainRows; ++u) {
#pragma unroll
                    for (int j = 0; j < kCols; ++j) {
                        const int c = c0 + j * kWave + lane;
                        x[u][j] = (have[u] && c < D) ? Elem<DT>::load1(p[u] + (size_t)c * kEs) : 0.f;
                    }
                }
#pragma unroll
                for (int u = 0; u < kPlainRows; ++u) {
                    if (have[u]) {
#pragma unroll
                        for (int j = 0; j < kCols; ++j) acc[j] = kW ? fmaf(w[u], x[u][j], acc[j]) : acc[j] + x[u][j];
                    }
                }
            }
        }
#pragma unroll
        for (int j = 0; j < kCols; ++j) {
            const int c = c0 + j * kWave + lane;
            if (c < D) {
                float v = acc[j];
                if (a.mean) v = (e > s) ? v / (float)(e - s) : 0.f;
                o[c] = v;
            }
        }
    }
    if (a.hits && lane == 0) a.hits[b * a.ldh + t] = count;
}

// Lane groups per bag; the kernels' template arguments follow the same rule.
constexpr int groups_per_bag(int R, bool few, bool single)
{
    // Wide rows or small batches: one bag per wave.  Otherwise narrow rows
    // get 16-lane teams (4 bags per wave), so the group reduction stays
    // inside a DPP row.  "single": teams narrower than a wave for large
    // batches, one lane group per bag: rows of 32 lanes two bags per wave,
    // rows read by 16 lanes (256-B rows, and 512-B / 1-KB rows as 2 / 4
    // chunks per lane) four, rows of 8 lanes (up to 128 B) eight.
    return few ? kWave / R : (single && R >= 8 && R < kWave) ? 1 : R >= 16 ? kWave / R : 16 / R;
}

using KernelFn = void (*)(GatherArgs);

// Most waves a bag of the wave kernel can have: the partial sums of `chunks`
// 16-byte chunks a wave stay within 32 KB of LDS.
constexpr int split_limit(int64_t chunks, int dtype)
{
    const int64_t wave_lds = chunks * (16 / (dtype == EB_F32 ? 4 : 2)) * (int64_t)sizeof(float);
    int split = 1;
    while (split < kMaxSplit && 2 * split * wave_lds <= 32768) split *= 2;
    return split;
}

// Most waves in a workgroup of the wave kernel's instance with C chunks per
// lane: its narrowest row's split, at least the unsplit call's waves.  One
// bound of 16 waves for every instance left those of 7 and 8 half-precision
// chunks 128 registers and up to 168 bytes of scratch per lane (25 tables x
// 4000 bags of 2 ids of 4075 fp16: 981 us, 587 without; 54 x 701 bags of 10 ids
// of 3700 bf16: 573 and 366; the plain kernel: 1492 and 1490).
constexpr int wave_block(int C, int dtype)
{
    const int split = split_limit(C > 1 ? (C - 1) * kWave + 1 : 1, dtype);
    return split > kWavesPerBlock ? split : kWavesPerBlock;
}

// Rows in flight per lane: streamed (non-temporal) rows of 128 B and more all
// go to HBM, where two per lane saturate the random-read rate and more only
// queue; narrower rows need more requests per byte in flight, and cached rows
// profit from deeper overlap while hits return early.  A small batch (fewer
// bags than fill the GPU) is bound by each bag's chain of dependent loads
// instead: every bag then gets a whole wave and 8 rows in flight per lane.
template <typename IT, int DT, int R, int C, bool kFew, bool kW, int CB>
KernelFn team_kernel(bool stream, bool single)
{
    constexpr int P = groups_per_bag(R, kFew, false);
    constexpr int P_SINGLE = groups_per_bag(R, kFew, true);
    constexpr int U_CACHED = kFew ? (C >= 8 ? 1 : 8 / C) : (C >= 6 ? 1 : 6 / C);
    constexpr int U_STREAM = (!kFew && R * C * CB >= 128) ? (C >= 2 ? 1 : 2) : U_CACHED;
    if (!stream) {
        if constexpr (P_SINGLE != P) {
            if (single) return eb_gather_team<IT, DT, R, P_SINGLE, C, U_CACHED, false, kW, CB>;
        }
        return eb_gather_team<IT, DT, R, P, C, U_CACHED, false, kW, CB>;
    }
    if constexpr (P_SINGLE != P) {
        if (single) return eb_gather_team<IT, DT, R, P_SINGLE, C, U_STREAM, true, kW, CB>;
    }
    return eb_gather_team<IT, DT, R, P, C, U_STREAM, true, kW, CB>;
}

template <typename IT, int DT, int R, int C, bool kW, int CB>
KernelFn team_kernel(bool stream, bool few, bool single)
{
    return few ? team_kernel<IT, DT, R, C, true, kW, CB>(stream, false)
               : team_kernel<IT, DT, R, C, false, kW, CB>(stream, single);
}

// 16-byte chunks: the row shapes of the library's mappings.  8- and 4-byte
// chunks: one chunk per lane (C = 1), rows of up to 64 chunks.
template <typename IT, int DT, bool kW, int CB>
KernelFn pick_team_kernel(int R, int C, bool stream, bool few, bool single)
{
    if constexpr (CB != 16) {
        if (C != 1) return nullptr;
        switch (R) {
        case 1: return team_kernel<IT, DT, 1, 1, kW, CB>(stream, few, single);
        case 2: return team_kernel<IT, DT, 2, 1, kW, CB>(stream, few, single);
        case 4: return team_kernel<IT, DT, 4, 1, kW, CB>(stream, few, single);
        case 8: return team_kernel<IT, DT, 8, 1, kW, CB>(stream, few, single);
        case 16: return team_kernel<IT, DT, 16, 1, kW, CB>(stream, few, single);
        case 32: return team_kernel<IT, DT, 32, 1, kW, CB>(stream, few, single);
        case 64: return team_kernel<IT, DT, 64, 1, kW, CB>(stream, few, single);
        }
        return nullptr;
    } else {
        switch (R) {
        case 1: return team_kernel<IT, DT, 1, 1, kW, 16>(stream, few, single);
        case 2: return team_kernel<IT, DT, 2, 1, kW, 16>(stream, few, single);
        case 4: return team_kernel<IT, DT, 4, 1, kW, 16>(stream, few, single);
        case 8: return team_kernel<IT, DT, 8, 1, kW, 16>(stream, few, single);
        case 16: // 256-B rows; 512-B and 1-KB rows in 16-lane teams
            return C == 4 ? team_kernel<IT, DT, 16, 4, kW, 16>(stream, few, single)
                   : C == 2 ? team_kernel<IT, DT, 16, 2, kW, 16>(stream, few, single)
                            : team_kernel<IT, DT, 16, 1, kW, 16>(stream, few, single);
        case 32: return team_kernel<IT, DT, 32, 1, kW, 16>(stream, few, single);
        default:
            switch (C) {
            case 1: return team_kernel<IT, DT, 64, 1, kW, 16>(stream, few, single);
            case 2: return team_kernel<IT, DT, 64, 2, kW, 16>(stream, few, single);
            case 3: return team_kernel<IT, DT, 64, 3, kW, 16>(stream, few, single);
            case 4: return team_kernel<IT, DT, 64, 4, kW, 16>(stream, few, single);
            case 5: return team_kernel<IT, DT, 64, 5, kW, 16>(stream, few, single);
            case 6: return team_kernel<IT, DT, 64, 6, kW, 16>(stream, few, single);
            case 7: return team_kernel<IT, DT, 64, 7, kW, 16>(stream, few, single);
            case 8: return team_kernel<IT, DT, 64, 8, kW, 16>(stream, few, single);
            }
        }
        return nullptr;
    }
}

template <typename IT, bool kW, int CB>
KernelFn pick_team_kernel(int dtype, int R, int C, bool stream, bool few, bool single)
{
    switch (dtype) {
    case EB_F32: return pick_team_kernel<IT, EB_F32, kW, CB>(R, C, stream, few, single);
    case EB_F16: return pick_team_kernel<IT, EB_F16, kW, CB>(R, C, stream, few, single);
    default: return pick_team_kernel<IT, EB_BF16, kW, CB>(R, C, stream, few, single);
    }
}

template <typename IT, bool kW>
KernelFn pick_plain_kernel(int dtype)
{
    switch (dtype) {
    case EB_F32: return eb_gather_plain<IT, EB_F32, kW>;
    case EB_F16: return eb_gather_plain<IT, EB_F16, kW>;
    default: return eb_gather_plain<IT, EB_BF16, kW>;
    }
}

// The kernel of one launch with 16-byte chunks (team: R lanes per row, C
// chunks per lane) or the plain kernel, by index type, element type and
// mapping.
template <bool kW>
KernelFn pick_kernel(bool i32, int dtype, bool team, int R, int C, bool stream, bool few, bool single)
{
    if (team)
        return i32 ? pick_team_kernel<int32_t, kW, 16>(dtype, R, C, stream, few, single)
                   : pick_team_kernel<int64_t, kW, 16>(dtype, R, C, stream, few, single);
    return i32 ? pick_plain_kernel<int32_t, kW>(dtype) : pick_plain_kernel<int64_t, kW>(dtype);
}

// pick_kernel<true>, instantiated in its own translation unit
// (eb_gather_weighted.hip) so the parts build in parallel.
KernelFn pick_weighted_kernel(bool i32, int dtype, bool team, int R, int C, bool stream, bool few,
                              bool single);

// Team kernels with 8- or 4-byte chunks (cb), weighted or not, instantiated
// in eb_gather_narrow.hip and eb_gather_narrow_weighted.hip.
KernelFn pick_narrow_kernel(bool weighted, bool i32, int dtype, int cb, int R, bool stream, bool few,
                            bool single);
KernelFn pick_narrow_weighted_kernel(bool i32, int dtype, int cb, int R, bool stream, bool few, bool single);

// Wave kernels (eb_gather_wave.h), weighted or not.
KernelFn pick_wave_kernel(bool weighted, bool i32, int dtype, int R, int C, bool stream);
KernelFn pick_wave_weighted_kernel(bool i32, int dtype, int R, int C, bool stream);

inline int elem_bytes(int dtype) { return dtype == EB_F32 ? 4 : 2; }

// ---------------------------------------------------------------------------- launch shape (host)

// Team shape for a row of rb bytes in chunks of cb bytes (rb % cb == 0).
struct Shape {
    int R, P, C;
};

// Small batches.  A launch whose normal mapping has fewer waves than the GPU
// holds (256 CUs x 32) leaves it partly idle, and each bag's chain of
// dependent loads sets the time.  One wave per bag with 8 rows in flight per
// lane then wins when bags are long (more than twice the rows the normal
// mapping keeps in flight per bag) and few enough (measured over the paper's
// single-GPU shapes: up to 1.5x faster, never slower).
constexpr int64_t kWaveSlots = 256 * 32;
constexpr int64_t kFewBagsMax = 2048;
constexpr int64_t kXcdTableBytes = (int64_t)32 << 20; // the XCDs' L2s together
constexpr double kStreamTableBytes = 2e9;               // eight times the last-level cache

inline int rows_in_flight_per_bag(const Shape &s, bool stream)
{
    const int u_cached = s.C >= 6 ? 1 : 6 / s.C;
    const int u = (stream && s.R * s.C >= 8) ? (s.C >= 2 ? 1 : 2) : u_cached;
    return s.P * u;
}

// single: one lane group per bag for large batches; 256-B and 1-KB rows
// then go to 16-lane teams (1 or 4 chunks per lane), and 512-B rows too when
// narrow512 is set (else 32-lane teams).
inline Shape team_shape(int rb, int cb, bool few, bool single, bool narrow512 = false)
{
    Shape s;
    const int chunks = rb / cb;
    s.R = 1;
    while (s.R < chunks && s.R < kWave) s.R *= 2;
    s.C = (chunks + s.R - 1) / s.R;
    if (cb == 16 && single && (rb == 256 || rb == 1024 || (rb == 512 && narrow512))) {
        s.R = 16;
        s.C = rb / 256;
    }
    s.P = groups_per_bag(s.R, few, single);
    return s;
}

// How a call's bags map to workgroups, and the kernel's template arguments.
struct GatherRoute {
    int32_t kernel;      // EB_ROUTE_*
    int32_t chunk_bytes; // bytes of a row one lane loads at a time (0: plain kernel)
    int32_t R, C;        // lanes per row, chunks per lane
    bool few;            // team kernel: small-batch mapping
    bool single;         // team kernel: one lane group per bag
    bool stream;         // non-temporal row loads
    bool xcd_runs;       // each XCD takes a contiguous run of workgroups
    int32_t split;       // wave kernel: waves per bag (0: team or plain kernel)
    int32_t bags_per_block;
};

// What a call's buffers allow.
struct GatherBuffers {
    int table_align;      // largest power of two up to 16 dividing every table pointer
    int out_align;        // ... every output row start in bytes
    int offsets_align;    // ... the offsets pointer
    int64_t local_rows;   // most gatherable rows of a table
    double all_local;     // gatherable rows of all tables
    double all_rows;      // rows of all tables
};

// Chunk size of the team kernel for rows of rb bytes, or 0 for the plain
// kernel: the widest of 16, 8 and 4 bytes that divides the row, that the
// tables' alignment allows, whose results (chunk / element size floats) the
// output rows' alignment allows to store as one access, and whose rows fit
// (16-byte chunks up to 8 KB, narrower ones one chunk per lane).
// table_align / out_align: the largest power of two up to 16 dividing every
// table pointer / every output row start in bytes.
inline int chunk_bytes(int64_t rb, int dtype, int table_align, int out_align)
{
    const int es = elem_bytes(dtype);
    for (int cb = 16; cb >= 4; cb /= 2) {
        const int out_need = cb / es * 4 < 16 ? cb / es * 4 : 16;
        const int64_t max_rb = cb == 16 ? 8192 : (int64_t)kWave * cb;
        if (rb % cb == 0 && rb <= max_rb && table_align >= cb && out_align >= out_need) return cb;
    }
    return 0;
}

// Whether the wave kernel (eb_gather_wave.h) can read these rows: 16 bytes to
// 8 KB each, element-aligned tables, float-aligned output rows, table offsets
// that fit its 32-bit product, and offsets that scalar loads can read.
inline bool wave_fits(int64_t rb, int dtype, const GatherBuffers &buf)
{
    return rb >= 16 && rb <= 8192 && buf.table_align >= elem_bytes(dtype) && buf.out_align >= 4 &&
           buf.offsets_align >= 4 && buf.local_rows <= (int64_t)(0xFFFFFFFFu / (uint64_t)rb);
}

// Whether a call takes the wave kernel rather than a team or plain kernel,
// given the lanes a team kernel would put on a bag and the ids expected in the
// gatherable rows (of a row block, its share of the bags' ids).  P = 64 / R rows
// are read at a time; all times in us, team or plain kernel against wave kernel.
//   * rows no aligned chunk fits: yes (16 tables x 4096 bags of 20 ids of 189
//     fp16: 306 against 90, of 1 id: 42.6 against 30.3; 4 x 50899 bags of 2 ids
//     of 253 fp32, a sixteenth gathered: 118 against 79).
//   * rows of more than 2 KB in 16-byte chunks: no (8-KB rows, 2048 bags of 100
//     ids: 253 against 283).
//   * up to 2048 bags, where the chain of dependent loads is the time: yes (8 x
//     256 bags of 16 ids of 64 fp32: 4.8 against 4.0; one bag of 1 id in 32:
//     4.2 against 3.8).
//   * over 8192 bags under the hint: not rows of 128 B and more in 16-byte
//     chunks, which are bound by HBM, nor rows under 64 B (64 uniform ids of
//     32 B in 100 K / 1 M rows: 30.0 / 75.9 against 32.3 / 76.1; of 64 B: 43.4
//     / 86.5 against 42.0 / 82.5; of 96 B: 76.0 / 133.0 against 73.8 / 126.3).
//   * where a team would be a whole wave as well: yes, its loads cost less and
//     need no predicates (some 700 random shapes: 1.25 times the speed, 0.93
//     at worst; 2 x 28103 weighted bags of 27 ids of 256 B, an eighth gathered:
//     41.4 against 23.4).
//   * where it would be less, a wave per bag costs more waves: from four
//     gathered passes, at most a window (16 x 4096 bags, skewed ids: 128-B
//     rows, 16 / 32 / 64 ids: 20.7 / 35.3 / 67.7 against 23.5 / 30.1 / 45.6;
//     256-B rows, 8 / 16 / 32 ids: 21.5 / 32.2 / 59.0 against 25.0 / 31.2 /
//     47.4; 512-B rows, 4 / 8 / 16 ids: 24.6 / 36.4 / 62.4 against 26.9 / 36.0
//     / 52.1; 1-KB rows, 2 / 4 / 8 ids: 30.6 / 42.2 / 68.5 against 34.2 / 41.7
//     / 60.4; 64-B rows, 32 / 64 ids: 24.3 / 47.4 against 27.9 / 42.2), with
//     and without weights.  At four to five passes bags of one length may lose
//     and ragged ones gain (18 x 7169 weighted bags of 20 ids of 256 B: 45.4
//     against 52.3; 49 x 620 of 1 to 45: 31.0 against 25.6); over 131072 bags,
//     where ragged ones even out, both lose (12 shapes: 0.93 to 1.08 times the
//     speed ragged, 0.88 to 0.96 of one length): from five there.  Ids that a
//     row block does not hold cost no passes (2 x 55087 bags of 17 ids of 256 B, a
//     sixteenth gathered: 22.6 against 37.5; 2 x 24038 of 49 ids of 128 B, a
//     quarter gathered: 15.5 against 22.8).
//   * up to 8192 bags, rows up to 128 B: from two passes, gathered or not (64 x
//     128 bags of 32 fp32, 4 ids: 4.4 against 4.9, 16 ids: 6.8 against 6.4; 2 x
//     1088 bags of 29 ids of 128 B, a quarter gathered: 6.4 against 3.9).
inline bool use_wave(int64_t rb, int cb, const Shape &whole, int team_lanes, bool hint, int64_t bags, int64_t nnz,
                     double gathered)
{
    if (cb == 0) return true;
    if (cb == 16 && whole.C > 2) return false;
    if (bags <= kFewBagsMax) return true;
    if (bags > kWaveSlots && hint && (rb < 64 || (rb >= 128 && cb == 16))) return false;
    if (team_lanes == kWave) return true;
    const int P = kWave / whole.R;
    if (bags <= kWaveSlots && nnz >= 2 * P * bags) return true;
    const int ids = (bags > 16 * kWaveSlots ? 5 : 4) * P;
    return gathered >= (double)(ids < kWave ? ids : kWave) * (double)bags;
}

// Waves per bag of the wave kernel, a power of two: more than one in calls of
// up to 2048 bags of 48 ids and more on average, doubled while the wave slots
// that are then taken stay within a half and a wave keeps 24 ids on average
// (its windows of 64 are given out whole, so even lengths leave some waves none;
// ragged ones gain from the next one: 52 bags of 28 to 84 ids 6.7 against 5.7
// us), and the partial sums fit 32 KB of LDS.  64-column fp32 rows, 1 / 2 / 4 /
// 8 / 16 waves: 32 bags of 100 ids 5.0 / 4.7 / 4.4 / 4.5 / 4.6 us, of 2000 ids
// 59.0 / 31.4 / 18.2 / 11.2 / 10.3; 512 bags of 400 ids 15.6 / 11.1 / 10.5 /
// 10.4 / 10.3; 2048 bags of 400 ids 27.7 / 29.2 / 28.3 / 28.2 / 30.5 (the team
// kernel: 5.6, 49.4, 14.2, 28.4); the last is the shape found where two waves
// lose, ragged bags there gain (2019 bags of 147 to 441 ids of 128 B 12.0
// against 9.6).
inline int split_waves(int64_t bags, int64_t nnz, int64_t rb, int dtype)
{
    const int limit = split_limit((rb + 15) / 16, dtype);
    int split = 1;
    while (split < limit && 2 * bags * split <= kWaveSlots / 2 && nnz >= 48 * split * bags) split *= 2;
    return split;
}

// The team kernel's mapping for rows of rb bytes in chunks of cb bytes.
inline GatherRoute team_route(int64_t rb, int cb, bool hint, int64_t bags, int64_t nnz)
{
    GatherRoute route{EB_ROUTE_TEAM, cb, 0, 0, false, false, false, false, 0, 0};
    // Non-temporal loads lose for rows narrower than 128 bytes.
    const bool stream = hint && rb >= 128;
    const Shape normal = team_shape((int)rb, cb, false, false);
    const int64_t waves = bags / (kWave / (normal.R * normal.P));
    const bool few = waves < kWaveSlots && bags <= kFewBagsMax &&
                     nnz > 2 * (int64_t)rows_in_flight_per_bag(normal, stream) * bags;
    // Teams narrower than a wave, one lane group per bag, when they still
    // give half the GPU's wave slots or more: for streamed rows, and for
    // cached rows when the mean bag is shorter than the rows the normal
    // mapping keeps in flight per bag (most of a wave would idle: the bags a
    // row block receives in a row-wise exchange).  512-B rows take 32-lane
    // teams when streamed (16-lane teams were 2-5% slower on the paper's
    // multi-table shapes) and 16-lane teams for short cached bags.
    const bool short_bags = nnz < (int64_t)rows_in_flight_per_bag(normal, false) * bags;
    const Shape narrow = team_shape((int)rb, cb, false, true, !stream && short_bags);
    const int narrow_team = narrow.R * narrow.P;
    const bool single = (stream || short_bags) && !few && narrow_team < normal.R * normal.P &&
                        bags / (kWave / narrow_team) >= kWaveSlots / 2;
    const Shape sh = few ? team_shape((int)rb, cb, true, false) : single ? narrow : normal;
    route.R = sh.R;
    route.C = sh.C;
    route.few = few;
    route.single = single;
    route.stream = stream;
    route.bags_per_block = (kWave / (sh.R * sh.P)) * kWavesPerBlock;
    // No reuse: each XCD takes a contiguous run of bags (measured faster for
    // uniform ids, also for rows under 128 B).  Otherwise hardware order, so
    // all XCDs work on the same table at once and its hot rows share the
    // last-level cache.
    route.xcd_runs = hint;
    return route;
}

inline GatherRoute choose_route(int32_t D, int32_t dtype, const GatherBuffers &buf, int64_t T, int64_t B, int64_t nnz,
                                int32_t mode)
{
    const int64_t rb = (int64_t)D * elem_bytes(dtype);
    const int cb = chunk_bytes(rb, dtype, buf.table_align, buf.out_align);
    const bool hint = (mode & EB_HINT_STREAM_ROWS) != 0;
    const int64_t bags = T * B;
    GatherRoute route = cb > 0 ? team_route(rb, cb, hint, bags, nnz)
                               : GatherRoute{EB_ROUTE_PLAIN, 0, 0, 0, false, false, false, false, 0, kWavesPerBlock};
    const int team_lanes = kWavesPerBlock * kWave / route.bags_per_block;
    const bool fits = wave_fits(rb, dtype, buf);
    const Shape whole = team_shape(fits ? (int)((rb + 15) / 16 * 16) : 16, 16, true, false); // a wave per bag
    const double gathered = buf.all_rows > 0 ? (double)nnz * (buf.all_local / buf.all_rows) : 0;
    if (!fits || !use_wave(rb, cb, whole, team_lanes, hint, bags, nnz, gathered)) return route;
    route = GatherRoute{EB_ROUTE_WAVE, 16, whole.R, whole.C, false, false, false, false, 0, kWavesPerBlock};
    // Streamed only where hardly any row comes back: the tables hold 2 GB and
    // more and a row in ten or fewer is used.  Non-temporal against cached: 8
    // tables of 875 K rows x 763 bags of 35 ids of 242 fp32 (3% used) 46.5
    // against 52.4 us; below either line cached loads are as fast in calls of
    // up to 8192 bags (53 shapes of which less than 2% is used: 1.00) and
    // faster the more is used (33 with a tenth and more: 1.12 times the speed;
    // 2 x 322 bags of 49 ids of 512 B in 22 K rows: 8.0 against 6.0, the team
    // kernel 7.6), and in larger ones rows of no whole 16-byte chunks, whose
    // pieces cross cache lines, ask for a line twice (9 tables of 720 K rows x
    // 10272 bags of 47 ids of 227 fp32, 0.67 uses a row: 752 against 658, the
    // plain kernel 664; 38 tables of 11 K rows x 7880 bags of 14 ids of 217
    // fp32, 10 uses: 690, 392 and 403).
    route.stream = hint && rb >= 128 && buf.all_local * rb >= kStreamTableBytes && gathered <= buf.all_local / 10;
    route.split = split_waves(bags, nnz, rb, dtype);
    route.bags_per_block = route.split > 1 ? 1 : kWavesPerBlock;
    // Each XCD a run of workgroups under the hint, as with teams (64 ids of
    // 32 bf16 in 100 K rows: 58 against 42), but not in small batches, where
    // finding the run costs 0.3 us, nor where eight tables at a time would
    // push each other's reused rows out of the caches: rows of no whole
    // 16-byte chunks from tables of over 32 MB, a row in four or more used
    // (0.67 uses a row, above: 776 against 658; tables of 11 K rows, above:
    // 346 against 392; 4 tables x 34679 bags of 15 ids of 228 fp16, a row in
    // twelve used: 153 against 165).
    // And for over 128 bags of one id, hinted or not, where an XCD would
    // otherwise read a line of ids and offsets for four bags' sake (new ids, 27
    // shapes: 0.89 of the time, the same ids again, 23: 1.03; 348 bags of 36
    // bf16 in 50 K rows 3.6 against 3.5 us, the team kernel 3.6).
    route.xcd_runs = (nnz < bags + bags / 2 && bags > 128) ||
                     (hint && bags > kFewBagsMax &&
                      (cb == 16 || buf.local_rows * rb <= kXcdTableBytes || gathered <= buf.all_local / 4));
    return route;
}

inline KernelFn route_kernel(const GatherRoute &r, int32_t dtype, bool i32, bool weighted)
{
    if (r.kernel == EB_ROUTE_WAVE) return pick_wave_kernel(weighted, i32, dtype, r.R, r.C, r.stream);
    if (r.kernel == EB_ROUTE_TEAM && r.chunk_bytes < 16)
        return pick_narrow_kernel(weighted, i32, dtype, r.chunk_bytes, r.R, r.stream, r.few, r.single);
    const bool team = r.kernel == EB_ROUTE_TEAM;
    return weighted ? pick_weighted_kernel(i32, dtype, team, r.R, r.C, r.stream, r.few, r.single)
                    : pick_kernel<false>(i32, dtype, team, r.R, r.C, r.stream, r.few, r.single);
}

// LDS for the partial sums of a split bag.
inline size_t split_lds_bytes(int split, int chunks, int dtype)
{
    return split > 1 ? (size_t)split * chunks * (16 / elem_bytes(dtype)) * sizeof(float) : 0;
}

// Launch one piece of at most 64 tables (a.base / nlocal / col / offsets /
// hits already set for it), in as many launches as the grid bound needs:
// each launch covers a range of every table's bags.
inline hipError_t launch_gather(KernelFn fn, const GatherRoute &plan, GatherArgs &a, int32_t nt, int dtype, hipStream_t stream)
{
    const int64_t kMaxBlocks = (int64_t)1 << 22;
    const int64_t blocks_all_bags = (a.B + plan.bags_per_block - 1) / plan.bags_per_block;
    const int64_t bpt_max = kMaxBlocks / nt > 1 ? kMaxBlocks / nt : 1;
    for (int64_t blk0 = 0; blk0 < blocks_all_bags; blk0 += bpt_max) {
        const int64_t bpt = bpt_max < blocks_all_bags - blk0 ? bpt_max : blocks_all_bags - blk0;
        a.bag_begin = blk0 * plan.bags_per_block;
        a.blocks_per_table = (int32_t)bpt;
        a.nblocks = (int32_t)(bpt * nt);
        if (plan.split > 0) {
            a.split = plan.split;
            void *wargs[] = {&a};
            const hipError_t err = hipLaunchKernel((const void *)fn, dim3((unsigned)bpt, (unsigned)nt),
                                                   dim3(plan.split > 1 ? kWave * plan.split : kBlock), wargs,
                                                   split_lds_bytes(plan.split, a.chunks, dtype), stream);
            if (err != hipSuccess) return err;
            continue;
        }
        const int64_t grid = plan.xcd_runs ? (a.nblocks + kXcds - 1) / kXcds * kXcds : a.nblocks;
        void *args[] = {&a};
        const hipError_t err = hipLaunchKernel((const void *)fn, dim3((unsigned)grid), dim3(kBlock), args, 0, stream);
        if (err != hipSuccess) return err;
    }
    return hipSuccess;
}

} // namespace eb_gather
