// Two-kernel bucketize, for up to 64 destinations and batches of a few million
// ids (part of eb_exchange.hip, which includes it inside its namespace).
//
// At these sizes count, scan and scatter spend their time on three to four
// dependent launches and on the counts' way through memory (82 K ids into 8
// blocks: 17.1 us; 2.6 M int32 ids: 32.2).  Here the first kernel only adds up
// every wave's ids per destination; in the second every workgroup adds up the
// totals of the workgroups before it, and its waves read their ids again (now
// in the L2s), place them, and write their bags' offsets from the same lane
// masks: 10.0 and 23.3 us (the kernels 3.6 + 6.2 and 6.8 + 16.9 under the
// profiler, which adds to each; the second is bound by vector issue, about 60
// instructions per 64 ids, and its start-up):
//   * a workgroup takes consecutive bags of one table and its waves even runs
//     of their ids, so that no wave waits for a long bag of another.  The
//     range comes by two scalar loads, so the ids are on their way before the
//     bags' offsets have arrived.
//   * lane g keeps destination g's running count.  Each 64-id chunk leaves, per
//     destination, the lanes it owns and the count before it in LDS; then a
//     lane per bag that starts in the wave's pass turns them into the bag's
//     offsets, so the rows are written in runs of bags.
//   * out-of-order offsets: the workgroup's waves share its bags and take them
//     one at a time, so the path needs no fallback.
// 4 waves per workgroup (8: 25.4, 16: 29.9 us for 2.6 M int32 ids at each
// one's best count of workgroups).
#pragma once

typedef int64_t i64x2 __attribute__((ext_vector_type(2)));

constexpr int kTwoWaves = 4;
constexpr int kTwoBlock = kTwoWaves * kWave;
constexpr int kTwoChunks = 8;             // 64-id chunks loaded together
constexpr int kTwoMaxOwners = kWave;      // a lane per destination
constexpr int64_t kTwoMaxIds = (int64_t)1 << 28;
constexpr int kTwoMaxBags = kTwoBlock - 1; // bags of a workgroup: a thread per offset

struct TwoArgs {
    const int64_t *bounds;  // [T][G+1]
    const void *indices;    // IT [nnz]
    const void *offsets;    // IT [T*B+1]
    int64_t *out_offsets;   // [G][T*B+1]
    void *out_indices;      // IT [out_cap]
    int64_t *segments;      // [G+1]
    int64_t *group_totals;  // [workgroups][kOwners]
    uint32_t *wave_before;  // [workgroups][waves][kOwners] (ordinary offsets)
    int64_t out_cap;
    int64_t nnz;
    int64_t B;
    int64_t TB;
    int32_t G;
    int32_t bags;             // per workgroup
    int32_t groups_per_table;
};

using eb_detail::scalar_load;

// The chunk's lanes by owner.  kOwners: 8 (3-bit compare tree), 16 (by pairs
// of blocks), 32 and 64 (binary search within the eighths).
template <int kOwners>
struct TwoOwners {
    static constexpr int kBits = kOwners == 8 ? 3 : kOwners == 16 ? 4 : kOwners == 32 ? 5 : 6;
    FewBounds fb;    // 8: the bounds; 32, 64: the eighths'
    TreeBounds tb;   // 16
    const int64_t *bnd;
    int G;
    uint32_t lbit[kBits]; // complements of the lane's bits as masks

    // b: the table's bounds in LDS (in memory for 8, read through the scalar cache)
    __device__ __forceinline__ TwoOwners(const int64_t *b, int g, int lane) : bnd(b), G(g)
    {
        if constexpr (kOwners == 8) {
            fb.lo = scalar_load(b);
            fb.hi = scalar_load(b + g);
#pragma unroll
            for (int j = 1; j < kFewShards; ++j) fb.inner[j - 1] = j < g ? scalar_load(b + min(j, g)) : INT64_MAX;
        }
        else if constexpr (kOwners == 16) tb = tree_bounds(b, g);
        else fb = eighth_bounds(b, g);
#pragma unroll
        for (int i = 0; i < kBits; ++i) lbit[i] = (uint32_t)((lane >> i) & 1) - 1u;
    }

    // For the lanes of `in`: valid = the lanes whose id has an owner, own = the
    // lanes whose id belongs to destination `lane`; with kRank also this lane's
    // owner (times 4) and its id's rank among the chunk's ids for it.
    template <bool kRank>
    __device__ __forceinline__ void split(int64_t id, uint64_t in, uint64_t &valid, uint64_t &own, int &owner4, int &rank) const
    {
        uint64_t b[kBits];
        if constexpr (kOwners == 8) {
            const FewMasks o = few_owner_masks(fb, id, in);
            valid = o.valid;
            b[0] = o.b0, b[1] = o.b1, b[2] = o.b2;
            if constexpr (kRank) owner4 = few_bits<4>(o);
        } else if constexpr (kOwners == 16) {
            const TreeMasks o = tree_owner_masks(tb, id, in);
            valid = o.valid;
#pragma unroll
            for (int i = 0; i < kBits; ++i) b[i] = o.b[i];
            if constexpr (kRank) owner4 = tree_bits<4>(o);
        } else {
            const int g = owner_by_eighths(bnd, G, fb, id, in);
            valid = __ballot(g >= 0);
#pragma unroll
            for (int i = 0; i < kBits; ++i) b[i] = __ballot(g >= 0 && ((g >> i) & 1));
            if constexpr (kRank) owner4 = g >= 0 ? g * 4 : 0;
        }
        uint32_t own_lo = (uint32_t)valid, own_hi = (uint32_t)(valid >> 32);
        uint32_t same_lo = own_lo, same_hi = own_hi;
#pragma unroll
        for (int i = 0; i < kBits; ++i) {
            own_lo &= (uint32_t)b[i] ^ lbit[i];
            own_hi &= (uint32_t)(b[i] >> 32) ^ lbit[i];
            if constexpr (kRank) {
                const uint32_t n = lane_bit(~b[i]) ? ~0u : 0u;
                same_lo &= (uint32_t)b[i] ^ n;
                same_hi &= (uint32_t)(b[i] >> 32) ^ n;
            }
        }
        own = ((uint64_t)own_hi << 32) | own_lo;
        if constexpr (kRank) {
            rank = (int)__builtin_amdgcn_mbcnt_hi(same_hi, __builtin_amdgcn_mbcnt_lo(same_lo, 0u));
        }
    }
};

// A workgroup's bags [p0, p0 + nb), its id range [S, E) if their offsets are
// in order, and wave w's share [s, e) of it: whole 64-id chunks, as even as
// they go.  S and E come by scalar loads, so that a wave's ids are on their
// way before the bags' offsets have arrived.
template <typename IT>
struct TwoGroup {
    const IT *o;          // the bags' offsets
    const int64_t *bnd;   // the table's bounds
    int64_t p0, E, s, e;
    int nb;

    __device__ __forceinline__ TwoGroup(const TwoArgs &a, int wg, int w)
    {
        const int t = wg / a.groups_per_table;
        const int64_t b0 = (int64_t)(wg - t * a.groups_per_table) * a.bags;
        nb = (int)min<int64_t>(a.bags, a.B - b0);
        p0 = (int64_t)t * a.B + b0;
        o = (const IT *)a.offsets + p0;
        bnd = a.bounds + (int64_t)t * (a.G + 1);
        int64_t S = (int64_t)scalar_load(o);
        E = (int64_t)scalar_load(o + nb);
        clamp_bag(S, E, a.nnz);
        const int64_t chunks = (E - S + kWave - 1) / kWave;
        const int64_t per = (chunks + kTwoWaves - 1) / kTwoWaves * kWave;
        s = min<int64_t>(S + w * per, E);
        e = min<int64_t>(s + per, E);
    }
    // Wave w's share of the bags where the offsets are out of order.
    __device__ __forceinline__ void bag_share(int w, int &j0, int &j1) const
    {
        const int per = (nb + kTwoWaves - 1) / kTwoWaves;
        j0 = min(w * per, nb);
        j1 = min(j0 + per, nb);
    }
};

// The bags' first positions (and the last one's end) in LDS, and whether each
// wave's threads found them in order; published by the next barrier.
struct TwoStarts {
    int64_t at[kTwoBlock];
    int bad[kTwoWaves];
};

__device__ __forceinline__ int64_t clamp_offset(int64_t x, int64_t nnz) { return x < 0 ? 0 : x > nnz ? nnz : x; }

__device__ __forceinline__ void two_publish(TwoStarts &st, int nb, int64_t x, int64_t next, int64_t nnz, int lane, int wave)
{
    const int64_t c = clamp_offset(x, nnz);
    if ((int)threadIdx.x <= nb) st.at[threadIdx.x] = c;
    const uint64_t bad = __ballot(clamp_offset(next, nnz) < c);
    if (lane == 0) st.bad[wave] = bad != 0;
}

__device__ __forceinline__ bool two_ordered(const TwoStarts &st, int lane)
{
    return __ballot(st.bad[lane % kTwoWaves] != 0) == 0;
}

// Positions past the pass re-read its last id: no predicates, and every load
// issues before the first is used.
template <typename IT>
__device__ __forceinline__ void two_load(const TwoArgs &a, int64_t k0, int R, int lane, IT (&id)[kTwoChunks])
{
    const IT *src = (const IT *)a.indices + k0;
#pragma unroll
    for (int u = 0; u < kTwoChunks; ++u) id[u] = src[min(u * kWave + lane, R - 1)];
}

// Every load of the pass has to be issued above this point: the compiler
// would otherwise move each one down to the chunk that uses it, one round
// trip per chunk.
template <typename IT>
__device__ __forceinline__ void two_pin(IT (&id)[kTwoChunks])
{
    static_assert(kTwoChunks == 8, "operands below");
    asm volatile("" : "+v"(id[0]), "+v"(id[1]), "+v"(id[2]), "+v"(id[3]), "+v"(id[4]), "+v"(id[5]), "+v"(id[6]), "+v"(id[7]));
}

constexpr int kTwoPass = kTwoChunks * kWave;

__device__ __forceinline__ int two_left(int64_t k0, int64_t e)
{
    return __builtin_amdgcn_readfirstlane((int)min<int64_t>(e - k0, (int64_t)kTwoPass));
}

// Adds up destination `lane`'s ids of [s, e).
template <typename IT, int kOwners>
__device__ __forceinline__ int64_t two_count(const TwoArgs &a, const TwoOwners<kOwners> &owners, int64_t s, int64_t e, int lane)
{
    int64_t total = 0;
    for (int64_t k0 = s; k0 < e; k0 += kTwoPass) {
        const int R = two_left(k0, e);
        IT id[kTwoChunks];
        two_load<IT>(a, k0, R, lane, id);
        two_pin(id);
#pragma unroll
        for (int u = 0; u < kTwoChunks; ++u) {
            if (u * kWave >= R) break;
            uint64_t valid, own;
            int owner4, rank;
            owners.template split<false>((int64_t)id[u], lanes_below(R - u * kWave), valid, own, owner4, rank);
            total += __popcll(own);
        }
    }
    return total;
}

template <typename IT, int kOwners>
__device__ __forceinline__ int64_t two_count_bags(const TwoArgs &a, const TwoOwners<kOwners> &owners,
                                                  const TwoGroup<IT> &v, const TwoStarts &st, int w, int lane)
{
    int64_t total = 0;
    int j0, j1;
    v.bag_share(w, j0, j1);
    for (int j = j0; j < j1; ++j) total += two_count<IT>(a, owners, st.at[j], st.at[j + 1], lane);
    return total;
}

template <typename IT, int kOwners>
__global__ __launch_bounds__(kTwoBlock) void eb_two_totals(const TwoArgs a)
{
    __shared__ TwoStarts st;
    __shared__ int64_t bnd[kOwners + 1];
    __shared__ int64_t totals[kTwoWaves][kOwners];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const int wg = xcd_run_block(blockIdx.x, gridDim.x);
    const TwoGroup<IT> v(a, wg, wave);
    const int64_t x = (int64_t)v.o[min((int)threadIdx.x, v.nb)], next = (int64_t)v.o[min((int)threadIdx.x + 1, v.nb)];
    if (kOwners > 8) {
        if ((int)threadIdx.x <= a.G) bnd[threadIdx.x] = v.bnd[threadIdx.x];
        __syncthreads();
    }
    const TwoOwners<kOwners> owners(kOwners > 8 ? bnd : v.bnd, a.G, lane);
    int64_t total = two_count<IT>(a, owners, v.s, v.e, lane);
    two_publish(st, v.nb, x, next, a.nnz, lane, wave);
    if (lane < kOwners) totals[wave][lane] = total;
    __syncthreads();
    if (!two_ordered(st, lane)) {
        total = two_count_bags<IT>(a, owners, v, st, wave, lane);
        if (lane < kOwners) totals[wave][lane] = total;
        __syncthreads();
    }
    if (wave == 0 && lane < kOwners) { // destinations past G have no ids
        int64_t run = 0;
        for (int w = 0; w < kTwoWaves; ++w) {
            a.wave_before[((int64_t)wg * kTwoWaves + w) * kOwners + lane] = (uint32_t)run;
            run += totals[w][lane];
        }
        a.group_totals[(int64_t)wg * kOwners + lane] = run;
    }
}

// What a pass leaves of each of its chunks for the bags that start in it, per
// destination: the lanes whose id goes there, and the ids for it before the
// chunk (all of them: the lanes that read it may be the only active ones, so
// nothing is fetched from the destination's own lane then).
struct __align__(16) TwoRecord {
    uint32_t own_lo, own_hi;
    int64_t before;
};

// Where offsets are out of order: wave w takes its share of the bags one at a
// time, with 64-bit slots (overlapping bags may send more ids than there are).
template <typename IT, int kOwners>
__device__ void two_place_bags(const TwoArgs &a, const TwoOwners<kOwners> &owners, const TwoGroup<IT> &v, const TwoStarts &st,
                               int w, int lane, int64_t segment, int64_t slot)
{
    int64_t *out = a.out_offsets + (int64_t)lane * (a.TB + 1) + v.p0;
    int j0, j1;
    v.bag_share(w, j0, j1);
    for (int j = j0; j < j1; ++j) {
        if (lane < a.G) out[j] = slot - segment;
        const int64_t e = st.at[j + 1];
        for (int64_t k0 = st.at[j]; k0 < e; k0 += kWave) {
            const int n = (int)min<int64_t>(e - k0, kWave);
            const IT id = ((const IT *)a.indices)[k0 + min(lane, n - 1)];
            uint64_t valid, own;
            int owner4, rank;
            owners.template split<true>((int64_t)id, lanes_below(n), valid, own, owner4, rank);
            const int base_lo = __builtin_amdgcn_ds_bpermute(owner4, (int)(uint32_t)slot);
            const int base_hi = __builtin_amdgcn_ds_bpermute(owner4, (int)(slot >> 32));
            const int64_t pos = (((int64_t)base_hi << 32) | (uint32_t)base_lo) + rank;
            if (lane_bit(valid) && (uint64_t)pos < (uint64_t)a.out_cap) ((IT *)a.out_indices)[pos] = id;
            slot += __popcll(own);
        }
    }
    if (v.p0 + v.nb == a.TB && w == kTwoWaves - 1 && lane < a.G) out[v.nb] = slot - segment;
}

template <typename IT, int kOwners>
__global__ __launch_bounds__(kTwoBlock) void eb_two_place(const TwoArgs a)
{
    using Owners = TwoOwners<kOwners>;
    __shared__ TwoStarts st;
    __shared__ int64_t bnd[kOwners + 1];
    __shared__ int64_t sums[2][kTwoWaves][kOwners];
    __shared__ TwoRecord records[kTwoWaves][kTwoChunks][kOwners];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const int wg = xcd_run_block(blockIdx.x, gridDim.x);
    const int G = a.G;
    const TwoGroup<IT> v(a, wg, wave);
    const int64_t x = (int64_t)v.o[min((int)threadIdx.x, v.nb)], next = (int64_t)v.o[min((int)threadIdx.x + 1, v.nb)];
    int64_t before_wave = (int64_t)a.wave_before[((int64_t)wg * kTwoWaves + wave) * kOwners + min(lane, kOwners - 1)];
    if (kOwners > 8 && (int)threadIdx.x <= G) bnd[threadIdx.x] = v.bnd[threadIdx.x];
    IT id[kTwoChunks] = {};
    if (v.s < v.e) two_load<IT>(a, v.s, two_left(v.s, v.e), lane, id);
    // Thread i adds up two destinations over every (kTwoBlock / kPairs)-th
    // workgroup: those before this one, and all.
    {
        constexpr int kPairs = kOwners / 2, kStep = kTwoBlock / kPairs;
        const i64x2 *t = (const i64x2 *)a.group_totals + threadIdx.x;
        i64x2 before = {0, 0}, all = {0, 0};
#pragma unroll 8
        for (int i = threadIdx.x / kPairs; i < (int)gridDim.x; i += kStep, t += kTwoBlock) {
            const i64x2 n = *t;
            all += n;
            if (i < wg) before += n;
        }
        for (int m = kPairs; m < kWave; m <<= 1) {
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                before[k] += shfl_xor64(before[k], m);
                all[k] += shfl_xor64(all[k], m);
            }
        }
        if (lane < kPairs) {
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                sums[0][wave][2 * lane + k] = before[k];
                sums[1][wave][2 * lane + k] = all[k];
            }
        }
    }
    two_publish(st, v.nb, x, next, a.nnz, lane, wave);
    __syncthreads();
    int64_t before = 0, all = 0;
    if (lane < kOwners) {
#pragma unroll
        for (int i = 0; i < kTwoWaves; ++i) {
            before += sums[0][i][lane];
            all += sums[1][i][lane];
        }
    }
    const int64_t upto = wave_inclusive_scan(all, lane);
    const int64_t segment = upto - all;
    if (wg == 0 && wave == 0) {
        if (lane < G) a.segments[lane] = segment;
        if (lane == G - 1) a.segments[G] = upto;
    }
    const Owners owners(kOwners > 8 ? bnd : v.bnd, G, lane);
    // Other workgroups' overlapping bags may send more ids than the batch holds,
    // which moves this one's positions past 32 bits although its own offsets
    // are in order: it then takes its bags one at a time too.
    const bool ordered = two_ordered(st, lane) && readlane64(upto, kWave - 1) <= kTwoMaxIds;
    if (!ordered) {
        // Bags may overlap, so a wave's share may exceed what wave_before
        // holds: count again.
        const int64_t total = two_count_bags<IT>(a, owners, v, st, wave, lane);
        __syncthreads(); // every wave has read the sums
        if (lane < kOwners) sums[0][wave][lane] = total;
        __syncthreads();
        before_wave = 0;
        if (lane < kOwners)
            for (int i = 0; i < wave; ++i) before_wave += sums[0][i][lane];
    }
    const int64_t first = before + before_wave; // destination `lane`'s ids before the wave's
    if (!ordered) {
        two_place_bags<IT>(a, owners, v, st, wave, lane, segment, segment + first);
        return;
    }
    // At most kTwoMaxIds ids are sent, so 32 bits hold every position, and every
    // byte offset into out_indices.
    int slot = (int)(segment + first), start = slot;
    const uint32_t cap = (uint32_t)min<int64_t>(a.out_cap, kTwoMaxIds);
    const int64_t row = a.TB + 1;
    int64_t *out_off = a.out_offsets + v.p0;
    TwoRecord(*rec)[kOwners] = records[wave];
    // The first bag that starts in the wave's share.
    int j = 0;
    for (int i = 0; i < v.nb; i += kWave)
        j += (int)__popcll(__ballot(i + lane < v.nb && st.at[min(i + lane, v.nb)] < v.s));
    for (int64_t k0 = v.s; k0 < v.e; k0 += kTwoPass) {
        const int R = two_left(k0, v.e);
        if (k0 > v.s) two_load<IT>(a, k0, R, lane, id);
        two_pin(id);
        uint32_t pos[kTwoChunks];
#pragma unroll
        for (int u = 0; u < kTwoChunks; ++u) {
            pos[u] = ~0u;
            if (u * kWave >= R) continue;
            uint64_t valid, own;
            int owner4, rank;
            owners.template split<true>((int64_t)id[u], lanes_below(R - u * kWave), valid, own, owner4, rank);
            const int base = __builtin_amdgcn_ds_bpermute(owner4, slot);
            if (lane_bit(valid)) pos[u] = (uint32_t)(base + rank);
            if (lane < kOwners) rec[u][lane] = TwoRecord{(uint32_t)own, (uint32_t)(own >> 32), first + (slot - start)};
            slot += __popcll(own);
        }
        // The bags that start in the pass, a lane each.
        wave_sync_lds();
        while (j < v.nb) {
            const int64_t at = j + lane < v.nb ? st.at[j + lane] : INT64_MAX;
            const uint64_t here = __ballot(at < k0 + R);
            if (lane_bit(here)) {
                const int rel = (int)(at - k0);
                const uint64_t below = (1ull << (rel % kWave)) - 1;
                const TwoRecord *r = rec[rel / kWave];
                for (int g = 0; g < G; ++g) {
                    const TwoRecord x = r[g];
                    const int n = __popc(x.own_lo & (uint32_t)below) + __popc(x.own_hi & (uint32_t)(below >> 32));
                    out_off[(int64_t)g * row + j + lane] = x.before + n;
                }
            }
            j += (int)__popcll(here);
            if (here != ~0ull) break;
        }
        wave_sync_lds();
#pragma unroll
        for (int u = 0; u < kTwoChunks; ++u)
            if (pos[u] < cap) *(IT *)((char *)a.out_indices + (uint32_t)(pos[u] * (uint32_t)sizeof(IT))) = id[u];
    }
    // Empty bags at the end, and the end of the destinations' last rows.
    if (wave == kTwoWaves - 1 && lane < G) {
        const int64_t end = first + (slot - start);
        for (; j < v.nb; ++j) out_off[(int64_t)lane * row + j] = end;
        if (v.p0 + v.nb == a.TB) out_off[(int64_t)lane * row + v.nb] = end;
    }
}
