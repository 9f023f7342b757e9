// device_common.h - device-side building blocks shared by the GSP-Louvain
// kernels: degree bins, the sub-round hash, edge-weight loads, open-addressing
// tables keyed by community id (in LDS and in global memory), and
// wavefront-group reductions.  gfx950 (CDNA4), wave64.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gsp {

constexpr int kWave = 64;
constexpr int kBlock = 256;            // threads per block for every kernel here
constexpr int kEmpty = -1;             // empty table key (community ids are >= 0)
constexpr int kIntMax = 0x7fffffff;     // "no community" in an argmax

// Degree bins.  A vertex (or a community, for aggregation) with d entries is
// processed by:
//   d <= 4, 8, 16, 32, 64 : a group of 4/8/16/32/64 lanes, one entry per lane
//                           (local moving: a quarter of the lanes with up to
//                           four entries each), table of 2*group slots in LDS;
//   d <= 512              : one wavefront, table in LDS (1024 slots on unit
//                           weights, 768 otherwise);
//   d <= 2048             : one 256-thread workgroup, table in LDS (4096 slots
//                           on unit weights, 3072 otherwise);
//   d > 2048              : several workgroups, table of nextpow2(2d) slots in
//                           global memory ("hub").
// Every table is at most half full (the local-moving scan's wave and
// workgroup tables on weighted graphs two thirds), and every probe sequence
// goes over all of its slots, so a probe always ends.
constexpr int kNumBins = 8;
enum { BIN_G4 = 0, BIN_G8, BIN_G16, BIN_G32, BIN_G64, BIN_WAVE, BIN_BLOCK, BIN_HUB };
constexpr int kNumSmallBins = 5;
constexpr int kWaveMaxDeg = 512;
constexpr int kWaveTable = 1024;
constexpr int kBlockMaxDeg = 2048;
constexpr int kBlockTable = 4096;
constexpr int kHubChunk = 2048;        // entries per workgroup in the hub kernels

__host__ __device__ inline int bin_of_degree(int64_t d) {
    if (d <= 0) return -1;
    if (d <= 4) return BIN_G4;
    if (d <= 8) return BIN_G8;
    if (d <= 16) return BIN_G16;
    if (d <= 32) return BIN_G32;
    if (d <= 64) return BIN_G64;
    if (d <= kWaveMaxDeg) return BIN_WAVE;
    if (d <= kBlockMaxDeg) return BIN_BLOCK;
    return BIN_HUB;
}

__host__ __device__ inline uint64_t hub_table_size(int64_t d) {
    uint64_t t = 1;
    while (t < (uint64_t)(2 * d)) t <<= 1;
    return t;
}

// Sub-round of vertex i when an iteration has 2^shift ordered sub-rounds:
// the top `shift` bits of i * 0x9E3779B97F4A7C15 (Fibonacci hashing).
__host__ __device__ inline int sub_round_of(int64_t i, int shift) {
    if (shift == 0) return 0;
    uint64_t x = (uint64_t)i * 0x9E3779B97F4A7C15ull;
    return (int)(x >> (64 - shift));
}

enum WType { W_UNIT = 0, W_F32 = 1, W_F64 = 2 };

__device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & (kWave - 1)); }

template <int WT>
__device__ __forceinline__ double edge_weight(const void *w, int64_t e) {
    if constexpr (WT == W_UNIT) {
        return 1.0;
    } else if constexpr (WT == W_F32) {
        return (double)((const float *)w)[e];
    } else {
        return ((const double *)w)[e];
    }
}

__device__ __forceinline__ int32_t load_col(const int32_t *col, int64_t e) {
    return col[e];
}

__device__ __forceinline__ uint32_t key_hash(int32_t k) {
    uint32_t h = (uint32_t)k * 0x9E3779B1u;
    return h ^ (h >> 15);
}

// Probing.  Every table probes by double hashing: a key's step is 1, 7, 13,
// ... or 43, coprime to the table sizes 2^k and 3 2^k, from hash bits that
// its first slot does not depend on (a mask takes the low bits, a
// multiply-shift reduction the high ones).  With linear probing the keys
// pile up in runs, and 64 lanes wait for the longest: at two thirds full
// (R-MAT 24, the hub chunks' tables) 1.43 -> 1.28 ms per launch.
__device__ __forceinline__ int step_mask(uint32_t h) { return 1 + 6 * (int)(h >> 29); }
__device__ __forceinline__ int step_shift(uint32_t h) { return 1 + 6 * (int)(h & 7u); }

// Adds w to the value of `key` in an LDS table of mask+1 slots.
__device__ __forceinline__ void lds_table_add(int *keys, double *vals, uint32_t mask, int key, double w) {
    const uint32_t h = key_hash(key);
    uint32_t s = h & mask;
    while (true) {
        int prev = atomicCAS(&keys[s], kEmpty, key);
        if (prev == kEmpty || prev == key) {
            atomicAdd(&vals[s], w);
            return;
        }
        s = (s + step_mask(h)) & mask;
    }
}

// Slot of `key` in an LDS table of mask+1 slots (claimed if absent).
__device__ __forceinline__ int lds_table_slot(int *keys, uint32_t mask, int key) {
    const uint32_t h = key_hash(key);
    uint32_t s = h & mask;
    while (true) {
        int prev = atomicCAS(&keys[s], kEmpty, key);
        if (prev == kEmpty || prev == key) return (int)s;
        s = (s + step_mask(h)) & mask;
    }
}

// Puts a thread's entries (c[r], x[r]), r < R with c[r] != kEmpty, into a table
// in LDS (the threads of a wavefront or a workgroup together): `first` and
// `after` give a key's first slot and the one probed next.  The first
// compare-and-swaps of all R entries are issued together, then those that
// met another community probe on together.  Leaves the entries' slots in q
// and returns the mask of the entries that claimed theirs: their thread
// scores the community and clears the slot later (take_owned), so that nothing
// reads the empty slots.  (Scoring by a pass over the table's slots instead
// kept the LDS busy with them: a wavefront's table has 768 slots for 65 to
// 512 entries.)
template <int R, typename V, typename First, typename After>
__device__ __forceinline__ unsigned table_put_all(int *keys, V *vals, const int (&c)[R], const double (&x)[R],
                                                  int (&q)[R], First first, After after) {
    int prev[R];
#pragma unroll
    for (int r = 0; r < R; r++) {
        q[r] = first(c[r]);
        prev[r] = c[r];
        if (c[r] != kEmpty) prev[r] = atomicCAS(&keys[q[r]], kEmpty, c[r]);
    }
    bool more = true;
    while (more) {
        more = false;
#pragma unroll
        for (int r = 0; r < R; r++)
            if (prev[r] != kEmpty && prev[r] != c[r]) {
                q[r] = after(q[r], c[r]);
                prev[r] = atomicCAS(&keys[q[r]], kEmpty, c[r]);
                more = true;
            }
    }
    unsigned own = 0;
#pragma unroll
    for (int r = 0; r < R; r++)
        if (c[r] != kEmpty) {
            if (prev[r] == kEmpty) own |= 1u << r;
            atomicAdd(&vals[q[r]], (V)x[r]);
        }
    return own;
}

// Same on a table in global memory (device-scope atomics).
__device__ __forceinline__ void gbl_table_add(int *keys, double *vals, uint64_t mask, int key, double w) {
    uint64_t s = key_hash(key) & mask;
    while (true) {
        int prev = atomicCAS(&keys[s], kEmpty, key);
        if (prev == kEmpty || prev == key) {
            unsafeAtomicAdd(&vals[s], w);
            return;
        }
        s = (s + 1) & mask;
    }
}

// Partition of community c among P (high bits of a second mix, independent
// of the LDS slot hash).
__device__ __forceinline__ int part_of(int c, int P) {
    uint32_t h = (uint32_t)c;
    h ^= h >> 16;
    h *= 0x85EBCA6Bu;
    h ^= h >> 13;
    h *= 0xC2B2AE35u;
    h ^= h >> 16;
    return (int)(((uint64_t)h * (uint64_t)(uint32_t)P) >> 32);
}

// Exclusive scan of v[0..P) in place over a block of kBlock threads, v[P] =
// total: each thread sums a run of ceil(P / kBlock) entries, the run sums
// are scanned across each wavefront with shuffles and across the
// wavefronts through LDS, then each thread rewrites its run.
__device__ __forceinline__ void block_scan_excl(int *v, int P) {
    __shared__ int wtot[kBlock / kWave];
    const int tid = threadIdx.x, lane = tid % kWave, w = tid / kWave;
    const int per = (P + kBlock - 1) / kBlock;
    const int b0 = tid * per, b1 = b0 + per < P ? b0 + per : P;
    int sum = 0;
    for (int b = b0; b < b1; b++) sum += v[b];
    int inc = sum;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        int y = __shfl_up(inc, off, kWave);
        if (lane >= off) inc += y;
    }
    if (lane == kWave - 1) wtot[w] = inc;
    __syncthreads();
    int run = inc - sum, all = 0;
#pragma unroll
    for (int q = 0; q < kBlock / kWave; q++) {
        if (q < w) run += wtot[q];
        all += wtot[q];
    }
    for (int b = b0; b < b1; b++) {
        int x = v[b];
        v[b] = run;
        run += x;
    }
    if (tid == 0) v[P] = all;
    __syncthreads();
}

// Largest s in [0, n) with v[s] <= t (v non-decreasing, v[0] = 0 <= t).
__device__ __forceinline__ int last_le(const int *v, int n, int t) {
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (v[mid] <= t) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// Merges staged (key, value) pairs t = 0 .. total - 1 into a table of S slots
// in LDS, a workgroup together: pair t of the window lies at at(s, t), s the
// source with pst[s] <= t < pst[s + 1], s < nw.  *nkeys counts the distinct
// keys; past CAP of them *ovf is set and the workgroup stops (fewer than kBlock
// inserts are in flight then: CAP + kBlock < S keeps the table open).
// A thread takes four pairs at a time: their sources by one binary search in
// step, then their loads together, then the inserts (a pair at a time left
// one trip to memory per 256 pairs on the workgroup's path).
template <int S, int CAP, typename V, typename At>
__device__ __forceinline__ void merge_pairs(const int *pst, int nw, int total, const int32_t *skey,
                                            const double *sval, int *tkeys, V *tvals, int *nkeys, int *ovf, At at) {
    static_assert(CAP + kBlock < S, "the merge table never fills");
    constexpr int R = 4;
    int top = 1;
    while (2 * top < nw) top <<= 1;
    for (int t0 = threadIdx.x; t0 < total; t0 += R * kBlock) {
        int src[R], key[R];
        double v[R];
#pragma unroll
        for (int r = 0; r < R; r++) src[r] = 0;
        for (int step = top; step > 0; step >>= 1)
#pragma unroll
            for (int r = 0; r < R; r++)
                if (src[r] + step < nw && pst[src[r] + step] <= t0 + r * kBlock) src[r] += step;
#pragma unroll
        for (int r = 0; r < R; r++) {
            const int t = t0 + r * kBlock;
            key[r] = kEmpty;
            v[r] = 0.0;
            if (t < total) {
                const int64_t idx = at(src[r], t);
                key[r] = skey[idx];
                v[r] = sval[idx];
            }
        }
#pragma unroll
        for (int r = 0; r < R; r++) {
            if (key[r] == kEmpty || *(volatile int *)ovf) continue;
            const uint32_t h = key_hash(key[r]);
            constexpr bool kMask = (S & (S - 1)) == 0;
            int q = kMask ? (int)(h & (uint32_t)(S - 1)) : (int)(((uint64_t)h * (uint32_t)S) >> 32);
            const int step = kMask ? step_mask(h) : step_shift(h);
            while (true) {
                const int prev = atomicCAS(&tkeys[q], kEmpty, key[r]);
                if (prev == kEmpty && atomicAdd(nkeys, 1) >= CAP) *(volatile int *)ovf = 1;
                if (prev == kEmpty || prev == key[r]) break;
                q = q + step >= S ? q + step - S : q + step;
            }
            atomicAdd(&tvals[q], (V)v[r]);
        }
    }
}

// (g, c) beats (g2, c2): larger score, ties to the lower community id.
// Community ids are vertex ids of the level; on a level stored in degree
// order (orig != nullptr) they are compared as the caller's vertex ids,
// orig[c], which are read on exact ties only.
__device__ __forceinline__ bool better(double g, int c, double g2, int c2, const int32_t *orig) {
    if (g != g2) return g > g2;
    if (!orig || c == kIntMax || c2 == kIntMax) return c < c2;
    return orig[c] < orig[c2];
}

template <int W>
__device__ __forceinline__ double group_sum(double x) {
#pragma unroll
    for (int off = W / 2; off > 0; off >>= 1) x += __shfl_xor(x, off, W);
    return x;
}

template <int W>
__device__ __forceinline__ long long group_sum_ll(long long x) {
#pragma unroll
    for (int off = W / 2; off > 0; off >>= 1) x += __shfl_xor(x, off, W);
    return x;
}

// Maximum / minimum over the W lanes of an aligned lane group, every lane
// gets it; the group's lanes must all be active.  Within a row of 16 lanes
// the partners come by data-parallel primitives (the neighbour, the other
// pair, the mirrored half row, the mirrored row: each combines groups that
// already agree), across rows by the row and half swaps of gfx950: vector
// instructions throughout, where a shuffle goes through the LDS (an
// argmax with its sum over 64 lanes: 1230 cycles of shuffles).
template <int CTRL>
__device__ __forceinline__ int dpp_i32(int x) {
    return __builtin_amdgcn_update_dpp(x, x, CTRL, 0xF, 0xF, false);
}
constexpr int kDppPair = 0xB1, kDppQuad = 0x4E, kDppHalfRow = 0x141, kDppRow = 0x140;
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double x) {
    const uint64_t u = __builtin_bit_cast(uint64_t, x);
    const uint32_t lo = (uint32_t)dpp_i32<CTRL>((int)(uint32_t)u), hi = (uint32_t)dpp_i32<CTRL>((int)(u >> 32));
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
// x of the other row of a pair (HALF: of the other half of the wavefront)
// beside x, in some order.
template <bool HALF>
__device__ __forceinline__ void swap_rows(uint32_t x, uint32_t &a, uint32_t &b) {
    const auto r = HALF ? __builtin_amdgcn_permlane32_swap(x, x, false, false)
                        : __builtin_amdgcn_permlane16_swap(x, x, false, false);
    a = r[0];
    b = r[1];
}
template <bool HALF>
__device__ __forceinline__ double max_rows(double x) {
    const uint64_t u = __builtin_bit_cast(uint64_t, x);
    uint32_t la, lb, ha, hb;
    swap_rows<HALF>((uint32_t)u, la, lb);
    swap_rows<HALF>((uint32_t)(u >> 32), ha, hb);
    return fmax(__builtin_bit_cast(double, ((uint64_t)ha << 32) | la),
                __builtin_bit_cast(double, ((uint64_t)hb << 32) | lb));
}
template <bool HALF>
__device__ __forceinline__ int min_rows(int x) {
    uint32_t a, b;
    swap_rows<HALF>((uint32_t)x, a, b);
    return min((int)a, (int)b);
}
template <int W>
__device__ __forceinline__ double group_max(double x) {
    if constexpr (W >= 2) x = fmax(x, dpp_f64<kDppPair>(x));
    if constexpr (W >= 4) x = fmax(x, dpp_f64<kDppQuad>(x));
    if constexpr (W >= 8) x = fmax(x, dpp_f64<kDppHalfRow>(x));
    if constexpr (W >= 16) x = fmax(x, dpp_f64<kDppRow>(x));
    if constexpr (W >= 32) x = max_rows<false>(x);
    if constexpr (W >= 64) x = max_rows<true>(x);
    return x;
}
template <int W>
__device__ __forceinline__ int group_min(int x) {
    if constexpr (W >= 2) x = min(x, dpp_i32<kDppPair>(x));
    if constexpr (W >= 4) x = min(x, dpp_i32<kDppQuad>(x));
    if constexpr (W >= 8) x = min(x, dpp_i32<kDppHalfRow>(x));
    if constexpr (W >= 16) x = min(x, dpp_i32<kDppRow>(x));
    if constexpr (W >= 32) x = min_rows<false>(x);
    if constexpr (W >= 64) x = min_rows<true>(x);
    return x;
}

// Argmax over the W lanes of an aligned lane group (W power of two <= 64):
// every lane gets the largest g and, of the communities that reach it, the
// first in the order of `better`.
template <int W>
__device__ __forceinline__ void group_argmax(double &g, int &c, const int32_t *orig) {
    const double top = group_max<W>(g);
    const bool at = g == top && c != kIntMax;
    g = top;
    if (orig) {
        // on a level in degree order ties go by the caller's ids, read only
        // where some group has a tie
        unsigned long long m = __ballot(at);
        if (W < kWave) m = (m >> (lane_id() & ~(W - 1))) & ((1ull << (W & 63)) - 1ull);
        if (__any(__popcll(m) > 1)) {
            const int o = at ? orig[c] : kIntMax;
            const int first = group_min<W>(o);   // every lane takes part
            c = group_min<W>(at && o == first ? c : kIntMax);
            return;
        }
    }
    c = group_min<W>(at ? c : kIntMax);
}

// The same over groups of G lanes, G a runtime power of two, at most 16 and
// the same in the whole wavefront.
__device__ __forceinline__ double group_max_rt(double x, int G) {
    if (G >= 2) x = fmax(x, dpp_f64<kDppPair>(x));
    if (G >= 4) x = fmax(x, dpp_f64<kDppQuad>(x));
    if (G >= 8) x = fmax(x, dpp_f64<kDppHalfRow>(x));
    if (G >= 16) x = fmax(x, dpp_f64<kDppRow>(x));
    return x;
}
__device__ __forceinline__ int group_min_rt(int x, int G) {
    if (G >= 2) x = min(x, dpp_i32<kDppPair>(x));
    if (G >= 4) x = min(x, dpp_i32<kDppQuad>(x));
    if (G >= 8) x = min(x, dpp_i32<kDppHalfRow>(x));
    if (G >= 16) x = min(x, dpp_i32<kDppRow>(x));
    return x;
}
__device__ __forceinline__ void group_argmax_rt(double &g, int &c, int G, const int32_t *orig) {
    const double top = group_max_rt(g, G);
    const bool at = g == top && c != kIntMax;
    g = top;
    if (orig) {
        const unsigned long long m = (__ballot(at) >> (lane_id() & ~(G - 1))) & ((1ull << G) - 1ull);
        if (__any(__popcll(m) > 1)) {
            const int o = at ? orig[c] : kIntMax;
            const int first = group_min_rt(o, G);
            c = group_min_rt(at && o == first ? c : kIntMax, G);
            return;
        }
    }
    c = group_min_rt(at ? c : kIntMax, G);
}

// Wave-aggregated atomics keyed by an index: lanes of one wavefront that hit
// the same element are combined into one atomic (a popular community would
// otherwise serialise thousands of same-address atomics).  Lanes are taken
// one distinct key at a time; at most 64 rounds, so for few distinct keys.
__device__ __forceinline__ void wave_add_u64_by_key(unsigned long long *base, int key, unsigned long long val,
                                                    bool pred) {
    unsigned long long pending = __ballot(pred);
    while (pending) {
        int leader = __ffsll((long long)pending) - 1;
        int lk = __shfl(key, leader);
        bool mine = pred && key == lk && ((pending >> lane_id()) & 1ull);
        unsigned long long m = __ballot(mine);
        long long sum = mine ? (long long)val : 0;
#pragma unroll
        for (int off = kWave / 2; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
        if (lane_id() == leader) atomicAdd(&base[lk], (unsigned long long)sum);
        pending &= ~m;
    }
}

__device__ __forceinline__ void wave_add_f64_by_key(double *base, int key, double val, bool pred) {
    unsigned long long pending = __ballot(pred);
    while (pending) {
        int leader = __ffsll((long long)pending) - 1;
        int lk = __shfl(key, leader);
        bool mine = pred && key == lk && ((pending >> lane_id()) & 1ull);
        unsigned long long m = __ballot(mine);
        double sum = mine ? val : 0.0;
#pragma unroll
        for (int off = kWave / 2; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
        if (lane_id() == leader && sum != 0.0) unsafeAtomicAdd(&base[lk], sum);
        pending &= ~m;
    }
}

// Each lane with `pred` gets a distinct slot of cursor[key].
__device__ __forceinline__ int wave_reserve_by_key(int *cursor, int key, bool pred) {
    unsigned long long pending = __ballot(pred);
    int pos = -1;
    while (pending) {
        int leader = __ffsll((long long)pending) - 1;
        int lk = __shfl(key, leader);
        bool mine = pred && key == lk && ((pending >> lane_id()) & 1ull);
        unsigned long long m = __ballot(mine);
        int base = 0;
        if (lane_id() == leader) base = atomicAdd(&cursor[lk], __popcll(m));
        base = __shfl(base, leader);
        if (mine) pos = base + __popcll(m & ((1ull << lane_id()) - 1ull));
        pending &= ~m;
    }
    return pos;
}

// Wave-aggregated append: every lane with `pred` gets a distinct slot of
// counter *ctr; returns the slot (or -1).
__device__ __forceinline__ int wave_append(bool pred, int *ctr) {
    unsigned long long m = __ballot(pred);
    if (m == 0) return -1;
    int leader = __ffsll((long long)m) - 1;
    int base = 0;
    if (lane_id() == leader) base = atomicAdd(ctr, __popcll(m));
    base = __shfl(base, leader);
    unsigned long long below = m & ((1ull << lane_id()) - 1ull);
    return pred ? base + __popcll(below) : -1;
}

}  // namespace gsp
