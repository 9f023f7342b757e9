// k_util.hip - fills, device-wide exclusive scans, input validation, vertex
// weights (Section 3: K_i = sum_j w_ij) and the parts of modularity (Eq. 1).
#include <math.h>

#include <chrono>

#include "gsp_internal.h"

namespace gsp {

namespace {

constexpr int kScanItems = 8;
constexpr int kScanTile = kBlock * kScanItems;

inline unsigned grid_for(int64_t n, int64_t per_block, unsigned cap = 1u << 20) {
    int64_t g = (n + per_block - 1) / per_block;
    if (g < 1) g = 1;
    if (g > (int64_t)cap) g = cap;
    return (unsigned)g;
}

template <class T>
__global__ void __launch_bounds__(kBlock) k_fill(T *p, T v, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBlock) p[i] = v;
}

__global__ void __launch_bounds__(kBlock) k_iota(int32_t *p, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBlock)
        p[i] = (int32_t)i;
}

__global__ void __launch_bounds__(kBlock) k_copy_i32(int32_t *d, const int32_t *s, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBlock) d[i] = s[i];
}

// Exclusive scan of the 256 values of a block (one per thread); returns the
// exclusive prefix of this thread and sets *total.
template <class T>
__device__ T block_exclusive_scan(T x, T *total) {
    __shared__ T wsum[kBlock / kWave];
    int lane = lane_id(), w = threadIdx.x / kWave;
    T inc = x;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        T y = __shfl_up(inc, off);
        if (lane >= off) inc += y;
    }
    if (lane == kWave - 1) wsum[w] = inc;
    __syncthreads();
    T before = 0, all = 0;
#pragma unroll
    for (int k = 0; k < kBlock / kWave; k++) {
        if (k < w) before += wsum[k];
        all += wsum[k];
    }
    __syncthreads();
    *total = all;
    return before + inc - x;
}

template <class TIn, class TAcc>
__global__ void __launch_bounds__(kBlock) k_scan_tile_sums(const TIn *in, int64_t n, TAcc *bsum) {
    int64_t base = (int64_t)blockIdx.x * kScanTile;
    TAcc s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; k++) {
        int64_t i = base + (int64_t)k * kBlock + threadIdx.x;
        if (i < n) s += (TAcc)in[i];
    }
    TAcc tot;
    block_exclusive_scan<TAcc>(s, &tot);
    if (threadIdx.x == 0) bsum[blockIdx.x] = tot;
}

template <class TAcc>
__global__ void __launch_bounds__(kBlock) k_scan_block_sums(TAcc *bsum, int64_t nb) {
    TAcc carry = 0;
    for (int64_t base = 0; base < nb; base += kBlock) {
        int64_t i = base + threadIdx.x;
        TAcc x = i < nb ? bsum[i] : 0;
        TAcc tot;
        TAcc ex = block_exclusive_scan<TAcc>(x, &tot);
        if (i < nb) bsum[i] = carry + ex;
        carry += tot;
    }
    if (threadIdx.x == 0) bsum[nb] = carry;
}

template <class TIn, class TOut>
__global__ void __launch_bounds__(kBlock) k_scan_down(const TIn *in, TOut *out, int64_t n, const TOut *bsum,
                                                    int64_t nb) {
    int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
    TOut v[kScanItems];
    TOut s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; k++) {
        int64_t i = base + k;
        v[k] = i < n ? (TOut)in[i] : 0;
        s += v[k];
    }
    TOut tot;
    TOut ex = block_exclusive_scan<TOut>(s, &tot) + bsum[blockIdx.x];
#pragma unroll
    for (int k = 0; k < kScanItems; k++) {
        int64_t i = base + k;
        if (i < n) out[i] = ex;
        ex += v[k];
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) out[n] = bsum[nb];
}

template <class TIn, class TOut>
void scan_exclusive(const TIn *in, TOut *out, int64_t n, void *tmp, hipStream_t s) {
    int64_t nb = (n + kScanTile - 1) / kScanTile;
    if (nb < 1) nb = 1;
    TOut *bsum = (TOut *)tmp;
    k_scan_tile_sums<TIn, TOut><<<(unsigned)nb, kBlock, 0, s>>>(in, n, bsum);
    k_scan_block_sums<TOut><<<1, kBlock, 0, s>>>(bsum, nb);
    k_scan_down<TIn, TOut><<<(unsigned)nb, kBlock, 0, s>>>(in, out, n, bsum, nb);
}

__global__ void __launch_bounds__(kBlock) k_validate_offsets(const int64_t *off, int64_t n, int64_t nnz, int *err) {
    for (int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBlock) {
        int64_t a = off[i], b = off[i + 1];
        if (a > b || a < 0 || b > nnz || b - a > 0x7fffffffLL) atomicOr(err, 1);
    }
    if (blockIdx.x == 0 && threadIdx.x == 0)
        if (off[0] != 0 || off[n] != nnz) atomicOr(err, 1);
}

template <int WT>
__global__ void __launch_bounds__(kBlock) k_validate_entries(const int32_t *col, const void *w, int64_t n,
                                                            int64_t nnz, int *err) {
    int bad = 0;
    for (int64_t e = blockIdx.x * (int64_t)kBlock + threadIdx.x; e < nnz; e += (int64_t)gridDim.x * kBlock) {
        int32_t c = col[e];
        if (c < 0 || (int64_t)c >= n) bad |= 2;
        if constexpr (WT != W_UNIT) {
            double x = edge_weight<WT>(w, e);
            if (!(x >= 0.0) || isinf(x)) bad |= 4;
        }
    }
    if (bad) atomicOr(err, bad);
}

__global__ void __launch_bounds__(kBlock) k_offsets_from_i32(const int32_t *in, int64_t *out, int64_t n1) {
    for (int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x; i < n1; i += (int64_t)gridDim.x * kBlock)
        out[i] = (int64_t)in[i];
}

__global__ void __launch_bounds__(kBlock) k_degrees(const int64_t *off, int32_t *deg, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBlock)
        deg[i] = (int32_t)(off[i + 1] - off[i]);
}

__global__ void __launch_bounds__(kBlock) k_weights_to_f64(const float *in, double *out, int64_t nnz) {
    for (int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x; i < nnz; i += (int64_t)gridDim.x * kBlock)
        out[i] = (double)in[i];
}

// K_i = sum of row i, *M2 += sum_i K_i.  A wavefront takes 64 consecutive
// rows: each lane sums its own row if it has at most kShortRow entries (most
// rows of sparse graphs), then the wavefront sums the longer ones together,
// one at a time.  Sums of weights are exact (weight grid), so the order of
// the additions does not matter.  On a level in degree order the first
// g.nlong rows (the long ones, side by side) are left to
// launch_vertex_weights_long, which cuts them into equal entry chunks.
constexpr int kShortRow = 32;

template <int WT>
__global__ void __launch_bounds__(kBlock) k_vertex_weights(Level g, double *K, double *M2) {
    __shared__ double part[kBlock / kWave];
    const int lane = lane_id(), w = threadIdx.x / kWave;
    double blk = 0.0;
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    for (int64_t r0 = g.nlong + (int64_t)blockIdx.x * kBlock + w * kWave; r0 < g.n; r0 += stride) {
        const int64_t i = r0 + lane;
        int64_t b = 0, d = 0;
        if (i < g.n) {
            b = g.off[i];
            d = g.deg[i];   // rows may be gapped
        }
        double s = 0.0;
        const bool shortrow = d <= kShortRow;
        if (shortrow)
            for (int64_t k = b; k < b + d; k++) s += edge_weight<WT>(g.w, k);
        unsigned long long longs = __ballot(!shortrow);
        while (longs) {
            const int src = __ffsll((long long)longs) - 1;
            longs &= longs - 1;
            const int64_t lb = __shfl(b, src), ld = __shfl(d, src);
            double t = 0.0;
            for (int64_t k = lb + lane; k < lb + ld; k += kWave) t += edge_weight<WT>(g.w, k);
            t = group_sum<kWave>(t);
            if (lane == src) s = t;
        }
        if (i < g.n) K[i] = s;
        blk += group_sum<kWave>(s);
    }
    if (lane == 0) part[w] = blk;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int k = 0; k < kBlock / kWave; k++) t += part[k];
        unsafeAtomicAdd(M2, t);
    }
}

// The short rows of a level in degree order (rows [nlong, n), dense CSR):
// a workgroup takes 256 consecutive rows and reads their entries as one
// contiguous range, 256 at a time (coalesced), each thread finding its
// entry's row by a binary search over the rows' offsets in LDS and adding
// the weight to the row's LDS sum (exact sums, so the order of the atomics
// does not matter).
template <int WT>
__global__ void __launch_bounds__(kBlock) k_vertex_weights_rows(Level g, double *K, double *M2) {
    __shared__ int64_t so[kBlock + 1];
    __shared__ double acc[kBlock];
    __shared__ double part[kBlock / kWave];
    const int tid = threadIdx.x;
    double blk = 0.0;
    for (int64_t r0 = g.nlong + (int64_t)blockIdx.x * kBlock; r0 < g.n; r0 += (int64_t)gridDim.x * kBlock) {
        const int nr = g.n - r0 < kBlock ? (int)(g.n - r0) : kBlock;
        so[tid] = g.off[r0 + (tid < nr ? tid : nr)];
        if (tid == 0) so[kBlock] = g.off[r0 + nr];
        acc[tid] = 0.0;
        __syncthreads();
        const int64_t e0 = so[0], e1 = so[kBlock];
        const int lane = lane_id();
        for (int64_t eb = e0; eb < e1; eb += kBlock) {   // the same trip count in every lane
            const int64_t e = eb + tid;
            int r = -1;   // the row r with so[r] <= e < so[r + 1]
            double v = 0.0;
            if (e < e1) {
                int lo = 0, hi = nr - 1;
                while (lo < hi) {
                    const int mid = (lo + hi + 1) >> 1;
                    if (so[mid] <= e) lo = mid; else hi = mid - 1;
                }
                r = lo;
                v = edge_weight<WT>(g.w, e);
            }
            // consecutive lanes hold consecutive entries, so a row's entries
            // are a run of lanes: sum each run into its first lane (exact on
            // the grid's weights), which adds it to the row
#pragma unroll
            for (int o = 1; o < kWave; o <<= 1) {
                const double y = __shfl_down(v, o, kWave);
                const int ry = __shfl_down(r, o, kWave);
                if (lane + o < kWave && ry == r) v += y;
            }
            const int rp = __shfl_up(r, 1, kWave);
            if (r >= 0 && (lane == 0 || rp != r)) atomicAdd(&acc[r], v);
        }
        __syncthreads();
        if (tid < nr) {
            K[r0 + tid] = acc[tid];
            blk += acc[tid];
        }
        __syncthreads();
    }
    blk = group_sum<kWave>(blk);
    if (lane_id() == 0) part[tid / kWave] = blk;
    __syncthreads();
    if (tid == 0) {
        double t = 0.0;
        for (int k = 0; k < kBlock / kWave; k++) t += part[k];
        if (t != 0.0) unsafeAtomicAdd(M2, t);
    }
}

// Entry weight inside communities: out += w_ij over the entries (i, j) with
// memb[i] = memb[j], or out[gid[i]] += of a batch.  Rows are dense (an input
// graph, loaded or in degree order).
//
// What bounds it: the random gathers of memb[j].  A wavefront per row kept
// one gather per lane in flight and left most lanes idle on short rows; here
// a workgroup takes tiles of kInTile consecutive entries, whatever rows they
// belong to, sixteen entries per thread with all their gathers in flight.
// The row of each entry comes from the tile's row starts, marked in LDS (the
// first row is found by a 64-way search of the offsets) and filled in by a
// running maximum.  A workgroup walks consecutive tiles and flushes its sum
// at their end (batch: where the graph changes), as thousands of atomics on
// one address take longer than the tiles.  Measured: R-MAT 24 (520 M entries,
// fp32 weights, degree order) 13.3 -> 6.3 ms, R-MAT 22 in the loaded order
// 2.29 -> 1.34 ms, a road-like graph of 31 M entries 3.07 -> 0.63 ms.
constexpr int kInPer = 16;
constexpr int kInTile = kBlock * kInPer;
// A tile's rows are walked by its workgroup, empty ones among them; between
// two ranges of ids there may be any number of those, and beyond this many
// rows each entry searches the offsets for its own.  Measured on one tile of
// a path, microseconds of the whole call, walked / searched: 16,384 empty
// rows 109 / 124, 32,768 127 / 130, 65,536 160 / 127, 1M 1,170 / 144, 67M
// 110,500 / 996.
constexpr int64_t kInWalk = 8 * kInTile;

// Largest r in [0, n) with off[r] <= e (off[0] = 0 <= e); by a whole wavefront.
__device__ __forceinline__ int64_t wave_row_of(const int64_t *off, int64_t n, int64_t e) {
    int64_t lo = 0, len = n;
    while (len > 1) {
        const int64_t step = (len + kWave - 1) / kWave, at = lane_id() * step;
        const bool ok = at < len && off[lo + at] <= e;
        const int64_t k = __popcll(__ballot(ok)) - 1;
        lo += k * step;
        len = step < len - k * step ? step : len - k * step;
    }
    return lo;
}

template <int WT, bool BATCH>
__global__ void __launch_bounds__(kBlock) k_inside_weight(Level g, const int32_t *memb, int64_t tiles, double *out) {
    __shared__ __align__(16) int srow[kInTile];
    __shared__ int64_t sr[2];
    __shared__ int wmax[kBlock / kWave];
    __shared__ double part[kBlock / kWave];
    const int tid = threadIdx.x, lane = lane_id(), w = tid / kWave;
    const int64_t t0 = tiles * blockIdx.x / gridDim.x, t1 = tiles * (blockIdx.x + 1) / gridDim.x;
    double s = 0.0;
    int cur = -1;   // batch: the graph s belongs to
    auto flush = [&](double *to) {
        const double v = group_sum<kWave>(s);
        s = 0.0;
        if (lane == 0) part[w] = v;
        __syncthreads();
        if (tid == 0) {
            double t = 0.0;
            for (int k = 0; k < kBlock / kWave; k++) t += part[k];
            if (t != 0.0) unsafeAtomicAdd(to, t);
        }
        __syncthreads();
    };
    for (int64_t t = t0; t < t1; t++) {
        const int64_t e0 = t * kInTile, e1 = e0 + kInTile < g.nnz ? e0 + kInTile : g.nnz;
        int j[kInPer];
#pragma unroll
        for (int k = 0; k < kInPer; k++) {
            const int64_t e = e0 + k * kBlock + tid;
            j[k] = e < e1 ? load_col(g.col, e) : -1;
        }
        if (w < 2) {
            const int64_t r = wave_row_of(g.off, g.n, w == 0 ? e0 : e1 - 1);
            if (lane == 0) sr[w] = r;
        }
#pragma unroll
        for (int k = 0; k < kInPer; k++) srow[k * kBlock + tid] = 0;
        __syncthreads();
        const int64_t r0 = sr[0], r1 = sr[1];
        if (r1 - r0 <= kInWalk) {
            for (int64_t r = r0 + 1 + tid; r <= r1; r += kBlock) atomicMax(&srow[g.off[r] - e0], (int)(r - r0));
        } else {
            int64_t top = 1;
            while (2 * top <= r1 - r0) top *= 2;
#pragma unroll 1
            for (int k = 0; k < kInPer; k += 4) {   // four searches in step
                int64_t lo[4] = {r0, r0, r0, r0};
                for (int64_t step = top; step > 0; step >>= 1)
#pragma unroll
                    for (int q = 0; q < 4; q++)
                        if (lo[q] + step <= r1 && g.off[lo[q] + step] <= e0 + (k + q) * kBlock + tid) lo[q] += step;
#pragma unroll
                for (int q = 0; q < 4; q++) srow[(k + q) * kBlock + tid] = (int)(lo[q] - r0);
            }
        }
        int cj[kInPer];
#pragma unroll
        for (int k = 0; k < kInPer; k++) cj[k] = j[k] >= 0 ? memb[j[k]] : -1;
        __syncthreads();
        // running maximum: a thread's sixteen consecutive entries, then the
        // wavefront's lanes, then the wavefronts
        int m[kInPer];
        int run = 0;
#pragma unroll
        for (int q = 0; q < kInPer / 4; q++) {
            const int4 v = *reinterpret_cast<const int4 *>(&srow[tid * kInPer + 4 * q]);
            m[4 * q] = run = max(run, v.x);
            m[4 * q + 1] = run = max(run, v.y);
            m[4 * q + 2] = run = max(run, v.z);
            m[4 * q + 3] = run = max(run, v.w);
        }
        int inc = run;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const int y = __shfl_up(inc, o);
            if (lane >= o) inc = max(inc, y);
        }
        int before = __shfl_up(inc, 1);
        if (lane == 0) before = 0;
        if (lane == kWave - 1) wmax[w] = inc;
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kBlock / kWave - 1; q++)
            if (q < w) before = max(before, wmax[q]);
#pragma unroll
        for (int q = 0; q < kInPer / 4; q++)
            *reinterpret_cast<int4 *>(&srow[tid * kInPer + 4 * q]) =
                make_int4(max(before, m[4 * q]), max(before, m[4 * q + 1]), max(before, m[4 * q + 2]),
                          max(before, m[4 * q + 3]));
        __syncthreads();
        if constexpr (BATCH) {
            const int ga = g.gid[r0], gb = g.gid[r1];
            if (ga != gb) {   // several graphs in the tile: each wavefront adds graph by graph
                if (cur >= 0) flush(&out[cur]);
                cur = -1;
#pragma unroll
                for (int k = 0; k < kInPer; k++) {
                    const int64_t r = r0 + srow[k * kBlock + tid];
                    const bool in = j[k] >= 0 && memb[r] == cj[k];
                    const double v = in ? edge_weight<WT>(g.w, e0 + k * kBlock + tid) : 0.0;
                    wave_add_f64_by_key(out, g.gid[r], v, in);
                }
                __syncthreads();   // srow is rewritten by the next tile
                continue;
            }
            if (ga != cur) {
                if (cur >= 0) flush(&out[cur]);
                cur = ga;
            }
        }
#pragma unroll
        for (int k = 0; k < kInPer; k++) {
            const bool in = j[k] >= 0 && memb[r0 + srow[k * kBlock + tid]] == cj[k];
            if (in) s += edge_weight<WT>(g.w, e0 + k * kBlock + tid);
        }
        __syncthreads();   // srow is rewritten by the next tile
    }
    if (!BATCH)
        flush(out);
    else if (cur >= 0)
        flush(&out[cur]);
}

// *out += sum_c (Sigma_c / M2)^2 in fixed point: each term rounded to the
// nearest multiple of 2^-62 (the sum of the terms is at most 1), so the
// total is an exact integer sum, the same in any order of the atomics.
__global__ void __launch_bounds__(kBlock) k_sum_squares(const double *sig, int64_t n, double M2,
                                                       unsigned long long *out) {
    unsigned long long s = 0;
    for (int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBlock) {
        const double x = sig[i] / M2;
        s += (unsigned long long)(long long)rint(ldexp(x * x, 62));
    }
    s = (unsigned long long)group_sum_ll<kWave>((long long)s);
    if (lane_id() == 0 && s) atomicAdd(out, s);
}

// Weight grid (exact sums).  Non-negative doubles order like their bit
// patterns, so the largest weight is an atomic max over the bits.
template <int WT>
__global__ void __launch_bounds__(kBlock) k_weight_max(const void *w, int64_t nnz, unsigned long long *out) {
    double m = 0.0;
    for (int64_t e = blockIdx.x * (int64_t)kBlock + threadIdx.x; e < nnz; e += (int64_t)gridDim.x * kBlock) {
        const double x = edge_weight<WT>(w, e);
        m = x > m ? x : m;
    }
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) {
        const double o = __shfl_xor(m, off);
        m = o > m ? o : m;
    }
    if (lane_id() == 0 && m > 0.0) atomicMax(out, (unsigned long long)__double_as_longlong(m));
}

// *U += max(1, ceil(w 2^T)) over the positive weights: an exact integer
// bound of 2^T times the weight total (T chosen so that it stays below 2^63).
template <int WT>
__global__ void __launch_bounds__(kBlock) k_weight_bound(const void *w, int64_t nnz, int T, unsigned long long *U) {
    unsigned long long s = 0;
    for (int64_t e = blockIdx.x * (int64_t)kBlock + threadIdx.x; e < nnz; e += (int64_t)gridDim.x * kBlock) {
        const double x = edge_weight<WT>(w, e);
        if (!(x > 0.0)) continue;
        const double t = ceil(ldexp(x, T));
        s += t < 1.0 ? 1ull : (unsigned long long)t;
    }
    s = (unsigned long long)group_sum_ll<kWave>((long long)s);
    if (lane_id() == 0 && s) atomicAdd(U, s);
}

// w <- nearest multiple of 2^-S (ties to even), in place; *moved counts the
// weights that changed.  A weight rounded to a coarser grid needs no more
// significand bits than it had, so an fp32 weight stays exact in fp32.
template <int WT>
__global__ void __launch_bounds__(kBlock) k_weight_grid(void *w, int64_t nnz, int S, unsigned long long *moved) {
    unsigned long long c = 0;
    for (int64_t e = blockIdx.x * (int64_t)kBlock + threadIdx.x; e < nnz; e += (int64_t)gridDim.x * kBlock) {
        const double x = edge_weight<WT>(w, e);
        const double q = ldexp(rint(ldexp(x, S)), -S);
        if (q == x) continue;
        c++;
        if constexpr (WT == W_F32)
            ((float *)w)[e] = (float)q;
        else
            ((double *)w)[e] = q;
    }
    c = (unsigned long long)group_sum_ll<kWave>((long long)c);
    if (lane_id() == 0 && c) atomicAdd(moved, c);
}

__global__ void __launch_bounds__(kBlock) k_check_labels(const int32_t *memb, int64_t n, int *err) {
    int bad = 0;
    for (int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBlock)
        if (memb[i] < 0 || (int64_t)memb[i] >= n) bad = 1;
    if (bad) atomicOr(err, 1);
}

__global__ void __launch_bounds__(kBlock) k_post(PostArgs a, uint64_t *box) {
    uint64_t *o = box + kBoxHead;
#pragma unroll
    for (int r = 0; r < 4; r++) {
        const uint64_t *src = static_cast<const uint64_t *>(a.src[r]);
        for (int64_t k = threadIdx.x; k < a.n[r]; k += kBlock) o[k] = src[k];
        o += a.n[r];
    }
    box_post(box);
}

}  // namespace

void launch_fill_i32(int32_t *p, int32_t v, int64_t n, hipStream_t s) {
    if (n > 0) k_fill<int32_t><<<grid_for(n, kBlock * 4, 8192), kBlock, 0, s>>>(p, v, n);
}
void launch_fill_u8(uint8_t *p, uint8_t v, int64_t n, hipStream_t s) {
    if (n > 0) k_fill<uint8_t><<<grid_for(n, kBlock * 4, 8192), kBlock, 0, s>>>(p, v, n);
}
void launch_fill_f64(double *p, double v, int64_t n, hipStream_t s) {
    if (n > 0) k_fill<double><<<grid_for(n, kBlock * 4, 8192), kBlock, 0, s>>>(p, v, n);
}
void launch_fill_f32(float *p, float v, int64_t n, hipStream_t s) {
    if (n > 0) k_fill<float><<<grid_for(n, kBlock * 4, 8192), kBlock, 0, s>>>(p, v, n);
}
void launch_fill_u64(unsigned long long *p, unsigned long long v, int64_t n, hipStream_t s) {
    if (n > 0) k_fill<unsigned long long><<<grid_for(n, kBlock * 4, 8192), kBlock, 0, s>>>(p, v, n);
}
void launch_fill_i64(int64_t *p, int64_t v, int64_t n, hipStream_t s) {
    if (n > 0) k_fill<int64_t><<<grid_for(n, kBlock * 4, 8192), kBlock, 0, s>>>(p, v, n);
}
void launch_iota_i32(int32_t *p, int64_t n, hipStream_t s) {
    if (n > 0) k_iota<<<grid_for(n, kBlock * 4, 8192), kBlock, 0, s>>>(p, n);
}
void box_arm(uint64_t *box) { __atomic_store_n(box, (uint64_t)0, __ATOMIC_RELEASE); }
// Polling for at most 200 us: a result that takes longer gains nothing from it
// (the stream's wait adds about 10 us to it).
hipError_t box_wait(uint64_t *box, hipStream_t s) {
    const auto t0 = std::chrono::steady_clock::now();
    do {
        for (int k = 0; k < 64; k++) {
            if (__atomic_load_n(box, __ATOMIC_ACQUIRE)) return hipSuccess;
            __builtin_ia32_pause();
        }
    } while (std::chrono::steady_clock::now() - t0 < std::chrono::microseconds(200));
    hipError_t e = hipStreamSynchronize(s);
    if (e != hipSuccess) return e;
    return __atomic_load_n(box, __ATOMIC_ACQUIRE) ? hipSuccess : hipErrorUnknown;
}
hipError_t fetch_words(const PostArgs &a, uint64_t *box, hipStream_t s) {
    box_arm(box);
    k_post<<<1, kBlock, 0, s>>>(a, box);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? box_wait(box, s) : e;
}
hipError_t fetch_i64(const int64_t *src, int64_t *out, uint64_t *box, hipStream_t s) {
    PostArgs a;
    a.src[0] = src;
    a.n[0] = 1;
    hipError_t e = fetch_words(a, box, s);
    if (e == hipSuccess) *out = (int64_t)box[kBoxHead];
    return e;
}
void launch_copy_i32(int32_t *dst, const int32_t *src, int64_t n, hipStream_t s) {
    if (n > 0) k_copy_i32<<<grid_for(n, kBlock * 4, 8192), kBlock, 0, s>>>(dst, src, n);
}

size_t scan_tmp_bytes(int64_t n) { return (size_t)((n + kScanTile - 1) / kScanTile + 2) * sizeof(int64_t); }

void scan_exclusive_i32_to_i64(const int32_t *in, int64_t *out, int64_t n, void *tmp, hipStream_t s) {
    scan_exclusive<int32_t, int64_t>(in, out, n, tmp, s);
}
void scan_exclusive_i64(const int64_t *in, int64_t *out, int64_t n, void *tmp, hipStream_t s) {
    scan_exclusive<int64_t, int64_t>(in, out, n, tmp, s);
}
void scan_exclusive_i32(const int32_t *in, int32_t *out, int64_t n, void *tmp, hipStream_t s) {
    scan_exclusive<int32_t, int32_t>(in, out, n, tmp, s);
}

void launch_validate(const int64_t *off, const int32_t *col, const void *w, int wt, int64_t n, int64_t nnz,
                     int *err, hipStream_t s) {
    k_validate_offsets<<<grid_for(n, kBlock * 4, 8192), kBlock, 0, s>>>(off, n, nnz, err);
    if (nnz == 0) return;
    unsigned gr = grid_for(nnz, kBlock * 8, 16384);
    if (wt == W_UNIT)
        k_validate_entries<W_UNIT><<<gr, kBlock, 0, s>>>(col, w, n, nnz, err);
    else if (wt == W_F32)
        k_validate_entries<W_F32><<<gr, kBlock, 0, s>>>(col, w, n, nnz, err);
    else
        k_validate_entries<W_F64><<<gr, kBlock, 0, s>>>(col, w, n, nnz, err);
}

void launch_offsets_from_i32(const int32_t *in, int64_t *out, int64_t n1, hipStream_t s) {
    k_offsets_from_i32<<<grid_for(n1, kBlock * 4, 8192), kBlock, 0, s>>>(in, out, n1);
}

void launch_degrees(const int64_t *off, int32_t *deg, int64_t n, hipStream_t s) {
    if (n > 0) k_degrees<<<grid_for(n, kBlock * 4, 8192), kBlock, 0, s>>>(off, deg, n);
}

void launch_weights_to_f64(const float *in, double *out, int64_t nnz, hipStream_t s) {
    if (nnz > 0) k_weights_to_f64<<<grid_for(nnz, kBlock * 4, 16384), kBlock, 0, s>>>(in, out, nnz);
}

void launch_vertex_weights(const Level &g, double *K, double *M2, hipStream_t s) {
    if (g.n == 0) return;
    launch_vertex_weights_long(g, K, M2, s);
    if (g.nlong >= g.n) return;
    unsigned gr = grid_for(g.n - g.nlong, kBlock, 8192);
    if (g.orig) {   // degree order: dense rows of similar length side by side
        if (g.wt == W_UNIT)
            k_vertex_weights_rows<W_UNIT><<<gr, kBlock, 0, s>>>(g, K, M2);
        else if (g.wt == W_F32)
            k_vertex_weights_rows<W_F32><<<gr, kBlock, 0, s>>>(g, K, M2);
        else
            k_vertex_weights_rows<W_F64><<<gr, kBlock, 0, s>>>(g, K, M2);
        return;
    }
    if (g.wt == W_UNIT)
        k_vertex_weights<W_UNIT><<<gr, kBlock, 0, s>>>(g, K, M2);
    else if (g.wt == W_F32)
        k_vertex_weights<W_F32><<<gr, kBlock, 0, s>>>(g, K, M2);
    else
        k_vertex_weights<W_F64><<<gr, kBlock, 0, s>>>(g, K, M2);
}

void launch_inside_weight(const Level &g, const int32_t *memb, double *out, hipStream_t s) {
    if (g.n == 0 || g.nnz == 0) return;
    const int64_t tiles = (g.nnz + kInTile - 1) / kInTile;
    const unsigned gr = grid_for(tiles, 1, 2048);   // eight workgroups per CU
    auto go = [&](auto kernel) { kernel<<<gr, kBlock, 0, s>>>(g, memb, tiles, out); };
    if (g.gid)
        g.wt == W_UNIT ? go(k_inside_weight<W_UNIT, true>)
                       : g.wt == W_F32 ? go(k_inside_weight<W_F32, true>) : go(k_inside_weight<W_F64, true>);
    else
        g.wt == W_UNIT ? go(k_inside_weight<W_UNIT, false>)
                       : g.wt == W_F32 ? go(k_inside_weight<W_F32, false>) : go(k_inside_weight<W_F64, false>);
}

void launch_sum_squares(const double *sig, int64_t n, double M2, unsigned long long *out, hipStream_t s) {
    if (n > 0) k_sum_squares<<<grid_for(n, kBlock * 4, 4096), kBlock, 0, s>>>(sig, n, M2, out);
}

void launch_weight_max(const void *w, int wt, int64_t nnz, unsigned long long *out, hipStream_t s) {
    if (nnz == 0 || wt == W_UNIT) return;
    unsigned gr = grid_for(nnz, kBlock * 8, 8192);
    if (wt == W_F32)
        k_weight_max<W_F32><<<gr, kBlock, 0, s>>>(w, nnz, out);
    else
        k_weight_max<W_F64><<<gr, kBlock, 0, s>>>(w, nnz, out);
}

void launch_weight_bound(const void *w, int wt, int64_t nnz, int T, unsigned long long *U, hipStream_t s) {
    if (nnz == 0 || wt == W_UNIT) return;
    unsigned gr = grid_for(nnz, kBlock * 8, 8192);
    if (wt == W_F32)
        k_weight_bound<W_F32><<<gr, kBlock, 0, s>>>(w, nnz, T, U);
    else
        k_weight_bound<W_F64><<<gr, kBlock, 0, s>>>(w, nnz, T, U);
}

void launch_weight_grid(void *w, int wt, int64_t nnz, int S, unsigned long long *moved, hipStream_t s) {
    if (nnz == 0 || wt == W_UNIT) return;
    unsigned gr = grid_for(nnz, kBlock * 8, 8192);
    if (wt == W_F32)
        k_weight_grid<W_F32><<<gr, kBlock, 0, s>>>(w, nnz, S, moved);
    else
        k_weight_grid<W_F64><<<gr, kBlock, 0, s>>>(w, nnz, S, moved);
}

void launch_check_labels(const int32_t *memb, int64_t n, int *err, hipStream_t s) {
    if (n > 0) k_check_labels<<<grid_for(n, kBlock * 4, 8192), kBlock, 0, s>>>(memb, n, err);
}

}  // namespace gsp
