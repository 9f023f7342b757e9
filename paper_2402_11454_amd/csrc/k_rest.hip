// k_rest.hip - the rest of a run on small levels: once a run's level has at
// most kRestVertices vertices and rest_entries entries, one workgroup takes
// it through every remaining pass of Algorithm "louvain" (local moving, split,
// renumbering, the pass tests, aggregation) with the level's state in LDS.
//
// What bounds such levels otherwise: a sub-round of a few hundred vertices
// is two launches of 5 to 15 us whose kernels wait for seven or eight trips
// to memory one after another, a sweep ends with a host read, and a pass
// takes some forty launches and six host reads more (a 125-vertex level of
// 12,000 entries: 130 us per sweep, 0.7 ms per pass).  One workgroup has the
// memberships, totals and tables in LDS and separates its steps by barriers:
// 3.4 us per sub-round on that level (of them 2.8 the scans: about 1000
// cycles for the row's entries from memory, 1700 for the compare-and-swaps,
// which share one LDS) and 15 us for its split and aggregation.  Whole runs:
// 1,013 vertices 2.60 -> 0.54 ms, 10,000 vertices (the first level goes
// through the level-wide kernels) 3.80 -> 1.84 ms, 1.50 since.  The entries stay in
// memory, read once per scan; beyond rest_entries the one compute unit's rate
// costs more than the launches do, and beyond kRestVertices the state does
// not fit the LDS.
//
// The method is the same, step for step: the scores come from the same
// exactly rounded operations on exact sums, so memberships, iteration
// counts and counters equal those of the level-wide kernels.
#include "gsp_internal.h"

namespace gsp {

namespace {

constexpr int kT = 1024;                 // threads
constexpr int kWaves = kT / kWave;
constexpr int kN = kRestVertices;
constexpr int kSlots = 8192;             // table slots of the workgroup
constexpr int kWaveSlots = kSlots / kWaves;
// Rows by length: up to 32 entries eight lanes, up to 64 sixteen, up to kRowC
// a wavefront, each with eight table slots per lane (half full, the
// wavefront's two thirds); longer ones a wavefront with a dense table over
// the communities, which up to kWaveSlots of them every wavefront has (the
// shorter wavefront rows then take it too: no compare-and-swaps), beyond as
// many wavefronts as the pool has room for.
constexpr int kClasses = 4;
constexpr int kPerLane = 8;
constexpr int kRow8 = 32, kRow16 = 64, kRowC = kWaveSlots * 2 / 3;
static_assert(kWave * kPerLane == kWaveSlots, "a wavefront's tables");
constexpr int kLanes = 16;               // per row outside the scans
// Aggregation: dense rows of kDense doubles in all, presence bits beside.
constexpr int kDense = 8192;

struct Pool {   // scans: hash tables; split: parents; aggregation: dense rows
    double vals[kSlots];
    int keys[kSlots];
};
static_assert(kN <= kSlots && kDense <= kSlots && kRestDense <= kWaveSlots, "pool views");

struct State {
    Pool pool;
    double sig[kN], K[kN];
    uint32_t rowb[kN];         // first entry of the row (from the level's base)
    uint16_t deg[kN];
    uint16_t cm[kN], csz[kN], dec[kN];
    uint16_t list[kN];         // vertices by (sub-round, class); aggregation: by community
    uint8_t flag[kN];          // unprocessed
    uint8_t next[kN];          // marked in this sub-round
    uint8_t rnd[kN];           // sub-round (255: no entries)
    int beg[kMaxRounds * kClasses + 1];
    int wi[kWaves];
    unsigned long long gain, verts, scanned[3];
    unsigned moved;            // at most 64 passes of 100 sweeps of kN
    int bad;
};

// The workgroup's state; an accessor, so that the functions below share it
// without being inlined into one body: inlined, the scans' copies and the
// phase's own values did not fit 128 registers (106 spilled).
__device__ __forceinline__ State &state() {
    __shared__ __align__(16) State s;
    return s;
}

__device__ __forceinline__ double entry_weight(const void *w, int wt, int64_t e) {
    return wt == W_UNIT ? 1.0 : wt == W_F32 ? (double)((const float *)w)[e] : ((const double *)w)[e];
}

// Sum over the workgroup of one int per thread, exclusive prefix returned,
// total in *total.
__device__ __forceinline__ int scan_block(State &s, int x, int *total) {
    const int lane = lane_id(), w = threadIdx.x / kWave;
    int inc = x;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const int y = __shfl_up(inc, o);
        if (lane >= o) inc += y;
    }
    if (lane == kWave - 1) s.wi[w] = inc;
    __syncthreads();
    int before = 0, all = 0;
#pragma unroll
    for (int q = 0; q < kWaves; q++) {
        if (q < w) before += s.wi[q];
        all += s.wi[q];
    }
    __syncthreads();
    *total = all;
    return before + inc - x;
}

// A candidate community of the scan (ties to the lower id).
__device__ __forceinline__ void offer(double g, int c, double &bg, int &bc) {
    if (g > bg || (g == bg && c < bc)) {
        bg = g;
        bc = c;
    }
}

// Scans of rows list[k0 ..] of one class by a wavefront: L lanes and a table
// of L kPerLane slots per row, R entries per lane.  Every step keeps all of
// its loads, compare-and-swaps or table reads in flight together.
template <int L, int R>
__device__ __noinline__ void scan_rows(const int32_t *col, const double *w, int k0, int k1, double m2) {
    State &s = state();
    constexpr uint32_t S = L * kPerLane;
    const int lane = lane_id(), grp = lane / L, gl = lane % L;
    int *keys = s.pool.keys + (threadIdx.x / kWave) * kWaveSlots + grp * S;
    double *vals = s.pool.vals + (threadIdx.x / kWave) * kWaveSlots + grp * S;
    const int k = k0 + grp;
    const int i = k < k1 ? s.list[k] : 0;
    const bool on = k < k1 && s.flag[i];
    if (!__any(on)) return;
    const int di = on ? s.deg[i] : 0;
    const int64_t b = s.rowb[i];
    int j[R], c[R];
    double x[R];
#pragma unroll
    for (int r = 0; r < R; r++) {
        const int e = gl + r * L;
        j[r] = e < di ? col[b + e] : i;
        x[r] = e < di ? w[b + e] : 0.0;
    }
    const int d = s.cm[i];
    const double ki = s.K[i], sgd = s.sig[d];
#pragma unroll
    for (int r = 0; r < R; r++) c[r] = j[r] != i ? s.cm[j[r]] : kEmpty;
    int q[R];
    const unsigned owned = table_put_all(
        keys, vals, c, x, q, [](int key) { return (int)(key_hash(key) >> (32 - __builtin_ctz(S))); },
        [](int at, int key) { return (at + step_shift(key_hash(key))) & (int)(S - 1); });
    __builtin_amdgcn_wave_barrier();
    // the lane that claimed a slot scores its community and clears the slot:
    // nothing reads the empty slots
    bool own[R];
    double v[R], sg[R];
#pragma unroll
    for (int r = 0; r < R; r++) {
        v[r] = sg[r] = 0.0;
        own[r] = (owned >> r) & 1u;
        if (own[r]) {
            v[r] = vals[q[r]];
            sg[r] = s.sig[c[r]];
            keys[q[r]] = kEmpty;
            vals[q[r]] = 0.0;
        }
    }
    double bg = -INFINITY, kid = 0.0;
    int bc = kIntMax;
#pragma unroll
    for (int r = 0; r < R; r++) {
        if (!own[r]) continue;
        if (c[r] == d)
            kid = v[r];
        else
            offer(m2 * v[r] - ki * sg[r], c[r], bg, bc);
    }
    const double top = group_max<L>(bg);
    bc = group_min<L>(bg == top ? bc : kIntMax);
    bg = top;
    kid = group_max<L>(kid);   // one lane's, 0 elsewhere; weights are >= 0
    // the decision, the same in every lane of the row
    bool mv = false;
    if (bc != kIntMax) {
        const double gstay = m2 * kid - ki * (sgd - ki);
        mv = on && bg > gstay && !(bc > d && s.csz[d] == 1 && s.csz[bc] == 1);
        if (mv && gl == 0) {
            atomicAdd(&s.gain, gain_units(bg - gstay, m2));
            atomicAdd(&s.moved, 1u);
        }
    }
    if (on && gl == 0) s.dec[i] = (uint16_t)(mv ? bc : d);
    if (mv)
#pragma unroll
        for (int r = 0; r < R; r++)
            if (j[r] != i) s.next[j[r]] = 1;
    __builtin_amdgcn_wave_barrier();
}

// Scan of row list[k] by a wavefront with a dense table over the level's n
// communities at slot `at` of the pool: no probing, any row length.  A key
// marks a community as met (one met through entries of weight 0 only is a
// candidate too).  Keys are empty and values 0 on entry and on return.
__device__ __noinline__ void scan_dense(const int32_t *col, const double *w, int k, int at, int n, double m2) {
    State &s = state();
    const int lane = lane_id();
    int *keys = s.pool.keys + at;
    double *vals = s.pool.vals + at;
    const int i = s.list[k];
    if (!s.flag[i]) return;   // the same in every lane
    const int di = s.deg[i];
    const int64_t b = s.rowb[i];
    constexpr int R = 8;
    for (int e0 = 0; e0 < di; e0 += R * kWave) {
        int j[R];
        double x[R];
#pragma unroll
        for (int r = 0; r < R; r++) {
            const int e = e0 + r * kWave + lane;
            j[r] = e < di ? col[b + e] : i;
            x[r] = e < di ? w[b + e] : 0.0;
        }
#pragma unroll
        for (int r = 0; r < R; r++) {
            if (j[r] == i) continue;
            const int c = s.cm[j[r]];
            keys[c] = c;
            atomicAdd(&vals[c], x[r]);
        }
    }
    __builtin_amdgcn_wave_barrier();
    const int d = s.cm[i];
    const double ki = s.K[i], sgd = s.sig[d];
    double bg = -INFINITY, kid = 0.0;
    int bc = kIntMax;
    for (int c = lane; c < n; c += kWave) {
        if (keys[c] == kEmpty) continue;
        const double v = vals[c];
        keys[c] = kEmpty;
        vals[c] = 0.0;
        if (c == d)
            kid = v;
        else
            offer(m2 * v - ki * s.sig[c], c, bg, bc);
    }
    const double top = group_max<kWave>(bg);
    bc = group_min<kWave>(bg == top ? bc : kIntMax);
    kid = group_max<kWave>(kid);
    bool mv = false;
    if (bc != kIntMax) {
        const double gstay = m2 * kid - ki * (sgd - ki);
        mv = top > gstay && !(bc > d && s.csz[d] == 1 && s.csz[bc] == 1);
        if (mv && lane == 0) {
            atomicAdd(&s.gain, gain_units(top - gstay, m2));
            atomicAdd(&s.moved, 1u);
        }
    }
    if (lane == 0) s.dec[i] = (uint16_t)(mv ? bc : d);
    if (mv)
        for (int e = lane; e < di; e += kWave) {
            const int j = col[b + e];
            if (j != i) s.next[j] = 1;
        }
    __builtin_amdgcn_wave_barrier();
}

// The local-moving phase; returns l_i (the same in every thread).
__device__ __noinline__ int move_phase(int shift, int max_iter, const int32_t *col, const double *w, int n, double m2,
                                       double tau) {
    State &s = state();
    const int tid = threadIdx.x, wv = tid / kWave;
    const int P = 1 << shift;
    for (int q = tid; q < kSlots; q += kT) {
        s.pool.keys[q] = kEmpty;
        s.pool.vals[q] = 0.0;
    }
    const bool dense = n <= kRestDense;
    const int room = kSlots / n < kWaves ? kSlots / n : kWaves;   // wavefronts with a dense table
    for (int q = tid; q <= P * kClasses; q += kT) s.beg[q] = 0;
    __syncthreads();
    auto bucket = [&](int i) {   // (sub-round, class) of a vertex with entries
        const int di = s.deg[i];
        return s.rnd[i] * kClasses + (di <= kRow8 ? 0 : di <= kRow16 ? 1 : di <= kRowC ? 2 : 3);
    };
    for (int i = tid; i < n; i += kT) {
        s.sig[i] = s.K[i];
        s.cm[i] = (uint16_t)i;
        s.csz[i] = 1;
        s.flag[i] = 1;
        s.next[i] = 0;
        s.rnd[i] = s.deg[i] ? (uint8_t)sub_round_of(i, shift) : 255;
        if (s.deg[i]) atomicAdd(&s.beg[bucket(i)], 1);
    }
    __syncthreads();
    {
        int total;
        const int x = tid < P * kClasses ? s.beg[tid] : 0;
        const int at = scan_block(s, x, &total);
        if (tid <= P * kClasses) s.beg[tid] = at;   // tid = P kClasses: the total
    }
    __syncthreads();
    for (int i = tid; i < n; i += kT)
        if (s.deg[i]) s.list[atomicAdd(&s.beg[bucket(i)], 1)] = (uint16_t)i;
    __syncthreads();
    // the cursors now stand at the buckets' ends: bucket k is [end[k - 1], end[k])
    unsigned verts = 0, sc[3] = {0, 0, 0};   // at most 100 sweeps of rest_entries
    int li = 0;
    while (li < max_iter) {
        if (tid == 0) s.gain = 0;
        __syncthreads();
        for (int p = 0; p < P; p++) {
            const int k0 = p ? s.beg[p * kClasses - 1] : 0, k1 = s.beg[p * kClasses], k2 = s.beg[p * kClasses + 1],
                      k3 = s.beg[p * kClasses + 2], k4 = s.beg[p * kClasses + 3];
            if (k0 == k4) continue;   // the same in every thread
            const int kw = dense ? k4 : k3;   // wavefront rows
            const int u8 = (k1 - k0 + 7) / 8, u16 = u8 + (k2 - k1 + 3) / 4, uw = u16 + (kw - k2);
            for (int u = wv; u < uw; u += kWaves) {
                if (u < u8)
                    scan_rows<8, 4>(col, w, k0 + 8 * u, k1, m2);
                else if (u < u16)
                    scan_rows<16, 4>(col, w, k1 + 4 * (u - u8), k2, m2);
                else if (dense)
                    scan_dense(col, w, k2 + (u - u16), wv * kWaveSlots, n, m2);
                else
                    scan_rows<kWave, (kRowC + kWave - 1) / kWave>(col, w, k2 + (u - u16), k3, m2);
            }
            __syncthreads();
            if (k4 > kw) {   // the tables change shape
                for (int k = kw + wv; wv < room && k < k4; k += room) scan_dense(col, w, k, wv * n, n, m2);
                __syncthreads();
            }
            // the moves, and the flags: a scanned vertex is processed unless
            // a mover marked it in this very sub-round
            for (int i = tid; i < n; i += kT) {
                const uint8_t f = s.flag[i], nx = s.next[i];
                uint8_t to = f;
                if (f && s.rnd[i] == p) {
                    to = 0;
                    const int di = s.deg[i];
                    verts++;
                    sc[0] += di <= 64 ? di : 0;
                    sc[1] += di > 64 && di <= kWaveMaxDeg ? di : 0;
                    sc[2] += di > kWaveMaxDeg ? di : 0;
                    const int c = s.dec[i], d = s.cm[i];
                    if (c != d) {
                        const double ki = s.K[i];
                        s.cm[i] = (uint16_t)c;
                        if (ki != 0.0) {
                            atomicAdd(&s.sig[d], -ki);
                            atomicAdd(&s.sig[c], ki);
                        }
                        // sizes are 16 bits in pairs of a word: no borrow or
                        // carry crosses, as a size stays in [0, n] whatever
                        // part of its changes is in
                        atomicAdd(reinterpret_cast<uint32_t *>(s.csz) + (c >> 1), 1u << (16 * (c & 1)));
                        atomicSub(reinterpret_cast<uint32_t *>(s.csz) + (d >> 1), 1u << (16 * (d & 1)));
                    }
                }
                if (nx) {
                    to = 1;
                    s.next[i] = 0;
                }
                if (to != f) s.flag[i] = to;
            }
            __syncthreads();
        }
        const double dq = ldexp((double)s.gain, -61);
        li++;
        __syncthreads();   // s.gain is cleared by the next sweep
        if (dq <= tau) break;
    }
    if (verts) atomicAdd(&s.verts, (unsigned long long)verts);
#pragma unroll
    for (int q = 0; q < 3; q++)
        if (sc[q]) atomicAdd(&s.scanned[q], (unsigned long long)sc[q]);
    __syncthreads();
    return li;
}

__device__ __forceinline__ int uf_root(volatile int *parent, int x) {
    while (true) {
        const int p = parent[x];
        if (p == x) return x;
        const int gp = parent[p];
        if (gp != p) parent[x] = gp;
        x = gp;
    }
}

// Split of the communities into components and renumbering by ascending
// smallest vertex: s.dec[i] <- number of i's component; returns their count.
__device__ __noinline__ int split_renumber(const int32_t *col, int n) {
    State &s = state();
    const int tid = threadIdx.x;
    int *parent = s.pool.keys;
    for (int i = tid; i < n; i += kT) parent[i] = i;
    __syncthreads();
    for (int i = tid / kLanes; i < n; i += kT / kLanes) {
        const int ci = s.cm[i], di = s.deg[i];
        const int64_t b = s.rowb[i];
        for (int e = tid % kLanes; e < di; e += kLanes) {
            const int j = col[b + e];
            if (j == i || s.cm[j] != ci) continue;
            int x = i, y = j;
            while (true) {   // hook the larger root under the smaller
                x = uf_root(parent, x);
                y = uf_root(parent, y);
                if (x == y) break;
                const int hi = x > y ? x : y, lo = x > y ? y : x;
                if (atomicCAS(&parent[hi], hi, lo) == hi) break;
            }
        }
    }
    __syncthreads();
    // roots in order; then every vertex takes its root's number
    int count = 0;
    for (int i0 = 0; i0 < n; i0 += kT) {
        const int i = i0 + tid;
        const bool root = i < n && parent[i] == i;
        int total;
        const int at = scan_block(s, root ? 1 : 0, &total);
        if (root) s.csz[i] = (uint16_t)(count + at);
        count += total;
    }
    __syncthreads();
    for (int i = tid; i < n; i += kT) {
        int r = i;
        while (parent[r] != r) r = parent[r];
        s.dec[i] = s.csz[r];
    }
    __syncthreads();
    return count;
}

// G'' of the level by s.dec (n2 communities) into ocol / ow, rows packed;
// s.rowb, s.deg and s.K then describe it.
__device__ __noinline__ void aggregate_level(const int32_t *col, const double *w, int n, int n2, int32_t *ocol,
                                             double *ow) {
    State &s = state();
    const int tid = threadIdx.x, wv = tid / kWave, lane = lane_id();
    // members of each community, side by side in s.list; first[c] in csz
    uint16_t *first = s.csz;
    int *cur = s.pool.keys;                                       // n2 cursors
    uint32_t *rowb2 = reinterpret_cast<uint32_t *>(s.pool.keys) + kN;   // rows of G''
    uint32_t *deg2 = rowb2 + kN;
    double *K2 = s.sig;                                           // Sigma is not needed any more
    uint32_t *bits = reinterpret_cast<uint32_t *>(s.pool.keys) + 3 * kN;   // presence, kBitWords words
    constexpr int kBitWords = kSlots - 3 * kN;
    double *acc = s.pool.vals;
    for (int c = tid; c < n2; c += kT) {
        cur[c] = 0;
        K2[c] = 0.0;
    }
    __syncthreads();
    for (int i = tid; i < n; i += kT) {
        atomicAdd(&cur[s.dec[i]], 1);
        if (s.K[i] != 0.0) atomicAdd(&K2[s.dec[i]], s.K[i]);
    }
    __syncthreads();
    int base = 0;
    for (int c0 = 0; c0 < n2; c0 += kT) {
        const int c = c0 + tid;
        int total;
        const int at = scan_block(s, c < n2 ? cur[c] : 0, &total);
        if (c < n2) {
            first[c] = (uint16_t)(base + at);
            cur[c] = base + at;
        }
        base += total;
    }
    __syncthreads();
    for (int i = tid; i < n; i += kT) s.list[atomicAdd(&cur[s.dec[i]], 1)] = (uint16_t)i;
    __syncthreads();
    const int wpr = (n2 + 31) / 32;   // presence words per row
    int rows = kDense / n2;
    if (rows > kBitWords / wpr) rows = kBitWords / wpr;
    if (rows > kT) rows = kT;
    uint32_t out = 0;   // entries of G'' so far (the same in every thread)
    for (int c0 = 0; c0 < n2; c0 += rows) {
        const int nr = n2 - c0 < rows ? n2 - c0 : rows;
        for (int q = tid; q < nr * n2; q += kT) acc[q] = 0.0;
        for (int q = tid; q < nr * wpr; q += kT) bits[q] = 0;
        __syncthreads();
        const int m0 = first[c0], m1 = c0 + nr < n2 ? first[c0 + nr] : n;
        for (int m = m0 + tid / kLanes; m < m1; m += kT / kLanes) {
            const int i = s.list[m], r = s.dec[i] - c0, di = s.deg[i];
            const int64_t b = s.rowb[i];
            for (int e = tid % kLanes; e < di; e += kLanes) {
                const int c = s.dec[col[b + e]];
                atomicAdd(&acc[r * n2 + c], w[b + e]);
                atomicOr(&bits[r * wpr + (c >> 5)], 1u << (c & 31));
            }
        }
        __syncthreads();
        for (int r = wv; r < nr; r += kWaves) {
            int k = 0;
            for (int q = lane; q < wpr; q += kWave) k += __popc(bits[r * wpr + q]);
            k = (int)group_sum_ll<kWave>(k);
            if (lane == 0) deg2[c0 + r] = (uint32_t)k;
        }
        __syncthreads();
        int total;
        const int at = scan_block(s, tid < nr ? (int)deg2[c0 + tid] : 0, &total);
        if (tid < nr) rowb2[c0 + tid] = out + (uint32_t)at;
        out += (uint32_t)total;
        __syncthreads();
        for (int r = wv; r < nr; r += kWaves) {
            int64_t at2 = rowb2[c0 + r];
            for (int d0 = 0; d0 < n2; d0 += kWave) {
                const int d = d0 + lane;
                const bool on = d < n2 && ((bits[r * wpr + (d >> 5)] >> (d & 31)) & 1u);
                const unsigned long long m = __ballot(on);
                if (on) {
                    const int64_t q = at2 + __popcll(m & ((1ull << lane) - 1ull));
                    ocol[q] = d;
                    ow[q] = acc[r * n2 + d];
                }
                at2 += __popcll(m);
            }
        }
        __syncthreads();
    }
    for (int c = tid; c < n2; c += kT) {
        s.rowb[c] = rowb2[c];
        s.deg[c] = (uint16_t)deg2[c];
        s.K[c] = K2[c];
    }
    __syncthreads();
}

__global__ void __launch_bounds__(kT) k_rest_of_run(RestArgs a) {
    State &s = state();
    const int tid = threadIdx.x;
    const double m2 = a.M2;
    RestOut *out = a.out;
    const int64_t nv = a.g.n;
    int n = (int)nv;
    // the level, and whether it fits
    if (tid == 0) {
        s.bad = nv > kN;
        s.moved = s.verts = 0;
        s.scanned[0] = s.scanned[1] = s.scanned[2] = 0;
        s.gain = 0;
    }
    __syncthreads();
    unsigned long long ent = 0;
    if (nv <= kN)
        for (int i = tid; i < n; i += kT) {
            const int64_t b = a.g.off[i];
            const int d = a.g.deg[i];
            if (d > kBlockMaxDeg || b > 0xffffffffll) s.bad = 1;
            s.rowb[i] = (uint32_t)b;
            s.deg[i] = (uint16_t)d;
            s.K[i] = a.K[i];
            ent += (unsigned)d;
        }
    if (ent) atomicAdd(&s.gain, ent);
    __syncthreads();
    if (s.bad || s.gain > (unsigned long long)rest_entries(nv, 1 << a.shift)) {
        if (tid == 0) out->status = 1;
        return;
    }
    // its columns, and its weights in fp64, into the first buffer
    int32_t *col = a.col[0];
    double *w = a.w[0];
    for (int i = tid / kLanes; i < n; i += kT / kLanes) {
        const int64_t b = s.rowb[i];
        for (int e = tid % kLanes; e < (int)s.deg[i]; e += kLanes) {
            col[b + e] = a.g.col[b + e];
            w[b + e] = entry_weight(a.g.w, a.g.wt, b + e);
        }
    }
    __syncthreads();
    double tau = a.tau;
    int sweeps = 0, next = 1, passes = 0;
    int32_t *label = a.label;
    while (true) {
        const int li = move_phase(a.shift, a.max_iter, col, w, n, m2, tau);
        sweeps += li;
        const int n2 = split_renumber(col, n);
        // the level's first vertices to the communities so far
        if (passes == 0) {
            for (int i = tid; i < (int)nv; i += kT) label[i] = s.dec[i];
        } else {
            for (int i = tid; i < (int)nv; i += kT) label[i] = s.dec[label[i]];
        }
        if (tid == 0 && passes < kRestPasses) {
            out->iterations[passes] = li;
            out->vertices[passes] = n;
            out->communities[passes] = n2;
        }
        passes++;
        const bool stop = li <= 1 || (double)n2 / (double)n > a.agg_tol || passes == a.passes;
        if (stop || passes == kRestPasses) {
            if (tid == 0) {
                out->status = stop ? 0 : 1;
                out->passes = passes;
                out->ncomm = n2;
                out->sweeps = sweeps;
                out->moved = s.moved;
                out->verts = s.verts;
                for (int q = 0; q < 3; q++) out->scanned[q] = s.scanned[q];
            }
            break;
        }
        aggregate_level(col, w, n, n2, a.col[next], a.w[next]);
        col = a.col[next];
        w = a.w[next];
        n = n2;
        next ^= 1;
        tau = tau / a.tol_drop;
    }
}

}  // namespace

void launch_rest_of_run(const RestArgs &a, hipStream_t s) { k_rest_of_run<<<1, kT, 0, s>>>(a); }

}  // namespace gsp
