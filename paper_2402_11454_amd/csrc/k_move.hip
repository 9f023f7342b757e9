// k_move.hip - the local-moving phase (Algorithm "louvainMove") as
// synchronous sub-rounds.  Per sub-round:
//   compact : unprocessed vertices of the sub-round -> per-bin queues (and
//             mark them processed: pruning);
//   small   : degree <= 64, a group of 4..64 lanes per vertex;
//   large   : degree <= 2048, a wavefront or a workgroup per vertex;
//   hub     : degree > 2048, chunks of the row into a global table, then a
//             workgroup per hub picks the best community;
//   apply   : moves of the sub-round, community totals Sigma and sizes.
// Each scan+decide kernel builds the table K_{i->c} of scanCommunities
// (self-loop skipped), evaluates Eq. 2 multiplied through by 2m^2:
//   G(c)    = M2 K_{i->c} - K_i Sigma_c            (candidate c != d)
//   G(stay) = M2 K_{i->d} - K_i (Sigma_d - K_i)
// so dQ_{i:d->c} = (G(c) - G(stay)) / (M2^2/2), takes the best candidate
// (ties to the lowest id), moves i only if G(best) > G(stay) unless i and the
// target are both one-vertex communities and the target id is larger, and
// marks every neighbour j != i of a mover unprocessed.  Everything is read
// from the sub-round's snapshot: memberships and totals change only in
// `apply`.  Built with -ffp-contract=off so every product and difference is
// a single IEEE operation.
#include <math.h>

#include "gsp_internal.h"

namespace gsp {

namespace {


struct Acc {          // per-thread counters, reduced per block at the end
    unsigned long long gain = 0;   // units of 2^-61 of delta-modularity (gain_units)
    unsigned long long moved = 0, verts = 0, scanned = 0, keys = 0, ginserts = 0, aux = 0;
};

// Adds a workgroup's counters to its stripe.  Workgroups that counted nothing
// leave at once; in the others only the counters that some lane of a
// wavefront has are summed over its lanes (summing all seven in every
// workgroup took 1.5 us at the end of each launch, as long as a unit's trips
// to memory).
__device__ __forceinline__ void flush_acc(const Acc &acc, IterCounters *ctr, int cls) {
    constexpr int F = 7;
    __shared__ unsigned long long part[F][kBlock / kWave];
    const unsigned long long v[F] = {acc.gain, acc.moved, acc.verts, acc.scanned, acc.keys, acc.ginserts, acc.aux};
    bool some = false;
#pragma unroll
    for (int f = 0; f < F; f++) some = some || v[f] != 0;
    if (!__syncthreads_or(some)) return;
#pragma unroll
    for (int f = 0; f < F; f++) {
        unsigned long long x = v[f];
        const unsigned long long has = __ballot(x != 0);
        if ((has & (has - 1)) != 0) x = (unsigned long long)group_sum_ll<kWave>((long long)x);
        if (lane_id() == (has ? __ffsll((long long)has) - 1 : 0)) part[f][threadIdx.x / kWave] = x;
    }
    __syncthreads();
    if (threadIdx.x < F) {
        const int f = threadIdx.x;
        unsigned long long t = 0;
#pragma unroll
        for (int w = 0; w < kBlock / kWave; w++) t += part[f][w];
        CounterStripe &st = ctr->st[blockIdx.x % kStripes];
        unsigned long long *to = f == 0 ? &st.gain : f == 1 ? &st.moved : f == 2 ? &st.verts[cls]
                                 : f == 3 ? &st.scanned[cls] : f == 4 ? &st.keys[cls]
                                 : f == 5 ? &st.ginserts[cls] : &st.aux[cls];
        if (t) atomicAdd(to, t);
    }
}

// What a scan serves beside the plain sweeps of one graph: a batch's graphs;
// the history, traces and D_i of the gate; move records and gain outputs.
// The scans of untimed sweeps are compiled for none, for a batch and for
// all: code that a sweep never runs costs it registers (the general scans
// spill) and, as a launch on a small level is one pass through the code,
// instruction fetches.
enum { kScanBatch = 1, kScanHist = 2, kScanOther = 4, kScanAll = 7 };

// Batch: a mover's gain and count into its graph's totals (one lane).
__device__ __forceinline__ void graph_totals(const MoveArgs &a, int i, unsigned long long gain) {
    int gk = a.g.gid[i];
    atomicAdd(&a.ggain[gk], gain);
    atomicAdd(&a.gmoved[gk], 1ull);
}

// The part of a mover's gain (i: d -> bc) that counts towards the sweep's
// total, in fixed point (gain_units): all of it, unless the return-move
// option gives move records (mhist).  Then a move back into the community i
// left at its move of the preceding sweep, which undoes a swap made from one
// snapshot, counts nothing (the move is still made), and this move is
// recorded.  One lane per mover.
template <int F = kScanAll>
__device__ __forceinline__ unsigned long long counted_gain(const MoveArgs &a, int i, int d, int bc, double gain,
                                                           double m2) {
    if ((F & kScanOther) && a.mhist) {
        const int32_t sw = (int32_t)*a.sweep_dev;
        const uint64_t h = (uint64_t)a.mhist[i];
        a.mhist[i] = (int64_t)(((uint64_t)(uint32_t)d << 32) | (uint32_t)sw);
        if ((int32_t)(h >> 32) == bc && (int32_t)(uint32_t)h == sw - 1) return 0ull;
    }
    return gain_units(gain, m2);
}

// 2m of vertex i's graph (the level's 2m unless it holds a batch).
template <int F = kScanAll>
__device__ __forceinline__ double m2_of(const MoveArgs &a, int i) {
    return (F & kScanBatch) && a.g.M2g ? a.g.M2g[a.g.gid[i]] : a.M2;
}

// Decision from the group's best candidate; identical on every lane.
// sig_d = Sigma_d and csz_d = |d| are loaded early by the callers;
// bc_single says whether the best community bc is a singleton (see
// best_single: looked up only when the rule can apply).
__device__ __forceinline__ bool decide(double m2, int d, double ki, double kid, double bg, int bc, double sig_d,
                                       int csz_d, int bc_single, double *gain) {
    if (bc == kIntMax) return false;
    double gstay = m2 * kid - ki * (sig_d - ki);
    if (!(bg > gstay)) return false;
    if (bc_single) return false;
    *gain = bg - gstay;
    return true;
}

// Whether community bc is a singleton, read only where the singleton rule
// can reject the move (d a singleton, bc > d).
__device__ __forceinline__ int best_single(const MoveArgs &a, int d, int csz_d, int bc) {
    if (csz_d != 1 || bc == kIntMax) return 0;
    const int32_t *o = a.g.orig;
    if (!(o ? o[bc] > o[d] : bc > d)) return 0;
    return a.csize[bc] == 1;
}

// History of a scan (for the learned gate's features) and, if sampled, a
// trace row with the features the vertex had before this scan and whether
// it moves.  Called by one lane per decided vertex; no-op unless enabled.
__device__ __forceinline__ void record_scan(const MoveArgs &a, double m2, int i, int d, int di, double ki, double kid,
                                           double bg, int bc, bool mv) {
    uint8_t hb = a.hbits[i];
    float hf = a.hfrac[i], hg = a.hgain[i];
    const int vid = a.g.orig ? a.g.orig[i] : i;   // the caller's id of i
    if (a.tr.x && trace_keep(a.tr.seed, a.pass, a.sweep, vid, a.tr.thr)) {
        uint16_t x[kGateFeatures];
        gate_features(di, ki, a.sig[d], hf, hg, hb, a.dsnap[i], a.pass, a.iter, x);
        int r = blockIdx.x % kStripes;
        unsigned long long slot = atomicAdd(&a.tr.cnt[r], 1ull);
        if ((int64_t)slot < a.tr.scap) {
            int64_t row = r * a.tr.scap + (int64_t)slot;
#pragma unroll
            for (int f = 0; f < kGateFeatures; f++) a.tr.x[row * kGateFeatures + f] = bf16_value(x[f]);
            a.tr.y[row] = mv ? 1 : 0;
            a.tr.v[row] = vid;
            a.tr.meta[row] = a.pass * 256 + a.sweep;
        }
    }
    float nf = 0.0f, ng = 0.0f;
    if (ki > 0.0) {
        nf = (float)(kid / ki);
        double gstay = m2 * kid - ki * (a.sig[d] - ki);
        double r = bc != kIntMax ? (bg - gstay) / (m2 * ki) : -1.0;
        if (r > 1.0) r = 1.0;
        if (r < -1.0) r = -1.0;
        ng = (float)r;
    }
    a.hfrac[i] = nf;
    a.hgain[i] = ng;
    a.hbits[i] = kHistScanned | (mv ? kHistMoved : 0);
    // D_i starts again at a scan.  Movers of this sub-round may be adding to
    // it right now; taking away exactly the value the features saw (which is
    // all D_i held before this sub-round's moves) leaves just their adds, in
    // any order, as the sums are exact.
    if (a.dsnap[i] != 0.0) unsafeAtomicAdd(&a.dmoved[i], -a.dsnap[i]);
}

// A mover's entry (i, j), j != i: j is unprocessed again and, with the
// gate's history on, D_j grows by w_ij.
template <int F = kScanAll>
__device__ __forceinline__ void mark_neighbour(const MoveArgs &a, int j, double w) {
    a.flag[j] = 1;
    if ((F & kScanHist) && a.dmoved) unsafeAtomicAdd(&a.dmoved[j], w);
}

// Folds the entry (key, v) of a scan table into (bg, bc, kid).
__device__ __forceinline__ void fold_key(const MoveArgs &a, double m2, int key, double v, int d, double ki, double &bg,
                                         int &bc, double &kid) {
    if (key == d) {
        kid = v;
    } else {
        double g = m2 * v - ki * a.sig[key];
        if (better(g, key, bg, bc, a.g.orig)) {
            bg = g;
            bc = key;
        }
    }
}

// Value type of the wave and workgroup LDS tables: on unit weights every
// K_{i->c} is a count (< 2^31), kept as an int (8-byte slots, a quarter
// more resident waves); otherwise the fp64 sum.
template <int WT> struct TabVal { using T = double; };
template <> struct TabVal<W_UNIT> { using T = int; };

// Scores a whole table of T slots with NT threads (t = this thread's
// index), resetting it: each thread reads CH slots, then the Sigma of their
// communities together, then folds them.  The argmax does not depend on the
// order of the slots.
template <int NT, int CH, typename V>
__device__ __forceinline__ void fold_table(const MoveArgs &a, double m2, int *keys, V *vals, int T, int t, int d,
                                           double ki, double &bg, int &bc, double &kid,
                                           unsigned long long &nkeys) {
    for (int s0 = 0; s0 < T; s0 += NT * CH) {
        int key[CH];
        double v[CH], sg[CH];
#pragma unroll
        for (int u = 0; u < CH; u++) {
            const int sl = s0 + u * NT + t;
            key[u] = sl < T ? keys[sl] : kEmpty;
            v[u] = 0.0;
            if (key[u] != kEmpty) {
                v[u] = (double)vals[sl];
                keys[sl] = kEmpty;
                vals[sl] = 0;
            }
        }
#pragma unroll
        for (int u = 0; u < CH; u++) sg[u] = (key[u] != kEmpty && key[u] != d) ? a.sig[key[u]] : 0.0;
#pragma unroll
        for (int u = 0; u < CH; u++) {
            if (key[u] == kEmpty) continue;
            nkeys++;
            if (key[u] == d) {
                kid = v[u];
            } else {
                double g = m2 * v[u] - ki * sg[u];
                if (better(g, key[u], bg, bc, a.g.orig)) {
                    bg = g;
                    bc = key[u];
                }
            }
        }
    }
}

// Reads and clears the slots the thread owns and folds their communities
// into (bg, bc, kid).
template <int R, typename V>
__device__ __forceinline__ void take_owned(const MoveArgs &a, double m2, int *keys, V *vals, const int (&c)[R],
                                           const int (&q)[R], unsigned own, int d, double ki, double &bg, int &bc,
                                           double &kid) {
    double v[R], sg[R];
#pragma unroll
    for (int r = 0; r < R; r++) {
        v[r] = sg[r] = 0.0;
        if ((own >> r) & 1u) {
            if (c[r] != d) sg[r] = a.sig[c[r]];
            v[r] = (double)vals[q[r]];
            keys[q[r]] = kEmpty;
            vals[q[r]] = 0;
        }
    }
#pragma unroll
    for (int r = 0; r < R; r++) {
        if (!((own >> r) & 1u)) continue;
        if (c[r] == d) {
            kid = v[r];
        } else {
            const double g = m2 * v[r] - ki * sg[r];
            if (better(g, c[r], bg, bc, a.g.orig)) {
                bg = g;
                bc = c[r];
            }
        }
    }
}

// ---------------------------------------------------------------- compact

// Unprocessed vertices of the sub-round's buckets -> per-bin queues (or,
// in a gated sweep, per-bin candidate lists for the gate).  A workgroup
// takes a range of 256 << shift entries of one bucket, all loaded together,
// and reserves its queue slots with one atomic.  The queue counters are shared
// by every workgroup, and each of their atomics costs the kernel about 9 ns, so
// ranges grow once there are 256 of them.  (Ranges across the buckets, staged
// in LDS with a rank per bin, took a level of 2,900,000 vertices with a nearly
// empty frontier 14.0 us a sub-round, with the moves' application, and one of
// 6,500,000 16.7 us; now 8.3 and 11.4.)
constexpr int kCompactMax = 3;                   // shift at most
constexpr int kCompactR = 1 << kCompactMax;      // entries per thread at most
constexpr int kBlockLog = 8;
static_assert(kBlock == 1 << kBlockLog, "a workgroup's entries by shifts");

__device__ void compact_range(const MoveArgs &a, const int32_t *bl, int shift, int64_t part) {
    const int64_t span = (int64_t)kBlock << shift;
    int b = 0;
    int64_t cap = 0, base = 0;
    bool found = false;
#pragma unroll
    for (int q = 0; q < kNumBins; q++) {
        const int64_t ranges = (a.qcap[q] + span - 1) >> (kBlockLog + shift);
        if (!found && part < ranges) {
            found = true;
            b = q;
            cap = a.qcap[q];
            base = a.qbase[q];
        } else if (!found) {
            part -= ranges;
        }
    }
    const bool gated = a.cand != nullptr;   // the gate fills the queue from the candidates
    const int64_t lo = part * span + threadIdx.x;
    int v[kCompactR];
    bool act[kCompactR];
#pragma unroll
    for (int r = 0; r < kCompactR; r++) {
        v[r] = -1;
        if (r < (1 << shift) && lo + r * kBlock < cap) v[r] = bl[base + lo + r * kBlock];
    }
#pragma unroll
    for (int r = 0; r < kCompactR; r++) act[r] = r < (1 << shift) && v[r] >= 0 && a.flag[v[r]] != 0;
    unsigned long long m[kCompactR];
    int total = 0;
#pragma unroll
    for (int r = 0; r < kCompactR; r++) {
        const int i = v[r];
        if (act[r] && a.gactive && !a.gactive[a.g.gid[i]]) act[r] = false;
        if (act[r] && a.single_only && a.csize[a.cm[i]] != 1) {
            a.flag[i] = 0;   // merged into a sub-community: stays
            act[r] = false;
        }
        if (b == BIN_HUB && i >= 0) a.hub_act[i] = act[r] ? 1 : 0;
        if (act[r]) {
            a.flag[i] = 0;
            if (a.dmoved) a.dsnap[i] = a.dmoved[i];   // the features' D_i
        }
        m[r] = __ballot(act[r]);
        total += __popcll(m[r]);
    }
    __shared__ int first[kBlock / kWave];
    const int w = threadIdx.x / kWave;
    if (lane_id() == 0) first[w] = total;
    __syncthreads();
    if (threadIdx.x == 0) {
        int sum = 0;
#pragma unroll
        for (int k = 0; k < kBlock / kWave; k++) sum += first[k];
        int at = 0;
        if (sum > 0) at = atomicAdd(gated ? &a.ctr->ccnt[a.round][b] : &a.ctr->qcnt[a.round][b], sum);
#pragma unroll
        for (int k = 0; k < kBlock / kWave; k++) {
            const int t = first[k];
            first[k] = at;
            at += t;
        }
    }
    __syncthreads();
    int32_t *out = (gated ? a.cand : a.queue) + base + first[w];
#pragma unroll
    for (int r = 0; r < kCompactR; r++) {
        if (act[r]) out[__popcll(m[r] & ((1ull << lane_id()) - 1ull))] = v[r];
        out += __popcll(m[r]);
    }
}

__global__ void __launch_bounds__(kBlock) k_move_compact(MoveArgs a, const int32_t *bl, int shift) {
    compact_range(a, bl, shift, blockIdx.x);
}

// ---------------------------------------------------------------- small

// Orders the LDS operations of one wavefront (its lanes are the only users
// of their table region): no workgroup barrier, so the waves of a block run
// their units independently.
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
    __builtin_amdgcn_wave_barrier();
}

// Small bins (degree <= G = 4, 8, ..., 64): a group of L = max(G /
// kSmallE, 1) lanes per vertex, up to kSmallE entries per lane (loaded
// together), a table of 2G slots per vertex in the wave's LDS; a wavefront
// takes 64 / L vertices.  G is a runtime value, so the five bins share one
// code path.
constexpr int kSmallE = 4;
__host__ __device__ inline int small_lanes(int G) { return G > kSmallE ? G / kSmallE : 1; }

template <int WT, int F>
__device__ void small_unit(const MoveArgs &a, int bin, int G, int64_t unit, int cnt, int *wkeys, double *wvals,
                           Acc &acc) {
    const int kSlots = 2 * G, L = small_lanes(G);
    const int lane = lane_id();
    const int grp = lane / L, gl = lane & (L - 1);
    const int64_t qi = unit * (kWave / L) + grp;
    const bool valid = qi < cnt;
    int *keys = wkeys + grp * kSlots;
    double *vals = wvals + grp * kSlots;
    int i = -1, di = 0, d = -1, csd = 0;
    int j[kSmallE], c[kSmallE], q[kSmallE];
    double w[kSmallE];
    double ki = 0.0, m2 = a.M2, sgd = 0.0;
    unsigned own = 0;
#pragma unroll
    for (int r = 0; r < kSmallE; r++) {
        j[r] = -1;
        c[r] = kEmpty;
        q[r] = 0;
        w[r] = 0.0;
    }
    if (valid) {
        i = a.queue[a.qbase[bin] + qi];
        m2 = m2_of<F>(a, i);
        di = a.g.deg[i];
        d = a.cm[i];
        ki = a.K[i];
        sgd = a.sig[d];
        csd = a.csize[d];
        const int64_t b0 = a.g.off[i];
#pragma unroll
        for (int r = 0; r < kSmallE; r++) {
            const int e = gl + r * L;
            if (e < di) {
                j[r] = load_col(a.g.col, b0 + e);
                w[r] = edge_weight<WT>(a.g.w, b0 + e);
            }
        }
#pragma unroll
        for (int r = 0; r < kSmallE; r++) c[r] = (j[r] >= 0 && j[r] != i) ? a.cm[j[r]] : kEmpty;
        own = table_put_all(
            keys, vals, c, w, q, [&](int key) { return (int)(key_hash(key) & (uint32_t)(kSlots - 1)); },
            [&](int at, int key) { return (at + step_mask(key_hash(key))) & (kSlots - 1); });
    }
    wave_lds_sync();
    double bg = -INFINITY, kid = 0.0;
    int bc = kIntMax;
    if (valid) take_owned(a, m2, keys, vals, c, q, own, d, ki, bg, bc, kid);
    acc.keys += __popc(own);
    group_argmax_rt(bg, bc, L, a.g.orig);
    kid = group_max_rt(kid, L);   // one lane's, 0 elsewhere; weights are >= 0
    double gain = 0.0;
    bool mv = valid && decide(m2, d, ki, kid, bg, bc, sgd, csd, best_single(a, d, csd, bc), &gain);
    if (mv)
#pragma unroll
        for (int r = 0; r < kSmallE; r++)
            if (j[r] >= 0 && j[r] != i) mark_neighbour<F>(a, j[r], w[r]);
    bool lead = valid && gl == 0;
    const unsigned long long cg = lead && mv ? counted_gain<F>(a, i, d, bc, gain, m2) : 0ull;
    if ((F & kScanBatch) && a.ggain) {   // batch: per-graph totals, one atomic per graph met by the wavefront
        int gk = valid ? a.g.gid[i] : 0;
        wave_add_u64_by_key(a.ggain, gk, cg, lead && mv);
        wave_add_u64_by_key(a.gmoved, gk, 1ull, lead && mv);
    }
    if (lead) {
        acc.verts++;
        acc.scanned += (unsigned long long)di;
        if ((F & kScanHist) && a.hbits) record_scan(a, m2, i, d, di, ki, kid, bg, bc, mv);
        a.dec[i] = mv ? bc : d;
        if (mv) {
            acc.gain += cg;
            acc.moved++;
        }
        if ((F & kScanOther) && a.gain_out) a.gain_out[i] = mv ? gain : 0.0;
    }
    wave_lds_sync();
}

// vertices of small bin b per wavefront
__host__ __device__ inline int small_vpw(int b) { return kWave / small_lanes(4 << b); }

constexpr int kWaveSlots = 2 * kWave * kSmallE;   // (64 / L) vertices x 2G slots, at most
struct SmallLds {
    double vals[kWaveSlots * (kBlock / kWave)];
    int keys[kWaveSlots * (kBlock / kWave)];
};

// The small bins' share of workgroup `part` of `parts`.
template <int WT, int F>
__device__ __forceinline__ void scan_small(const MoveArgs &a, SmallLds &lds, int part, int parts) {
    int *tkeys = lds.keys;
    double *tvals = lds.vals;
    const int w = threadIdx.x / kWave;
    int *wkeys = tkeys + w * kWaveSlots;
    double *wvals = tvals + w * kWaveSlots;
    int cnt[kNumSmallBins];
    int64_t pre[kNumSmallBins + 1];
    pre[0] = 0;
#pragma unroll
    for (int b = 0; b < kNumSmallBins; b++) {
        cnt[b] = a.ctr->qcnt[a.round][b];
        int vpw = small_vpw(b);
        pre[b + 1] = pre[b] + (cnt[b] + vpw - 1) / vpw;
    }
    // late sweeps queue little: a workgroup without a unit leaves here
    if ((int64_t)part * (kBlock / kWave) >= pre[kNumSmallBins]) return;
    for (int k = lane_id(); k < kWaveSlots; k += kWave) {
        wkeys[k] = kEmpty;
        wvals[k] = 0.0;
    }
    wave_lds_sync();
    Acc acc;
    const int64_t nw = (int64_t)parts * (kBlock / kWave);
    for (int64_t u = (int64_t)part * (kBlock / kWave) + w; u < pre[kNumSmallBins]; u += nw) {
        int b = 0;
        while (u >= pre[b + 1]) b++;
        small_unit<WT, F>(a, b, 4 << b, u - pre[b], cnt[b], wkeys, wvals, acc);
    }
    flush_acc(acc, a.ctr, 0);
}

template <int WT>
__global__ void __launch_bounds__(kBlock, WT == W_UNIT ? 5 : 4) k_move_small(MoveArgs a) {
    __shared__ SmallLds lds;
    scan_small<WT, kScanAll>(a, lds, blockIdx.x, gridDim.x);
}

// ---------------------------------------------------------------- large

// Block-wide argmax, and the one non-zero x (K_{i->d}, >= 0), through LDS;
// every thread gets the result.
__device__ void block_argmax_kid(double &bg, int &bc, double &x, const int32_t *orig) {
    __shared__ double sg[kBlock / kWave], sx[kBlock / kWave];
    __shared__ int sc[kBlock / kWave];
    group_argmax<kWave>(bg, bc, orig);
    x = group_max<kWave>(x);
    int w = threadIdx.x / kWave;
    if (lane_id() == 0) { sg[w] = bg; sc[w] = bc; sx[w] = x; }
    __syncthreads();
    bg = sg[0];
    bc = sc[0];
    x = sx[0];
#pragma unroll
    for (int q = 1; q < kBlock / kWave; q++) {
        if (better(sg[q], sc[q], bg, bc, orig)) { bg = sg[q]; bc = sc[q]; }
        x = fmax(x, sx[q]);
    }
    __syncthreads();
}

// The LDS tables of the wave and workgroup bins (and of the hub chunks).
// With fp64 values they have 768 and 3072 slots, at most two thirds full for
// 512 and 2048 entries: 36 KB per workgroup of four wave tables or one
// workgroup table, so four workgroups share a CU's LDS where half-full
// tables let three (R-MAT 26: 3 % less time per run).  A key's first slot is
// then the multiply-shift reduction of its hash onto the slots.  On unit weights (int values) the
// half-full power-of-two tables already fit four workgroups, and the
// fuller ones only lengthened the probes (R-MAT 20: 2.6 % more time), so
// they stay.  Only claimed slots are read back, so a short row costs the
// same in the whole table as in a part of it.
template <int WT> struct ScanSlots {
    static constexpr int wave = WT == W_UNIT ? kWaveTable : 3 * kWaveMaxDeg / 2;
    static constexpr int block = WT == W_UNIT ? kBlockTable : 3 * kBlockMaxDeg / 2;
};
// Puts a thread's R entries into a table of T slots (table_put_all).
template <int T, int R, typename V>
__device__ __forceinline__ unsigned scan_put_all(int *keys, V *vals, const int (&c)[R], const double (&x)[R],
                                                 int (&q)[R]) {
    return table_put_all(
        keys, vals, c, x, q,
        [](int key) {
            const uint32_t h = key_hash(key);
            return (T & (T - 1)) == 0 ? (int)(h & (uint32_t)(T - 1)) : (int)(((uint64_t)h * (uint32_t)T) >> 32);
        },
        [](int at, int key) {
            const uint32_t h = key_hash(key);
            const int to = at + ((T & (T - 1)) == 0 ? step_mask(h) : step_shift(h));
            return to >= T ? to - T : to;
        });
}

template <int WT> struct WaveLds {
    static constexpr int S = ScanSlots<WT>::wave;
    typename TabVal<WT>::T vals[kBlock / kWave * S];
    int keys[kBlock / kWave * S];
};
template <int WT> struct BlockLds {
    static constexpr int S = ScanSlots<WT>::block;
    typename TabVal<WT>::T vals[S];
    int keys[S];
};

// One wavefront per vertex of 65..512 entries, table in its LDS: workgroup
// `part` of `parts`.
template <int WT, int F>
__device__ __forceinline__ void scan_wave(const MoveArgs &a, WaveLds<WT> &lds, int part, int parts) {
    using V = typename TabVal<WT>::T;
    constexpr int S = WaveLds<WT>::S;
    const int w = threadIdx.x / kWave, lane = lane_id();
    int *keys = lds.keys + w * S;
    V *vals = lds.vals + w * S;
    for (int k = lane; k < S; k += kWave) {
        keys[k] = kEmpty;
        vals[k] = 0;
    }
    wave_lds_sync();
    const int cnt = a.ctr->qcnt[a.round][BIN_WAVE];
    const int64_t nw = (int64_t)parts * (kBlock / kWave);
    Acc acc;
    for (int64_t qi = (int64_t)part * (kBlock / kWave) + w; qi < cnt; qi += nw) {
        int i = a.queue[a.qbase[BIN_WAVE] + qi];
        const double m2 = m2_of<F>(a, i);
        int di = a.g.deg[i];
        int64_t beg = a.g.off[i];
        int d = a.cm[i];
        double ki = a.K[i];
        const double sgd = a.sig[d];
        const int csd = a.csize[d];
        // the lane's entries (at most R) are loaded together, then their
        // memberships: two round trips to memory instead of 2R
        constexpr int R = kWaveMaxDeg / kWave;
        int jj[R];
        double ww[R];
#pragma unroll
        for (int r = 0; r < R; r++) {
            const int e = lane + r * kWave;
            jj[r] = e < di ? load_col(a.g.col, beg + e) : i;
            ww[r] = e < di ? edge_weight<WT>(a.g.w, beg + e) : 0.0;
        }
        int cj[R];
#pragma unroll
        for (int r = 0; r < R; r++) cj[r] = jj[r] != i ? a.cm[jj[r]] : kEmpty;
        int sl[R];
        const unsigned own = scan_put_all<S>(keys, vals, cj, ww, sl);
        wave_lds_sync();
        double bg = -INFINITY, kid = 0.0;
        int bc = kIntMax;
        take_owned(a, m2, keys, vals, cj, sl, own, d, ki, bg, bc, kid);
        acc.keys += __popc(own);
        group_argmax<kWave>(bg, bc, a.g.orig);
        kid = group_max<kWave>(kid);   // one lane's, 0 elsewhere; weights are >= 0
        double gain = 0.0;
        bool mv = decide(m2, d, ki, kid, bg, bc, sgd, csd, best_single(a, d, csd, bc), &gain);
        if (mv)   // the lane's columns are still in registers (weights reloaded)
#pragma unroll
            for (int r = 0; r < R; r++)
                if (jj[r] != i) mark_neighbour<F>(a, jj[r], (F & kScanHist) && a.dmoved ? edge_weight<WT>(a.g.w, beg + lane + r * kWave) : 0.0);
        if (lane == 0) {
            acc.verts++;
            acc.scanned += (unsigned long long)di;
            if ((F & kScanHist) && a.hbits) record_scan(a, m2, i, d, di, ki, kid, bg, bc, mv);
            a.dec[i] = mv ? bc : d;
            if (mv) {
                const unsigned long long cg = counted_gain<F>(a, i, d, bc, gain, m2);
                acc.gain += cg;
                acc.moved++;
                if ((F & kScanBatch) && a.ggain) graph_totals(a, i, cg);
            }
            if ((F & kScanOther) && a.gain_out) a.gain_out[i] = mv ? gain : 0.0;
        }
        wave_lds_sync();
    }
    flush_acc(acc, a.ctr, 1);
}

template <int WT>
__global__ void __launch_bounds__(kBlock, 4) k_move_wave(MoveArgs a) {
    __shared__ WaveLds<WT> lds;
    scan_wave<WT, kScanAll>(a, lds, blockIdx.x, gridDim.x);
}

// One workgroup per vertex of 513..2048 entries, table in LDS: workgroup
// `part` of `parts`.
template <int WT, int F>
__device__ __forceinline__ void scan_block(const MoveArgs &a, BlockLds<WT> &lds, int part, int parts) {
    using V = typename TabVal<WT>::T;
    constexpr int S = BlockLds<WT>::S;
    int *keys = lds.keys;
    V *vals = lds.vals;
    const int tid = threadIdx.x;
    for (int k = tid; k < S; k += kBlock) {
        keys[k] = kEmpty;
        vals[k] = 0;
    }
    __syncthreads();
    const int cnt = a.ctr->qcnt[a.round][BIN_BLOCK];
    Acc acc;
    for (int64_t qi = part; qi < cnt; qi += parts) {
        int i = a.queue[a.qbase[BIN_BLOCK] + qi];
        const double m2 = m2_of<F>(a, i);
        int di = a.g.deg[i];
        int64_t beg = a.g.off[i];
        int d = a.cm[i];
        double ki = a.K[i];
        const double sgd = a.sig[d];
        const int csd = a.csize[d];
        constexpr int R = kBlockMaxDeg / kBlock;   // entries per thread, loaded together
        int jj[R];
        double ww[R];
#pragma unroll
        for (int r = 0; r < R; r++) {
            const int e = tid + r * kBlock;
            jj[r] = e < di ? load_col(a.g.col, beg + e) : i;
            ww[r] = e < di ? edge_weight<WT>(a.g.w, beg + e) : 0.0;
        }
        int cj[R];
#pragma unroll
        for (int r = 0; r < R; r++) cj[r] = jj[r] != i ? a.cm[jj[r]] : kEmpty;
        int sl[R];
        const unsigned own = scan_put_all<S>(keys, vals, cj, ww, sl);
        __syncthreads();
        double bg = -INFINITY, kid = 0.0;
        int bc = kIntMax;
        take_owned(a, m2, keys, vals, cj, sl, own, d, ki, bg, bc, kid);
        acc.keys += __popc(own);
        block_argmax_kid(bg, bc, kid, a.g.orig);
        double gain = 0.0;
        bool mv = decide(m2, d, ki, kid, bg, bc, sgd, csd, best_single(a, d, csd, bc), &gain);
        if (mv)   // the thread's columns are still in registers (weights reloaded)
#pragma unroll
            for (int r = 0; r < R; r++)
                if (jj[r] != i) mark_neighbour<F>(a, jj[r], (F & kScanHist) && a.dmoved ? edge_weight<WT>(a.g.w, beg + tid + r * kBlock) : 0.0);
        if (tid == 0) {
            acc.verts++;
            acc.scanned += (unsigned long long)di;
            if ((F & kScanHist) && a.hbits) record_scan(a, m2, i, d, di, ki, kid, bg, bc, mv);
            a.dec[i] = mv ? bc : d;
            if (mv) {
                const unsigned long long cg = counted_gain<F>(a, i, d, bc, gain, m2);
                acc.gain += cg;
                acc.moved++;
                if ((F & kScanBatch) && a.ggain) graph_totals(a, i, cg);
            }
            if ((F & kScanOther) && a.gain_out) a.gain_out[i] = mv ? gain : 0.0;
        }
        __syncthreads();
    }
    flush_acc(acc, a.ctr, 2);
}

template <int WT>
__global__ void __launch_bounds__(kBlock, 4) k_move_block(MoveArgs a) {
    __shared__ BlockLds<WT> lds;
    scan_block<WT, kScanAll>(a, lds, blockIdx.x, gridDim.x);
}

// The three scans above in one launch: workgroups [0, nb) take the workgroup
// bin, [nb, nb + nw) the wave bin, the others the small bins.  One launch
// after the compaction instead of three on forked streams: a fork and its
// join cost two dependency points of about 10 us, and the three scans of a
// level without hubs then follow the compaction with no gap (batch of 64
// graphs, levels of 12k-177k super-vertices: 52 -> 22 us per sub-round
// together with the fused apply and compaction below).
template <int WT> union ScanLds {
    SmallLds small;
    WaveLds<WT> wave;
    BlockLds<WT> block;
};

template <int WT, int F>
__global__ void __launch_bounds__(kBlock, 4) k_move_scan(MoveArgs a, int nb, int nw) {
    __shared__ ScanLds<WT> lds;
    const int k = blockIdx.x;
    if (k < nb)
        scan_block<WT, F>(a, lds.block, k, nb);
    else if (k < nb + nw)
        scan_wave<WT, F>(a, lds.wave, k - nb, nw);
    else
        scan_small<WT, F>(a, lds.small, k - nb - nw, gridDim.x - nb - nw);
}

// ---------------------------------------------------------------- hubs

// One workgroup per chunk of kHubChunk entries of an active hub: the chunk
// is first reduced in an LDS table (so a community met many times in the
// chunk costs one global atomic), then each distinct (community, partial
// sum) goes into the hub's global table.
template <int WT>
__global__ void __launch_bounds__(kBlock) k_move_hub_insert(MoveArgs a) {
    __shared__ int tkeys[kBlockTable];
    __shared__ double tvals[kBlockTable];
    for (int k = threadIdx.x; k < kBlockTable; k += kBlock) {
        tkeys[k] = kEmpty;
        tvals[k] = 0.0;
    }
    __syncthreads();
    Acc acc;
    for (int64_t k = a.ch_first + blockIdx.x; k < a.ch_first + a.ch_count; k += gridDim.x) {
        int i = a.ch_vert[k];
        if (!a.hub_act[i]) continue;
        int64_t beg = a.ch_beg[k];
        int64_t end = a.g.off[i] + a.g.deg[i];
        if (end > beg + kHubChunk) end = beg + kHubChunk;
        for (int64_t e = beg + threadIdx.x; e < end; e += kBlock) {
            int j = load_col(a.g.col, e);
            double wt = edge_weight<WT>(a.g.w, e);
            if (j != i) lds_table_add(tkeys, tvals, kBlockTable - 1, a.cm[j], wt);
        }
        __syncthreads();
        int64_t tb = a.hub_off[i];
        uint64_t mask = hub_table_size(a.g.deg[i]) - 1;
        int *gk = a.hkeys + tb;
        double *gv = a.hvals + tb;
        // batches of 4 slots: the first compare-and-swaps are issued together
        for (int s0 = threadIdx.x; s0 < kBlockTable; s0 += 4 * kBlock) {
            int key[4], prev[4];
            double v[4];
            uint64_t gs[4];
#pragma unroll
            for (int u = 0; u < 4; u++) {
                int sl = s0 + u * kBlock;
                key[u] = tkeys[sl];
                v[u] = tvals[sl];
                tkeys[sl] = kEmpty;
                tvals[sl] = 0.0;
            }
#pragma unroll
            for (int u = 0; u < 4; u++) {
                prev[u] = kEmpty;
                if (key[u] != kEmpty) {
                    gs[u] = key_hash(key[u]) & mask;
                    prev[u] = atomicCAS(&gk[gs[u]], kEmpty, key[u]);
                }
            }
#pragma unroll
            for (int u = 0; u < 4; u++) {
                if (key[u] == kEmpty) continue;
                acc.ginserts++;
                if (prev[u] == kEmpty || prev[u] == key[u])
                    unsafeAtomicAdd(&gv[gs[u]], v[u]);
                else
                    gbl_table_add(gk, gv, mask, key[u], v[u]);
            }
        }
        if (threadIdx.x == 0) acc.scanned += (unsigned long long)(end - beg);
        __syncthreads();
    }
    flush_acc(acc, a.ctr, 3);
}

// ---------------------------------------------------------------- hubs by hash partitions
//
// A hub's distinct neighbour communities are split into P hash partitions
// (P = its number of chunks).  Phase 1, per chunk: reduce the chunk's entries
// in LDS and write the distinct (community, weight) pairs to staging at the
// chunk's own entry positions, grouped by partition, plus one word per
// partition (start << 16 | count).  Phase 2, per partition: gather that
// partition's pairs from every chunk of the hub into one LDS table and score
// it.  Each (chunk, community) pair is written once and read once; nothing
// goes through a global hash table.

template <int WT>
__global__ void __launch_bounds__(kBlock) k_hub_bucket(MoveArgs a) {
    using V = typename TabVal<WT>::T;
    constexpr int S = ScanSlots<WT>::block;   // a chunk's <= 2048 communities
    __shared__ int tkeys[S];
    __shared__ V tvals[S];
    __shared__ int pcnt[kMaxParts + 1];
    const int tid = threadIdx.x;
    for (int k = tid; k < S; k += kBlock) {
        tkeys[k] = kEmpty;
        tvals[k] = 0;
    }
    __syncthreads();
    Acc acc;
    for (int64_t k = a.ch_first + blockIdx.x; k < a.ch_first + a.ch_count; k += gridDim.x) {
        int i = a.ch_vert[k];
        if (a.hub_act[i] != 1) continue;
        int di = a.g.deg[i];
        int P = (di + kHubChunk - 1) / kHubChunk;
        if (P > a.max_parts) {   // too many partitions: the hub's global table
            if (tid == 0) a.hub_act[i] = 3;
            continue;
        }
        int64_t beg = a.ch_beg[k];
        int64_t end = a.g.off[i] + di;
        if (end > beg + kHubChunk) end = beg + kHubChunk;
        int s = (int)((beg - a.g.off[i]) / kHubChunk);
        constexpr int R = kHubChunk / kBlock;   // entries per thread, loaded together
        int jj[R];
        double ww[R];
#pragma unroll
        for (int r = 0; r < R; r++) {
            const int64_t e = beg + tid + r * kBlock;
            jj[r] = e < end ? load_col(a.g.col, e) : i;
            ww[r] = e < end ? edge_weight<WT>(a.g.w, e) : 0.0;
        }
        int cj[R], sl[R];
#pragma unroll
        for (int r = 0; r < R; r++) cj[r] = jj[r] != i ? a.cm[jj[r]] : kEmpty;
        const unsigned own = scan_put_all<S>(tkeys, tvals, cj, ww, sl);
        for (int b = tid; b <= P; b += kBlock) pcnt[b] = 0;
        __syncthreads();
        // a thread counts, then stages, the communities whose slots it claimed
#pragma unroll
        for (int r = 0; r < R; r++)
            if ((own >> r) & 1u) atomicAdd(&pcnt[part_of(cj[r], P)], 1);
        __syncthreads();
        block_scan_excl(pcnt, P);
        uint32_t *words = a.hbuck + a.hub_b0[i] + (int64_t)s * P;
        for (int b = tid; b < P; b += kBlock) words[b] = ((uint32_t)pcnt[b] << 16) | (uint32_t)(pcnt[b + 1] - pcnt[b]);
        if (tid == 0) acc.aux += (unsigned long long)P;
        __syncthreads();
#pragma unroll
        for (int r = 0; r < R; r++) {
            if (!((own >> r) & 1u)) continue;
            const double v = (double)tvals[sl[r]];
            tkeys[sl[r]] = kEmpty;
            tvals[sl[r]] = 0;
            const int pos = atomicAdd(&pcnt[part_of(cj[r], P)], 1);
            a.skey[beg + pos] = cj[r];
            a.sval[beg + pos] = v;
            acc.ginserts++;
        }
        if (tid == 0) acc.scanned += (unsigned long long)(end - beg);
        __syncthreads();
    }
    flush_acc(acc, a.ctr, 3);
}

// A hub's decision from (bg, bc, kid) (block-uniform): records it, counts
// it in acc (class of the hub decisions) and leaves hub_act = 2 (moves: its
// neighbours are marked chunk by chunk in apply) or 0.  Thread 0 writes.
__device__ __forceinline__ void hub_decide(const MoveArgs &a, int i, double bg, int bc, double kid, int nch,
                                           Acc &acc) {
    if (threadIdx.x != 0) return;
    const double m2 = m2_of(a, i);
    const int d = a.cm[i], di = a.g.deg[i];
    const double ki = a.K[i];
    const int csd = a.csize[d];
    double gain = 0.0;
    bool mv = decide(m2, d, ki, kid, bg, bc, a.sig[d], csd, best_single(a, d, csd, bc), &gain);
    acc.verts++;
    acc.aux += (unsigned long long)nch;
    a.hub_act[i] = mv ? 2 : 0;
    if (a.hbits) record_scan(a, m2, i, d, di, ki, kid, bg, bc, mv);
    a.dec[i] = mv ? bc : d;
    if (mv) {
        const unsigned long long cg = counted_gain(a, i, d, bc, gain, m2);
        acc.gain += cg;
        acc.moved++;
        if (a.ggain) graph_totals(a, i, cg);
    }
    if (a.gain_out) a.gain_out[i] = mv ? gain : 0.0;
}

// A hub's decision after its partitions (all results in part_*): combine
// the P partitions' best candidates and decide.  If a partition overflowed
// or the hub has more than max_parts chunks (hub_act = 3), the workgroup
// takes the whole hub through its global table instead: insert every entry,
// then score and reset the table (rare; slow for enormous hubs, but exact).
template <int WT>
__device__ void hub_finish_block(const MoveArgs &a, int i, int P, Acc &acc) {
    const int tid = threadIdx.x;
    const int d = a.cm[i];
    const double ki = a.K[i];
    const double m2 = m2_of(a, i);
    double bg = -INFINITY, kid = 0.0;
    int bc = kIntMax;
    if (a.hub_act[i] == 3) {
        const int di = a.g.deg[i];
        const int64_t beg = a.g.off[i], T = (int64_t)hub_table_size(di), tb = a.hub_off[i];
        int *gk = a.hkeys + tb;
        double *gv = a.hvals + tb;
        for (int64_t e = beg + tid; e < beg + di; e += kBlock) {
            int j = load_col(a.g.col, e);
            if (j != i) gbl_table_add(gk, gv, (uint64_t)(T - 1), a.cm[j], edge_weight<WT>(a.g.w, e));
        }
        __threadfence();   // the table was built with device-scope atomics
        __syncthreads();
        for (int64_t q = tid; q < T; q += kBlock) {
            int key = __hip_atomic_load(gk + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (key == kEmpty) continue;
            double v = __hip_atomic_load(gv + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            gk[q] = kEmpty;
            gv[q] = 0.0;
            acc.keys++;
            fold_key(a, m2, key, v, d, ki, bg, bc, kid);
        }
    } else {
        const int64_t c0 = a.hub_ch0[i];
        for (int q = tid; q < P; q += kBlock) {
            double g = a.part_g[c0 + q];
            int c = a.part_c[c0 + q];
            if (better(g, c, bg, bc, a.g.orig)) {
                bg = g;
                bc = c;
            }
            kid += a.part_kid[c0 + q];
        }
    }
    block_argmax_kid(bg, bc, kid, a.g.orig);
    hub_decide(a, i, bg, bc, kid, P, acc);
    __syncthreads();
}

// One workgroup per active hub of the sub-round (partition path).
template <int WT>
__global__ void __launch_bounds__(kBlock) k_hub_decide(MoveArgs a) {
    const int cnt = a.ctr->qcnt[a.round][BIN_HUB];
    Acc acc;
    for (int64_t qi = blockIdx.x; qi < cnt; qi += gridDim.x) {
        int i = a.queue[a.qbase[BIN_HUB] + qi];
        hub_finish_block<WT>(a, i, (a.g.deg[i] + kHubChunk - 1) / kHubChunk, acc);
    }
    flush_acc(acc, a.ctr, 4);
}

// Per partition of an active hub: merges the partition's pairs from every
// chunk of the hub (source chunks taken kHubWin at a time) in one LDS table
// and scores it.  On unit weights the values are counts (int slots).
constexpr int kHubWin = 512;

// A hub partition's merge table: on unit weights (int values, 32 KB) 4096
// slots and at most kPartCap distinct communities; otherwise 3072 slots and
// at most 2560 (a partition holds about 2048 on average, as a hub has one
// partition per chunk of 2048 entries), so that four workgroups share a
// CU's LDS where the 4096-slot fp64 table let three.  Past the cap the hub
// takes its global table.
template <int WT> struct GatherSlots {
    static constexpr int slots = WT == W_UNIT ? kBlockTable : 3 * kBlockMaxDeg / 2;
    static constexpr int cap = WT == W_UNIT ? kPartCap : 2560;
};

template <int WT>
__global__ void __launch_bounds__(kBlock) k_hub_gather(MoveArgs a) {
    using V = typename TabVal<WT>::T;
    constexpr int S = GatherSlots<WT>::slots;
    __shared__ int tkeys[S];
    __shared__ V tvals[S];
    __shared__ int pst[kHubWin + 1];
    __shared__ short srcst[kHubWin];   // this partition's start within each source chunk
    __shared__ int nkeys, ovf;
    const int tid = threadIdx.x;
    for (int k = tid; k < S; k += kBlock) {
        tkeys[k] = kEmpty;
        tvals[k] = 0;
    }
    __syncthreads();
    Acc acc;
    for (int64_t k = a.ch_first + blockIdx.x; k < a.ch_first + a.ch_count; k += gridDim.x) {
        int i = a.ch_vert[k];
        // 0: not in this sub-round's frontier; more chunks than max_parts: the
        // hub goes through its global table.  A partition that overflows
        // sends its hub there too (3) while other workgroups gather the hub's
        // other partitions: 1 and 3 are the same here, so that the threads
        // of a workgroup take the barriers below together whichever they see
        if (a.hub_act[i] == 0) continue;
        int di = a.g.deg[i];
        int P = (di + kHubChunk - 1) / kHubChunk;
        if (P > a.max_parts) continue;
        {
        int p = (int)((a.ch_beg[k] - a.g.off[i]) / kHubChunk);
        const uint32_t *words = a.hbuck + a.hub_b0[i];
        const int64_t base = a.g.off[i];
        if (tid == 0) {
            nkeys = 0;
            ovf = 0;
            acc.verts++;   // chunks (partitions) gathered
            acc.aux += (unsigned long long)P;
        }
        for (int w0 = 0; w0 < P; w0 += kHubWin) {
            const int nw = P - w0 < kHubWin ? P - w0 : kHubWin;
            for (int s = tid; s < nw; s += kBlock) {
                uint32_t wd = words[(int64_t)(w0 + s) * P + p];
                pst[s] = (int)(wd & 0xFFFFu);
                srcst[s] = (short)(wd >> 16);
            }
            __syncthreads();
            block_scan_excl(pst, nw);
            const int total = pst[nw];
            if (tid == 0) acc.ginserts += (unsigned long long)total;
            merge_pairs<S, GatherSlots<WT>::cap>(
                pst, nw, total, a.skey, a.sval, tkeys, tvals, &nkeys, &ovf,
                [&](int s, int t) { return base + (int64_t)(w0 + s) * kHubChunk + (int64_t)srcst[s] + (t - pst[s]); });
            __syncthreads();
            if (ovf) break;
        }
        if (ovf) {   // rare: this hub goes through its global table
            for (int q = tid; q < S; q += kBlock) {
                tkeys[q] = kEmpty;
                tvals[q] = 0;
            }
            if (tid == 0) a.hub_act[i] = 3;
        } else {
            int d = a.cm[i];
            double ki = a.K[i];
            const double m2 = m2_of(a, i);
            double bg = -INFINITY, kid = 0.0;
            int bc = kIntMax;
            fold_table<kBlock, 8>(a, m2, tkeys, tvals, S, tid, d, ki, bg, bc, kid, acc.keys);
            block_argmax_kid(bg, bc, kid, a.g.orig);
            if (tid == 0) {
                a.part_g[k] = bg;
                a.part_c[k] = bc;
                a.part_kid[k] = kid;
            }
        }
        }
        __syncthreads();
    }
    flush_acc(acc, a.ctr, 5);
}

// One workgroup per chunk again: chunk s of a hub with nch chunks scores and
// resets the slice [s*seg, (s+1)*seg) of the hub's table (seg = ceil(T /
// nch) <= 8192 slots; the table is complete now) and leaves the slice's best
// candidate and its share of K_{i->d} in part_*[chunk].
__global__ void __launch_bounds__(kBlock) k_move_hub_part(MoveArgs a) {
    Acc acc;
    for (int64_t k = a.ch_first + blockIdx.x; k < a.ch_first + a.ch_count; k += gridDim.x) {
        int i = a.ch_vert[k];
        if (!a.hub_act[i]) continue;
        int di = a.g.deg[i];
        int64_t T = (int64_t)hub_table_size(di);
        int64_t nch = (di + kHubChunk - 1) / kHubChunk;
        int64_t seg = (T + nch - 1) / nch;
        int64_t sidx = (a.ch_beg[k] - a.g.off[i]) / kHubChunk;
        int64_t s0 = sidx * seg, s1 = s0 + seg < T ? s0 + seg : T;
        int d = a.cm[i];
        double ki = a.K[i];
        const double m2 = m2_of(a, i);
        int64_t tb = a.hub_off[i];
        double bg = -INFINITY, kid = 0.0;
        int bc = kIntMax;
        int *gk = a.hkeys + tb;
        double *gv = a.hvals + tb;
        for (int64_t q0 = s0 + threadIdx.x; q0 < s1; q0 += 4 * kBlock) {
            int key[4];
#pragma unroll
            for (int u = 0; u < 4; u++) {
                int64_t q = q0 + u * kBlock;
                key[u] = q < s1 ? gk[q] : kEmpty;
            }
            double v[4];
#pragma unroll
            for (int u = 0; u < 4; u++) {
                v[u] = 0.0;
                if (key[u] != kEmpty) {
                    int64_t q = q0 + u * kBlock;
                    v[u] = gv[q];
                    gk[q] = kEmpty;
                    gv[q] = 0.0;
                    acc.keys++;
                }
            }
#pragma unroll
            for (int u = 0; u < 4; u++)
                if (key[u] != kEmpty) fold_key(a, m2, key[u], v[u], d, ki, bg, bc, kid);
        }
        block_argmax_kid(bg, bc, kid, a.g.orig);
        if (threadIdx.x == 0) {
            a.part_g[k] = bg;
            a.part_c[k] = bc;
            a.part_kid[k] = kid;
        }
    }
    flush_acc(acc, a.ctr, 4);
}

// One wavefront per active hub: combines its chunks' partial results and
// decides (the neighbours of a moving hub are marked by the apply kernel).
__global__ void __launch_bounds__(kBlock) k_move_hub_final(MoveArgs a) {
    const int w = threadIdx.x / kWave, lane = lane_id();
    const int cnt = a.ctr->qcnt[a.round][BIN_HUB];
    const int64_t nw = (int64_t)gridDim.x * (kBlock / kWave);
    Acc acc;
    for (int64_t qi = (int64_t)blockIdx.x * (kBlock / kWave) + w; qi < cnt; qi += nw) {
        int i = a.queue[a.qbase[BIN_HUB] + qi];
        const double m2 = m2_of(a, i);
        int di = a.g.deg[i];
        int d = a.cm[i];
        double ki = a.K[i];
        int64_t c0 = a.hub_ch0[i];
        int nch = (di + kHubChunk - 1) / kHubChunk;
        double bg = -INFINITY, kid = 0.0;
        int bc = kIntMax;
        for (int q = lane; q < nch; q += kWave) {
            double g = a.part_g[c0 + q];
            int c = a.part_c[c0 + q];
            if (better(g, c, bg, bc, a.g.orig)) { bg = g; bc = c; }
            kid += a.part_kid[c0 + q];
        }
        group_argmax<kWave>(bg, bc, a.g.orig);
        kid = group_max<kWave>(kid);   // one chunk's, 0 elsewhere
        double gain = 0.0;
        const int csd = a.csize[d];
        bool mv = decide(m2, d, ki, kid, bg, bc, a.sig[d], csd, best_single(a, d, csd, bc), &gain);
        if (lane == 0) {
            acc.verts++;
            acc.aux += (unsigned long long)nch;
            a.hub_act[i] = mv ? 2 : 0;   // 2: its neighbours are marked chunk by chunk in apply
            if (a.hbits) record_scan(a, m2, i, d, di, ki, kid, bg, bc, mv);
            a.dec[i] = mv ? bc : d;
            if (mv) {
                const unsigned long long cg = counted_gain(a, i, d, bc, gain, m2);
                acc.gain += cg;
                acc.moved++;
                if (a.ggain) graph_totals(a, i, cg);
            }
            if (a.gain_out) a.gain_out[i] = mv ? gain : 0.0;
        }
    }
    flush_acc(acc, a.ctr, 4);
}

// ---------------------------------------------------------------- apply

// Moves of the sub-round.  Workgroups [0, nq) walk the sub-round's queue: every
// vertex whose decision differs from its community moves (C'[i] <- c*);
// the Sigma and size changes of a tile are summed per community in LDS
// first (movers crowd into a few popular communities).  Workgroups [nq, ...)
// take the sub-round's hub chunks and mark the chunk's neighbours of a hub
// that moved.
//
// Atomics to one address follow each other at about 25 ns, so a popular
// community costs a sub-round that times the tiles with movers into it: long
// queues go in tiles of 1,024 entries (4M-vertex DC-SBM, 232,000 entries with
// 68,000 movers among 1,992 tiles of 256: 54 us, now 29; 4.3 -> 2.9 ms of its
// run).  A shorter queue leaves the chip idle in such tiles and waits for four
// rounds of table operations instead (139,000 entries with few movers: 26 us
// with the next compaction, 40 in wide tiles).  Where no community is popular
// wide tiles gain nothing: the moves of a run over a random graph whose whole
// queue is one sub-round take 0.76 of their time in tiles of 256 at 160,000
// vertices, 0.80 at 200,000, 0.90 at 500,000 and 0.94 at 1M (blocks of 200:
// 0.79, 0.83, 0.94, 0.99); the line is where the DC-SBM's queues gain.
constexpr int kApplyR = 4;                     // queue entries per thread and tile, of long queues
constexpr int64_t kApplyWide = 163840;         // those above this many entries
constexpr int kApplyTable = 2 * kApplyR * kBlock;   // slots
constexpr int kApplyProbes = 12;               // a community that finds no slot in as many goes straight on
struct ApplyLds {
    double tv[kApplyTable];
    int tk[kApplyTable], tc[kApplyTable];
};

// Tiles of R queue entries per thread; the workgroup's table is empty before
// and after.
template <int R>
__device__ __forceinline__ void apply_tiles(const MoveArgs &a, const int64_t (&pre)[kNumBins + 1], int part, int nq,
                                            ApplyLds &lds) {
    constexpr int kTile = R * kBlock;
    int *tk = lds.tk, *tc = lds.tc;
    double *tv = lds.tv;
    int32_t *cm = const_cast<int32_t *>(a.cm);
    double *sig = const_cast<double *>(a.sig);
    int32_t *csize = const_cast<int32_t *>(a.csize);
    for (int64_t t0 = part * (int64_t)kTile; t0 < pre[kNumBins]; t0 += (int64_t)nq * kTile) {
        int i[R], c[R], d[R];
#pragma unroll
        for (int r = 0; r < R; r++) {
            const int64_t t = t0 + r * kBlock + threadIdx.x;
            i[r] = -1;
            if (t < pre[kNumBins]) {
                int64_t at = t + a.qbase[0];
#pragma unroll
                for (int b = 1; b < kNumBins; b++)
                    if (t >= pre[b]) at = t - pre[b] + a.qbase[b];
                i[r] = a.queue[at];
            }
        }
#pragma unroll
        for (int r = 0; r < R; r++) {
            c[r] = i[r] >= 0 ? a.dec[i[r]] : 0;
            d[r] = i[r] >= 0 ? cm[i[r]] : 0;
        }
        double ki[R];
#pragma unroll
        for (int r = 0; r < R; r++) ki[r] = c[r] != d[r] ? a.K[i[r]] : 0.0;
        // entry 2k: the community left, 2k + 1: the one joined; the first
        // compare-and-swaps of all go out together
        int at[2 * R];
        unsigned own = 0, open = 0;
#pragma unroll
        for (int r = 0; r < 2 * R; r++) {
            const int key = r & 1 ? c[r / 2] : d[r / 2];
            at[r] = (int)(key_hash(key) & (kApplyTable - 1));
            if (c[r / 2] == d[r / 2]) continue;
            if (r & 1) cm[i[r / 2]] = key;
            const int prev = atomicCAS(&tk[at[r]], kEmpty, key);
            own |= (prev == kEmpty ? 1u : 0u) << r;
            open |= (prev != kEmpty && prev != key ? 1u : 0u) << r;
        }
        for (int probe = 1; open && probe < kApplyProbes; probe++) {
#pragma unroll
            for (int r = 0; r < 2 * R; r++) {
                if (!((open >> r) & 1u)) continue;
                const int key = r & 1 ? c[r / 2] : d[r / 2];
                at[r] = (int)((at[r] + step_mask(key_hash(key))) & (kApplyTable - 1));
                const int prev = atomicCAS(&tk[at[r]], kEmpty, key);
                own |= (prev == kEmpty ? 1u : 0u) << r;
                if (prev == kEmpty || prev == key) open &= ~(1u << r);
            }
        }
#pragma unroll
        for (int r = 0; r < 2 * R; r++) {
            if (c[r / 2] == d[r / 2]) continue;
            const int one = r & 1 ? 1 : -1;
            const double x = r & 1 ? ki[r / 2] : -ki[r / 2];
            if ((open >> r) & 1u) {
                const int key = r & 1 ? c[r / 2] : d[r / 2];
                if (x != 0.0) unsafeAtomicAdd(&sig[key], x);
                atomicAdd(&csize[key], one);
            } else {
                if (x != 0.0) atomicAdd(&tv[at[r]], x);
                atomicAdd(&tc[at[r]], one);
            }
        }
        __syncthreads();
        // who claimed a slot empties it
#pragma unroll
        for (int r = 0; r < 2 * R; r++) {
            if (!((own >> r) & 1u)) continue;
            const int s = at[r], key = r & 1 ? c[r / 2] : d[r / 2], n = tc[s];
            const double x = tv[s];
            if (x != 0.0) unsafeAtomicAdd(&sig[key], x);
            if (n != 0) atomicAdd(&csize[key], n);
            tk[s] = kEmpty;
            tv[s] = 0.0;
            tc[s] = 0;
        }
        __syncthreads();
    }}

__device__ __forceinline__ void apply_moves(const MoveArgs &a, int part, int nq, int nh, ApplyLds &lds) {
    int *tk = lds.tk, *tc = lds.tc;
    double *tv = lds.tv;
    if (part >= nq) {
        for (int64_t k = a.ch_first + (part - nq); k < a.ch_first + a.ch_count; k += nh) {
            int i = a.ch_vert[k];
            if (a.hub_act[i] != 2) continue;
            int64_t beg = a.ch_beg[k];
            int64_t end = a.g.off[i] + a.g.deg[i];
            if (end > beg + kHubChunk) end = beg + kHubChunk;
            for (int64_t e = beg + threadIdx.x; e < end; e += kBlock) {
                int j = load_col(a.g.col, e);
                if (j == i) continue;
                double w = 0.0;
                if (a.dmoved)
                    w = a.g.wt == W_UNIT ? 1.0
                                         : (a.g.wt == W_F32 ? edge_weight<W_F32>(a.g.w, e) : edge_weight<W_F64>(a.g.w, e));
                mark_neighbour(a, j, w);
            }
        }
        return;
    }
    int64_t pre[kNumBins + 1];
    pre[0] = 0;
#pragma unroll
    for (int b = 0; b < kNumBins; b++) pre[b + 1] = pre[b] + a.ctr->qcnt[a.round][b];
    if (part * (int64_t)kBlock * (pre[kNumBins] > kApplyWide ? kApplyR : 1) >= pre[kNumBins]) return;
    for (int s = threadIdx.x; s < kApplyTable; s += kBlock) {
        tk[s] = kEmpty;
        tv[s] = 0.0;
        tc[s] = 0;
    }
    __syncthreads();
    if (pre[kNumBins] > kApplyWide)
        apply_tiles<kApplyR>(a, pre, part, nq, lds);
    else
        apply_tiles<1>(a, pre, part, nq, lds);
}

__global__ void __launch_bounds__(kBlock) k_move_apply(MoveArgs a, int nq) {
    __shared__ ApplyLds lds;
    apply_moves(a, blockIdx.x, nq, gridDim.x - nq, lds);
}

// Apply of one sub-round and, in workgroups [0, nc), the compaction of the
// next (`next`): on a level without hubs every mover's neighbours are marked
// by the scans, so the next sub-round's frontier is final when they end, and
// neither half reads what the other writes (apply: memberships, Sigma,
// sizes; compaction: flags, queues).  One dependent launch fewer per
// sub-round.
__global__ void __launch_bounds__(kBlock) k_move_apply_compact(MoveArgs a, int nc, MoveArgs next, const int32_t *bl,
                                                              int shift) {
    __shared__ ApplyLds lds;
    if ((int)blockIdx.x < nc)
        compact_range(next, bl, shift, blockIdx.x);
    else
        apply_moves(a, blockIdx.x - nc, gridDim.x - nc, 0, lds);
}

// sig[c] += K_i and csize[c] += 1 over the vertices i of community c.  A
// tile of kTotalsTile vertices is summed per community in LDS first, so a
// popular community costs one atomic per tile and distinct communities one
// each.  (Combining the lanes of a wavefront key by key instead takes 64
// rounds of shuffles when they all differ: R-MAT 24, 16.8 M vertices in 7.9 M
// communities, 1.03 ms against 12.5.)
constexpr int kTotalsTile = 4 * kBlock;
constexpr int kTotalsTable = 2 * kTotalsTile;

template <bool SIZES>
__global__ void __launch_bounds__(kBlock) k_community_totals(const double *K, const int32_t *cm, int64_t n,
                                                            double *sig, int32_t *csize) {
    __shared__ int tk[kTotalsTable];
    __shared__ double tv[kTotalsTable];
    __shared__ int tc[SIZES ? kTotalsTable : 1];
    for (int q = threadIdx.x; q < kTotalsTable; q += kBlock) {
        tk[q] = kEmpty;
        tv[q] = 0.0;
        if (SIZES) tc[q] = 0;
    }
    __syncthreads();
    for (int64_t i0 = blockIdx.x * (int64_t)kTotalsTile; i0 < n; i0 += (int64_t)gridDim.x * kTotalsTile) {
        int c[4];
        double k[4];
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const int64_t i = i0 + r * kBlock + threadIdx.x;
            c[r] = i < n ? cm[i] : kEmpty;
            k[r] = i < n ? K[i] : 0.0;
        }
#pragma unroll
        for (int r = 0; r < 4; r++) {
            if (c[r] == kEmpty) continue;
            const int q = lds_table_slot(tk, kTotalsTable - 1, c[r]);
            if (k[r] != 0.0) atomicAdd(&tv[q], k[r]);
            if (SIZES) atomicAdd(&tc[q], 1);
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kTotalsTable / kBlock; r++) {
            const int q = r * kBlock + threadIdx.x;
            const int key = tk[q];
            if (key == kEmpty) continue;
            if (tv[q] != 0.0) unsafeAtomicAdd(&sig[key], tv[q]);
            if (SIZES) atomicAdd(&csize[key], tc[q]);
            tk[q] = kEmpty;
            tv[q] = 0.0;
            if (SIZES) tc[q] = 0;
        }
        __syncthreads();
    }
}

// The same for many vertices: a workgroup per CU keeps one table over all of its
// tiles and empties it when half of the slots are taken, so that few
// communities cost an atomic per workgroup instead of one per tile (4M
// vertices in 606 communities, where each took one from nearly every tile:
// 0.56 ms, now 0.06; 16.8M in 7.9M, some giant: 1.03, now 0.18).  It is the
// few or uneven communities that gain; many even ones cost a little more here
// (8.4M vertices, kept / by tiles: 128 random communities 0.08 / 1.38 ms, 8,192
// 0.28 / 0.34, 131,072 0.37 / 0.36; eight in a row each 0.12 / 0.07), and below
// a tile for every workgroup more of them do (131,072 vertices, 8 to 15 us / 5
// to 10).
constexpr int kKeptThreads = 1024;
constexpr int kKeptTable = 8192;
constexpr int kKeptR = 2;
constexpr int64_t kKeptFrom = 256 * kKeptThreads * kKeptR;   // a tile for every workgroup
template <bool SIZES>
__global__ void __launch_bounds__(kKeptThreads) k_community_totals_kept(const double *K, const int32_t *cm, int64_t n,
                                                                       double *sig, int32_t *csize) {
    constexpr int kTile = kKeptThreads * kKeptR;
    static_assert(kKeptTable / 2 + kTile <= kKeptTable, "a tile fits beside a half full table");
    __shared__ int tk[kKeptTable];
    __shared__ double tv[kKeptTable];
    __shared__ int tc[SIZES ? kKeptTable : 1];
    __shared__ int taken;
    const int tid = threadIdx.x;
    for (int q = tid; q < kKeptTable; q += kKeptThreads) {
        tk[q] = kEmpty;
        tv[q] = 0.0;
        if (SIZES) tc[q] = 0;
    }
    if (tid == 0) taken = 0;
    __syncthreads();
    for (int64_t i0 = blockIdx.x * (int64_t)kTile; i0 < n; i0 += (int64_t)gridDim.x * kTile) {
        int c[kKeptR];
        double k[kKeptR];
#pragma unroll
        for (int r = 0; r < kKeptR; r++) {
            const int64_t i = i0 + r * kKeptThreads + tid;
            c[r] = i < n ? cm[i] : kEmpty;
            k[r] = i < n ? K[i] : 0.0;
        }
        int own = 0;
#pragma unroll
        for (int r = 0; r < kKeptR; r++) {
            if (c[r] == kEmpty) continue;
            const uint32_t h = key_hash(c[r]);
            int q = (int)(h & (kKeptTable - 1));
            while (true) {
                const int prev = tk[q] == c[r] ? c[r] : atomicCAS(&tk[q], kEmpty, c[r]);
                own += prev == kEmpty;
                if (prev == kEmpty || prev == c[r]) break;
                q = (int)((q + step_mask(h)) & (kKeptTable - 1));
            }
            if (k[r] != 0.0) atomicAdd(&tv[q], k[r]);
            if (SIZES) atomicAdd(&tc[q], 1);
        }
        own = (int)group_sum_ll<kWave>(own);
        if (own && lane_id() == 0) atomicAdd(&taken, own);
        __syncthreads();
        const bool empty = taken > kKeptTable / 2 || i0 + (int64_t)gridDim.x * kTile >= n;
        __syncthreads();   // every thread has read the count before any adds the next tile's to it
        if (empty) {
            if (tid == 0) taken = 0;
#pragma unroll
            for (int r = 0; r < kKeptTable / kKeptThreads; r++) {
                const int q = r * kKeptThreads + tid, key = tk[q];
                if (key == kEmpty) continue;
                if (tv[q] != 0.0) unsafeAtomicAdd(&sig[key], tv[q]);
                if (SIZES) atomicAdd(&csize[key], tc[q]);
                tk[q] = kEmpty;
                tv[q] = 0.0;
                if (SIZES) tc[q] = 0;
            }
            __syncthreads();
        }
    }
}

inline unsigned cap_grid(int64_t units, int64_t cap) {
    if (units < 1) units = 1;
    return (unsigned)(units < cap ? units : cap);
}

// A kernel's cap under the run's launch schedule.
inline int64_t sched_cap(const MoveArgs &a, int64_t cap) { return a.grid_cap > 0 && a.grid_cap < cap ? a.grid_cap : cap; }

// One workgroup; the stripes are 6 KB, so it is a chain of one read, the
// stores to the host's memory and the flag behind them.  Clearing here and not
// before the sweep saves the fill's launch.
__global__ void __launch_bounds__(kBlock) k_sweep_end(IterCounters *ctr, unsigned long long *ggain,
                                                     unsigned long long *gmoved, int64_t G, uint64_t *box) {
    static_assert(kSweepWords <= kBlock && sizeof(CounterStripe) >= kSweepWords * 8, "a thread per counter");
    __shared__ int cands;
    const int t = threadIdx.x;
    if (t == 0) cands = 0;
    __syncthreads();
    int *q = &ctr->qcnt[0][0], *c = &ctr->ccnt[0][0];
    for (int k = t; k < kMaxRounds * kNumBins; k += kBlock) {
        const int v = c[k];
        if (v) atomicAdd(&cands, v);
        c[k] = 0;
        q[k] = 0;
    }
    uint64_t *o = box + kBoxHead;
    if (t < kSweepWords) {
        unsigned long long sum = 0;
#pragma unroll
        for (int r = 0; r < kStripes; r++) {
            unsigned long long *w = reinterpret_cast<unsigned long long *>(&ctr->st[r]) + t;
            sum += *w;   // integer units: exact, in any order
            *w = 0;
        }
        o[t] = sum;
    }
    __syncthreads();
    if (t == 0) o[kSweepWords] = (uint64_t)cands;
    for (int64_t k = t; k < G; k += kBlock) {
        o[kSweepWords + 1 + k] = ggain[k];
        o[kSweepWords + 1 + G + k] = gmoved[k];
        ggain[k] = 0;
        gmoved[k] = 0;
    }
    box_post(box);
}

}  // namespace

void launch_community_totals(const double *K, const int32_t *cm, int64_t n, double *sig, int32_t *csize,
                             hipStream_t s) {
    if (n == 0) return;
    const unsigned gr = cap_grid((n + kTotalsTile - 1) / kTotalsTile, 8192);
    if (n >= kKeptFrom && csize)
        k_community_totals_kept<true><<<256, kKeptThreads, 0, s>>>(K, cm, n, sig, csize);
    else if (n >= kKeptFrom)
        k_community_totals_kept<false><<<256, kKeptThreads, 0, s>>>(K, cm, n, sig, nullptr);
    else if (csize)
        k_community_totals<true><<<gr, kBlock, 0, s>>>(K, cm, n, sig, csize);
    else
        k_community_totals<false><<<gr, kBlock, 0, s>>>(K, cm, n, sig, nullptr);
}

static int64_t bucket_total(const MoveArgs &a) {
    int64_t total = 0;
    for (int b = 0; b < kNumBins; b++) total += a.qcap[b];
    return total;
}

// Workgroups of a compaction: ranges of 256 << *shift entries of one bucket.
static int64_t compact_blocks(const MoveArgs &a, int *shift) {
    const int64_t total = bucket_total(a);
    *shift = 0;
    while (*shift < kCompactMax && total > (int64_t)256 * (kBlock << *shift)) (*shift)++;
    const int64_t span = (int64_t)kBlock << *shift;
    int64_t blocks = 0;
    for (int b = 0; b < kNumBins; b++) blocks += (a.qcap[b] + span - 1) / span;
    return blocks;
}

void launch_sweep_end(IterCounters *ctr, unsigned long long *ggain, unsigned long long *gmoved, int64_t G,
                      uint64_t *box, hipStream_t s) {
    k_sweep_end<<<1, kBlock, 0, s>>>(ctr, ggain, gmoved, G, box);
}

void launch_move_compact(const MoveArgs &a, const WorkLists &wl, hipStream_t s) {
    int shift = 0;
    const int64_t blocks = compact_blocks(a, &shift);
    if (blocks > 0) k_move_compact<<<(unsigned)blocks, kBlock, 0, s>>>(a, wl.bl, shift);
}

// wave units of the small bins, at most
static int64_t small_units(const MoveArgs &a) {
    int64_t units = 0;
    for (int b = 0; b < kNumSmallBins; b++) {
        int vpw = small_vpw(b);
        units += (a.qcap[b] + vpw - 1) / vpw;
    }
    return units;
}

void launch_move_small(const MoveArgs &a, const WorkLists &wl, hipStream_t s) {
    (void)wl;
    const int64_t units = small_units(a);
    if (units == 0) return;
    unsigned gr = cap_grid((units + 3) / 4, sched_cap(a, 8192));
    if (a.g.wt == W_UNIT)
        k_move_small<W_UNIT><<<gr, kBlock, 0, s>>>(a);
    else if (a.g.wt == W_F32)
        k_move_small<W_F32><<<gr, kBlock, 0, s>>>(a);
    else
        k_move_small<W_F64><<<gr, kBlock, 0, s>>>(a);
}

void launch_move_wave(const MoveArgs &a, hipStream_t s) {
    if (a.qcap[BIN_WAVE] == 0) return;
    unsigned gr = cap_grid((a.qcap[BIN_WAVE] + 3) / 4, sched_cap(a, 4096));
    if (a.g.wt == W_UNIT)
        k_move_wave<W_UNIT><<<gr, kBlock, 0, s>>>(a);
    else if (a.g.wt == W_F32)
        k_move_wave<W_F32><<<gr, kBlock, 0, s>>>(a);
    else
        k_move_wave<W_F64><<<gr, kBlock, 0, s>>>(a);
}

void launch_move_block(const MoveArgs &a, hipStream_t s) {
    if (a.qcap[BIN_BLOCK] == 0) return;
    unsigned gr = cap_grid(a.qcap[BIN_BLOCK], sched_cap(a, 2048));
    if (a.g.wt == W_UNIT)
        k_move_block<W_UNIT><<<gr, kBlock, 0, s>>>(a);
    else if (a.g.wt == W_F32)
        k_move_block<W_F32><<<gr, kBlock, 0, s>>>(a);
    else
        k_move_block<W_F64><<<gr, kBlock, 0, s>>>(a);
}

void launch_move_scan(const MoveArgs &a, hipStream_t s) {
    const int nb = a.qcap[BIN_BLOCK] ? (int)cap_grid(a.qcap[BIN_BLOCK], sched_cap(a, 2048)) : 0;
    const int nw = a.qcap[BIN_WAVE] ? (int)cap_grid((a.qcap[BIN_WAVE] + 3) / 4, sched_cap(a, 4096)) : 0;
    const int64_t units = small_units(a);
    const int ns = units ? (int)cap_grid((units + 3) / 4, sched_cap(a, 8192)) : 0;
    const int gr = nb + nw + ns;
    if (gr == 0) return;
    const int f = (a.g.gid ? kScanBatch : 0) | (a.hbits || a.dmoved ? kScanHist : 0) |
                  (a.mhist || a.gain_out ? kScanOther : 0);
    auto go = [&](auto none, auto batch, auto all) {
        if (f == 0)
            none<<<gr, kBlock, 0, s>>>(a, nb, nw);
        else if (f == kScanBatch)
            batch<<<gr, kBlock, 0, s>>>(a, nb, nw);
        else
            all<<<gr, kBlock, 0, s>>>(a, nb, nw);
    };
    if (a.g.wt == W_UNIT)
        go(k_move_scan<W_UNIT, 0>, k_move_scan<W_UNIT, kScanBatch>, k_move_scan<W_UNIT, kScanAll>);
    else if (a.g.wt == W_F32)
        go(k_move_scan<W_F32, 0>, k_move_scan<W_F32, kScanBatch>, k_move_scan<W_F32, kScanAll>);
    else
        go(k_move_scan<W_F64, 0>, k_move_scan<W_F64, kScanBatch>, k_move_scan<W_F64, kScanAll>);
}

void launch_move_hub_scan(const MoveArgs &a, hipStream_t s) {
    if (a.qcap[BIN_HUB] == 0) return;
    unsigned gr = cap_grid(a.ch_count, 4096);
    if (a.g.wt == W_UNIT)
        k_move_hub_insert<W_UNIT><<<gr, kBlock, 0, s>>>(a);
    else if (a.g.wt == W_F32)
        k_move_hub_insert<W_F32><<<gr, kBlock, 0, s>>>(a);
    else
        k_move_hub_insert<W_F64><<<gr, kBlock, 0, s>>>(a);
}

void launch_move_hub_parts(const MoveArgs &a, hipStream_t s) {
    if (a.qcap[BIN_HUB] == 0) return;
    unsigned gr = cap_grid(a.ch_count, sched_cap(a, 4096));
    if (a.g.wt == W_UNIT)
        k_hub_bucket<W_UNIT><<<gr, kBlock, 0, s>>>(a);
    else if (a.g.wt == W_F32)
        k_hub_bucket<W_F32><<<gr, kBlock, 0, s>>>(a);
    else
        k_hub_bucket<W_F64><<<gr, kBlock, 0, s>>>(a);
}

void launch_move_hub_gather(const MoveArgs &a, hipStream_t s) {
    if (a.qcap[BIN_HUB] == 0) return;
    unsigned gr = cap_grid(a.ch_count, sched_cap(a, 4096));
    if (a.g.wt == W_UNIT)
        k_hub_gather<W_UNIT><<<gr, kBlock, 0, s>>>(a);
    else
        k_hub_gather<W_F64><<<gr, kBlock, 0, s>>>(a);   // staged values are fp64 sums
}

void launch_move_hub_decide(const MoveArgs &a, hipStream_t s) {
    if (a.qcap[BIN_HUB] == 0) return;
    unsigned gr = cap_grid(a.qcap[BIN_HUB], sched_cap(a, 2048));
    if (a.g.wt == W_UNIT)
        k_hub_decide<W_UNIT><<<gr, kBlock, 0, s>>>(a);
    else if (a.g.wt == W_F32)
        k_hub_decide<W_F32><<<gr, kBlock, 0, s>>>(a);
    else
        k_hub_decide<W_F64><<<gr, kBlock, 0, s>>>(a);
}

void launch_move_hub_finish(const MoveArgs &a, hipStream_t s) {
    if (a.qcap[BIN_HUB] == 0) return;
    k_move_hub_part<<<cap_grid(a.ch_count, 4096), kBlock, 0, s>>>(a);
    k_move_hub_final<<<cap_grid((a.qcap[BIN_HUB] + 3) / 4, 1024), kBlock, 0, s>>>(a);
}

void launch_move_apply(const MoveArgs &a, int64_t cap, hipStream_t s) {
    if (cap == 0) return;
    int nq = (int)cap_grid((cap + kBlock - 1) / kBlock, sched_cap(a, 2048));
    int nh = a.qcap[BIN_HUB] ? (int)cap_grid(a.ch_count, sched_cap(a, 2048)) : 0;
    k_move_apply<<<nq + nh, kBlock, 0, s>>>(a, nq);
}

void launch_move_apply_compact(const MoveArgs &a, const MoveArgs &next, const WorkLists &wl, hipStream_t s) {
    const int nq = (int)cap_grid((bucket_total(a) + kBlock - 1) / kBlock, sched_cap(a, 2048));
    int shift = 0;
    const int64_t blocks = compact_blocks(next, &shift);
    k_move_apply_compact<<<(unsigned)(blocks + nq), kBlock, 0, s>>>(a, (int)blocks, next, wl.bl, shift);
}

}  // namespace gsp
