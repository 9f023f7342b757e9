// k_bins.hip - per-level work lists: every vertex with at least one entry is
// put in bucket (bin of its degree, its sub-round); hubs are cut into chunks
// and get a slot range in the global hub-table pool.
#include <algorithm>

#include "gsp_internal.h"

namespace gsp {

namespace {

// Vertices per tile and workgroup: a bucket's counters take an atomic from
// every tile that meets it, and atomics to one address follow each other at
// about 25 ns, so tiles grow with the level (kBinTiles of them at most, 16
// vertices a thread).  (16.8M vertices in tiles of 1,024: 120 us to fill, now 48;
// 15M 130, now 62.)
constexpr int kBinTile = kBlock * 4;
constexpr int kBinWide = kBlock * 16;
constexpr int64_t kBinTiles = 512;

// Sub-round of vertex v: by its id within its graph when the level holds a
// batch of graphs (gid: graph of each vertex, vbase: first vertex of each
// graph), so every graph of a batch sees the groups it would see alone; by
// its caller's id orig[v] when the level is stored in degree order.
__device__ __forceinline__ int vertex_round(int64_t v, int shift, const int32_t *gid, const int64_t *vbase,
                                            const int32_t *orig) {
    if (orig) return sub_round_of(orig[v], shift);
    return sub_round_of(gid ? v - vbase[gid[v]] : v, shift);
}

__global__ void __launch_bounds__(kBlock) k_bin_count(const int32_t *deg, int64_t n, int rounds, int shift,
                                                     const int32_t *gid, const int64_t *vbase, const int32_t *orig,
                                                     unsigned long long *cnt, unsigned long long *ent) {
    __shared__ unsigned int lcnt[kNumBuckets];
    __shared__ unsigned long long lent[kNumBuckets];
    int nb = kNumBins * rounds;
    for (int k = threadIdx.x; k < nb; k += kBlock) { lcnt[k] = 0; lent[k] = 0; }
    __syncthreads();
    for (int64_t i = blockIdx.x * (int64_t)kBinTile + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBinTile) {
#pragma unroll
        for (int r = 0; r < 4; r++) {
            int64_t v = i + (int64_t)r * kBlock;
            if (v >= n) break;
            int d = deg[v];
            int b = bin_of_degree(d);
            if (b < 0) continue;
            int k = b * rounds + vertex_round(v, shift, gid, vbase, orig);
            atomicAdd(&lcnt[k], 1u);
            atomicAdd(&lent[k], (unsigned long long)d);
        }
    }
    __syncthreads();
    for (int k = threadIdx.x; k < nb; k += kBlock)
        if (lcnt[k]) {
            atomicAdd(&cnt[k], (unsigned long long)lcnt[k]);
            atomicAdd(&ent[k], lent[k]);
        }
}

// The counts to the host's box; cnt[k] becomes the begin of bucket k, so that
// the fill need not wait for the host.
__global__ void __launch_bounds__(kBlock) k_bin_post(unsigned long long *cnt, const unsigned long long *ent, int nb,
                                                    uint64_t *box) {
    __shared__ unsigned long long c[kNumBuckets];
    for (int k = threadIdx.x; k < nb; k += kBlock) {
        c[k] = cnt[k];
        box[kBoxHead + k] = c[k];
        box[kBoxHead + nb + k] = ent[k];
    }
    __syncthreads();
    for (int k = threadIdx.x; k < nb; k += kBlock) {
        unsigned long long b = 0;
        for (int j = 0; j < k; j++) b += c[j];
        cnt[k] = b;
    }
    box_post(box);
}

// Places vertex ids into their buckets.  cursor[k] starts at the bucket's
// begin; each block reserves its slots with one atomic per bucket.
template <int TILE>
__global__ void __launch_bounds__(kBlock) k_bin_fill(const int32_t *deg, int64_t n, int rounds, int shift,
                                                    const int32_t *gid, const int64_t *vbase, const int32_t *orig,
                                                    unsigned long long *cursor, int32_t *bl) {
    __shared__ unsigned int lcnt[kNumBuckets];
    __shared__ unsigned long long lbase[kNumBuckets];
    int nb = kNumBins * rounds;
    for (int64_t t0 = blockIdx.x * (int64_t)TILE; t0 < n; t0 += (int64_t)gridDim.x * TILE) {
        for (int k = threadIdx.x; k < nb; k += kBlock) lcnt[k] = 0;
        __syncthreads();
        int bk[TILE / kBlock];
        unsigned rk[TILE / kBlock];
#pragma unroll
        for (int r = 0; r < TILE / kBlock; r++) {
            int64_t v = t0 + (int64_t)r * kBlock + threadIdx.x;
            bk[r] = -1;
            if (v < n) {
                int b = bin_of_degree(deg[v]);
                if (b >= 0) {
                    bk[r] = b * rounds + vertex_round(v, shift, gid, vbase, orig);
                    rk[r] = atomicAdd(&lcnt[bk[r]], 1u);
                }
            }
        }
        __syncthreads();
        for (int k = threadIdx.x; k < nb; k += kBlock)
            if (lcnt[k]) lbase[k] = atomicAdd(&cursor[k], (unsigned long long)lcnt[k]);
        __syncthreads();
#pragma unroll
        for (int r = 0; r < TILE / kBlock; r++) {
            int64_t v = t0 + (int64_t)r * kBlock + threadIdx.x;
            if (bk[r] >= 0) bl[lbase[bk[r]] + rk[r]] = (int32_t)v;
        }
        __syncthreads();
    }
}

__global__ void __launch_bounds__(kBlock) k_hub_sizes(const int32_t *bl, int64_t hb, int64_t H, const int32_t *deg,
                                                     int64_t *tsize, int64_t *nch, int64_t *bsz) {
    for (int64_t k = blockIdx.x * (int64_t)kBlock + threadIdx.x; k < H; k += (int64_t)gridDim.x * kBlock) {
        int d = deg[bl[hb + k]];
        tsize[k] = (int64_t)hub_table_size(d);
        int64_t c = (d + kHubChunk - 1) / kHubChunk;
        nch[k] = c;
        bsz[k] = c <= kMaxParts ? c * c : 0;   // partition words of the hub
    }
}

// The totals of the hubs' tables, partition words and chunks, and the first
// chunk of each sub-round's hubs (pos: their positions among the hubs).
struct HubPositions {
    int64_t at[kMaxRounds + 1];
};
__global__ void __launch_bounds__(kBlock) k_hub_post(const int64_t *toff, const int64_t *boff, const int64_t *coff,
                                                    int64_t H, HubPositions pos, int rounds, uint64_t *box) {
    static_assert(kMaxRounds + 1 <= kBlock, "a thread per sub-round");
    const int p = threadIdx.x;
    if (p <= rounds) box[kBoxHead + 2 + p] = (uint64_t)coff[pos.at[p]];
    if (p == 0) {
        box[kBoxHead] = (uint64_t)toff[H];
        box[kBoxHead + 1] = (uint64_t)boff[H];
    }
    box_post(box);
}

__global__ void __launch_bounds__(kBlock) k_hub_fill(const int32_t *bl, int64_t hb, int64_t H, const int32_t *deg,
                                                    const int64_t *off, const int64_t *toff, const int64_t *coff,
                                                    const int64_t *boff, int64_t *hub_off, int32_t *hub_ch0,
                                                    int64_t *hub_b0, int32_t *ch_vert, int64_t *ch_beg) {
    for (int64_t k = blockIdx.x * (int64_t)kBlock + threadIdx.x; k < H; k += (int64_t)gridDim.x * kBlock) {
        int32_t i = bl[hb + k];
        hub_off[i] = toff[k];
        hub_b0[i] = boff[k];
        hub_ch0[i] = (int32_t)coff[k];
        int64_t nc = coff[k + 1] - coff[k];
        for (int64_t c = 0; c < nc; c++) {
            ch_vert[coff[k] + c] = i;
            ch_beg[coff[k] + c] = off[i] + c * kHubChunk;
        }
    }
}

}  // namespace

hipError_t bin_vertices(const int32_t *deg, int64_t n, int rounds, WorkLists &wl, Scratch &sc, hipStream_t s,
                        const int32_t *gid, const int64_t *vbase, const int32_t *orig) {
    int shift = 0;
    while ((1 << shift) < rounds) shift++;
    wl.rounds = rounds;
    wl.shift = shift;
    int nb = kNumBins * rounds;
    unsigned long long *cnt = sc.u64;          // nb counters at u64[0..nb)
    unsigned long long *ent = sc.u64 + kNumBuckets;
    const bool wide = n > kBinTiles * kBinTile;
    const int64_t gc = std::min<int64_t>((n + kBinTile - 1) / kBinTile, kBinTiles);
    const int64_t gf = std::min<int64_t>((n + (wide ? kBinWide : kBinTile) - 1) / (wide ? kBinWide : kBinTile), 4096);
    launch_fill_u64(sc.u64, 0, 2 * kNumBuckets, s);
    if (n > 0) k_bin_count<<<(unsigned)gc, kBlock, 0, s>>>(deg, n, rounds, shift, gid, vbase, orig, cnt, ent);
    box_arm(sc.box);
    k_bin_post<<<1, kBlock, 0, s>>>(cnt, ent, nb, sc.box);
    if (n > 0 && wide)
        k_bin_fill<kBinWide><<<(unsigned)gf, kBlock, 0, s>>>(deg, n, rounds, shift, gid, vbase, orig, sc.u64, wl.bl);
    else if (n > 0)
        k_bin_fill<kBinTile><<<(unsigned)gf, kBlock, 0, s>>>(deg, n, rounds, shift, gid, vbase, orig, sc.u64, wl.bl);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = box_wait(sc.box, s);
    if (e != hipSuccess) return e;
    wl.boff[0] = 0;
    for (int k = 0; k < nb; k++) {
        wl.boff[k + 1] = wl.boff[k] + (int64_t)sc.box[kBoxHead + k];
        wl.bucket_entries[k] = (int64_t)sc.box[kBoxHead + nb + k];
    }
    return hipSuccess;
}

hipError_t build_work_lists(const Level &g, int rounds, WorkLists &wl, Scratch &sc, hipStream_t s) {
    hipError_t e = bin_vertices(g.deg, g.n, rounds, wl, sc, s, g.gid, g.vbase, g.orig);
    if (e != hipSuccess) return e;
    // hubs
    int64_t hb = wl.bin_begin(BIN_HUB), H = wl.bin_size(BIN_HUB);
    wl.nchunks = 0;
    wl.hub_table_total = 0;
    for (int p = 0; p <= rounds; p++) wl.ch_poff[p] = 0;
    if (H > 0) {
        unsigned gr = (unsigned)((H + kBlock - 1) / kBlock);
        if (gr > 4096) gr = 4096;
        // table sizes -> offsets
        k_hub_sizes<<<gr, kBlock, 0, s>>>(wl.bl, hb, H, g.deg, sc.i64a, sc.i64c, sc.i64d);
        scan_exclusive_i64(sc.i64a, sc.i64b, H, sc.scan_tmp, s);   // i64b = table offsets
        scan_exclusive_i64(sc.i64c, sc.i64a, H, sc.scan_tmp, s);   // i64a = chunk offsets
        scan_exclusive_i64(sc.i64d, sc.i64e, H, sc.scan_tmp, s);   // i64e = partition word offsets
        HubPositions pos;
        for (int p = 0; p <= rounds; p++)
            pos.at[p] = (p < rounds ? wl.bucket_begin(BIN_HUB, p) : wl.bin_begin(BIN_HUB) + H) - hb;
        box_arm(sc.box);
        k_hub_post<<<1, kBlock, 0, s>>>(sc.i64b, sc.i64e, sc.i64a, H, pos, rounds, sc.box);
        e = hipGetLastError();
        if (e == hipSuccess) e = box_wait(sc.box, s);
        if (e != hipSuccess) return e;
        wl.hub_table_total = sc.box[kBoxHead];
        wl.bucket_total = sc.box[kBoxHead + 1];
        for (int p = 0; p <= rounds; p++) wl.ch_poff[p] = (int64_t)sc.box[kBoxHead + 2 + p];
        wl.nchunks = wl.ch_poff[rounds];
        if (wl.nchunks > sc.ch_cap) return hipErrorInvalidValue;
        e = ensure_hub_tables(sc, wl.hub_table_total, s);
        if (e != hipSuccess) return e;
        e = ensure_hub_buckets(sc, wl.bucket_total, s);
        if (e != hipSuccess) return e;
        k_hub_fill<<<gr, kBlock, 0, s>>>(wl.bl, hb, H, g.deg, g.off, sc.i64b, sc.i64a, sc.i64e, wl.hub_off,
                                         wl.hub_ch0, wl.hub_b0, sc.ch_vert, sc.ch_beg);
    }
    wl.ch_vert = sc.ch_vert;
    wl.ch_beg = sc.ch_beg;
    return hipGetLastError();
}

}  // namespace gsp
