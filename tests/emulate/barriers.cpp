// Kernels whose branches around barriers rest on a value that other
// wavefronts or workgroups change, run on the CPU with each wavefront in turn
// behind the others (see hip/hip_runtime.h), and their results.  KERNELS is a
// kernel source up to its host part.
#include KERNELS

using namespace gsp;

static int fail(const char *what, long at) {
    printf("%s is wrong at %ld\n", what, at);
    return 1;
}

#ifdef TOTALS
// Five tiles and a part per workgroup, more than half a table of communities
// in any three: the tables are emptied before the last tile.
template <bool SIZES>
static int totals(int waves) {
    const int64_t n = 2 * 5 * kKeptThreads * kKeptR + 137;
    const int comm = 60000;
    std::mt19937 r(7);
    std::vector<int32_t> cm(n), size0(comm, 0);
    std::vector<double> K(n), sig0(comm, 0.0);
    for (int64_t i = 0; i < n; i++) {
        cm[i] = (int32_t)(r() % comm);
        K[i] = (double)(r() % 9) / 4.0;
        sig0[cm[i]] += K[i];
        size0[cm[i]]++;
    }
    for (int late = 0; late < waves; late++) {
        std::vector<double> sig(comm, 0.0);
        std::vector<int32_t> size(comm, 0);
        emu::launch(2, kKeptThreads, late,
                    [&] { k_community_totals_kept<SIZES>(K.data(), cm.data(), n, sig.data(), SIZES ? size.data() : nullptr); });
        for (int c = 0; c < comm; c++)
            if (sig[c] != sig0[c] || (SIZES && size[c] != size0[c])) return fail("community", c);
    }
    return 0;
}
static int run(int waves) { return totals<true>(waves) ? 1 : totals<false>(waves); }
#endif

#ifdef HUBS
// A hub of three partitions; at some instant another workgroup, whose
// partition overflowed, marks the hub for its global table.
static int run(int) {
    const int D = 2 * kHubChunk + 500, P = 3, comm = 3000;
    std::mt19937 r(3);
    std::vector<int64_t> off(D + 2), ch_beg = {0, kHubChunk, 2 * kHubChunk}, hub_b0(D + 1, 0);
    std::vector<int32_t> col(D), deg(D + 1, 0), cm(D + 1), csize(D + 1, 1), ch_vert(P, 0);
    std::vector<float> w(D);
    std::vector<double> K(D + 1, 1.0), sig(comm, 0.0), part_g(P), part_kid(P), sval(D);
    std::vector<int> part_c(P), skey(D);
    std::vector<uint32_t> hbuck(P * P);
    std::vector<uint8_t> act(D + 1, 0);
    std::vector<IterCounters> ctr(1);
    deg[0] = D;
    for (int v = 1; v <= D + 1; v++) off[v] = D;
    for (int e = 0; e < D; e++) {
        col[e] = e + 1;
        w[e] = (float)(1 + r() % 7) / 4.0f;
    }
    for (int v = 0; v <= D; v++) cm[v] = (int32_t)(r() % comm);
    for (double &x : sig) x = (double)(r() % 50);
    MoveArgs a = {};
    a.g.n = D + 1;
    a.g.nnz = D;
    a.g.off = off.data();
    a.g.col = col.data();
    a.g.w = w.data();
    a.g.wt = W_F32;
    a.g.deg = deg.data();
    a.K = K.data();
    a.sig = sig.data();
    a.csize = csize.data();
    a.cm = cm.data();
    a.M2 = 64.0;
    a.ctr = ctr.data();
    a.ch_vert = ch_vert.data();
    a.ch_beg = ch_beg.data();
    a.ch_count = P;
    a.hub_act = act.data();
    a.part_g = part_g.data();
    a.part_kid = part_kid.data();
    a.part_c = part_c.data();
    a.max_parts = kMaxParts;
    a.skey = skey.data();
    a.sval = sval.data();
    a.hbuck = hbuck.data();
    a.hub_b0 = hub_b0.data();
    std::vector<double> tot(comm, 0.0), best(P, -INFINITY), kid(P, 0.0);
    std::vector<int> at(P, kIntMax);
    for (int e = 0; e < D; e++) tot[cm[e + 1]] += (double)w[e];
    for (int c = 0; c < comm; c++) {
        if (tot[c] == 0.0) continue;
        const int p = part_of(c, P);
        const double g = a.M2 * tot[c] - K[0] * sig[c];
        if (c == cm[0])
            kid[p] = tot[c];
        else if (better(g, c, best[p], at[p], nullptr)) {
            best[p] = g;
            at[p] = c;
        }
    }
    act[0] = 1;
    emu::launch(P, kBlock, 0, [&] { k_hub_bucket<W_F32>(a); });
    long instants = 1;
    for (long k = 0; k < instants; k++) {
        long now = 0;
        act[0] = 1;
        emu::after_wave = [&](int) {
            if (now++ == k) act[0] = 3;
        };
        emu::launch(1, kBlock, kBlock / kWave - 1, [&] { k_hub_gather<W_F32>(a); });
        emu::after_wave = nullptr;
        instants = now;
        // the hub goes through its global table then, whatever is here; a
        // partition that was gathered is right all the same
        for (int p = 0; p < P && k + 1 == instants; p++)
            if (part_g[p] != best[p] || part_c[p] != at[p] || part_kid[p] != kid[p]) return fail("partition", p);
    }
    return 0;
}
#endif

#ifdef PLACES
// As the totals: members, degrees and places, some members without entries.
static int run(int waves) {
    const int64_t range = 5 * kKeptTile, n = 2 * range - 900;
    const int comm = 60000;
    std::mt19937 r(11);
    std::vector<int32_t> cm(n), deg(n), zero0(comm, 0), full0(comm, 0);
    std::vector<unsigned long long> deg0(comm, 0);
    int64_t nnz = 0;
    for (int64_t i = 0; i < n; i++) {
        cm[i] = (int32_t)(r() % comm);
        deg[i] = (int32_t)(r() % 5);
        nnz += deg[i];
        deg0[cm[i]] += (unsigned long long)deg[i];
        (deg[i] ? full0 : zero0)[cm[i]]++;
    }
    int shift = 1;
    while (nnz >> shift) shift++;
    Level g;
    g.n = n;
    g.nnz = nnz;
    g.deg = deg.data();
    for (int late = 0; late < waves; late++) {
        std::vector<unsigned long long> packed(comm, 0);
        std::vector<int32_t> zero(comm, 0), rank(n, 0x7fffffff);
        emu::launch(2, kKeptThreads, late,
                    [&] { k_agg_count_kept(g, cm.data(), shift, range, packed.data(), zero.data(), rank.data()); });
        std::vector<std::vector<char>> front(comm), back(comm);
        for (int c = 0; c < comm; c++) {
            if (packed[c] >> shift != (unsigned long long)full0[c] || zero[c] != zero0[c] ||
                (packed[c] & ((1ull << shift) - 1)) != deg0[c])
                return fail("community", c);
            front[c].resize((size_t)full0[c]);
            back[c].resize((size_t)zero0[c]);
        }
        for (int64_t i = 0; i < n; i++) {   // every place of a community taken once
            const int at = deg[i] ? rank[i] : ~rank[i];
            std::vector<char> &side = (deg[i] ? front : back)[cm[i]];
            if (at < 0 || at >= (int)side.size() || side[(size_t)at]++) return fail("vertex", i);
        }
    }
    return 0;
}
#endif

int main() { return run(16); }
