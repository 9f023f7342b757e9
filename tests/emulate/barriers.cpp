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
