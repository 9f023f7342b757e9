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

int main() { return run(16); }
