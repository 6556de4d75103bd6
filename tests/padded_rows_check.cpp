// Checks the padded row layout of the step kernels (pat::build_padded_rows) on a mesh read from a
// binary file written by test_padded_rows.py: every row's slots and further entries are its CSR
// entries, the diagonal first, and a boundary row's B values start on a multiple of four, since the
// kernels load them four at a time.
#include <cstdio>
#include <map>
#include <string>

#include "mesh_file.h"

int main(int argc, char **argv) {
    pat::HostProblem hp;
    std::string err;
    if (argc < 2 || !read_problem(argv[1], hp, err)) {
        std::printf("FAIL %s\n", err.c_str());
        return 1;
    }
    const int W = pat::HostProblem::kEll;
    int bnd = 0, over = 0;
    for (int32_t i = 0; i < hp.n; ++i) {
        auto fail = [&](const char *what) {
            std::printf("FAIL row %d: %s\n", i, what);
            return 1;
        };
        const int32_t k0 = hp.rowptr[size_t(i)], len = hp.rowptr[size_t(i) + 1] - k0;
        const int32_t x0 = hp.xptr[size_t(i)], nx = hp.xptr[size_t(i) + 1] - x0, bo = hp.bsoff[size_t(i)];
        const bool b = hp.boff[size_t(i)] >= 0;
        if (nx != (len > W ? len - W : 0)) return fail("entries beyond the slots");
        if (b != (bo >= 0)) return fail("boundary row");
        if (b && bo % 4) return fail("B values not on a multiple of four");
        if (b && size_t(bo) + size_t(W) + size_t((nx + 3) / 4 * 4) > hp.bslot.size()) return fail("B values end");
        std::map<int32_t, std::pair<double, double>> want;
        for (int32_t k = 0; k < len; ++k)
            want[hp.col[size_t(k0 + k)]] = {hp.kval[size_t(k0 + k)],
                                            b ? hp.bval[size_t(hp.boff[size_t(i)] + k)] : 0.0};
        if (hp.ell_col[size_t(i) * W] != i) return fail("diagonal first");
        for (int32_t j = 0; j < W + nx; ++j) {
            const int32_t c = j < W ? hp.ell_col[size_t(i) * W + size_t(j)] : hp.xcol[size_t(x0 + j - W)];
            const double v = j < W ? hp.ell_val[size_t(i) * W + size_t(j)] : hp.xval[size_t(x0 + j - W)];
            if (j >= len) {
                if (c != i || v != 0.0) return fail("padding");
                continue;
            }
            const auto it = want.find(c);
            if (it == want.end() || it->second.first != v) return fail("K entry");
            if (b && it->second.second != hp.bslot[size_t(bo + j)]) return fail("B entry");
            if (b && (j < hp.bnum[size_t(i)]) != (it->second.second != 0.0) && j > 0) return fail("B order");
            want.erase(it);
        }
        if (!want.empty()) return fail("missing entries");
        bnd += b;
        over += b && nx % 4;
    }
    std::printf("OK boundary rows %d, with a ragged end %d\n", bnd, over);
    return 0;
}
