// Checks the tables of the step kernels as the device holds them (pat::build_device_rows,
// pat::build_device_tiles) against the plain layouts, on a mesh read from a binary file written by
// test_device_rows.py.
#include <cstdio>
#include <cstring>
#include <string>

#include "mesh_file.h"

static int fail(const std::string &m) {
    std::printf("FAIL %s\n", m.c_str());
    return 1;
}

int main(int argc, char **argv) {
    pat::HostProblem hp;
    std::string err;
    if (argc < 2 || !read_problem(argv[1], hp, err)) return fail(err);
    pat::DeviceRows dr;
    pat::build_device_rows(hp, dr);
    pat::HaloTiles ht;
    pat::build_halo_tiles(hp, ht);
    pat::DeviceTiles dt;
    pat::build_device_tiles(hp, ht, dt);
    const size_t N = size_t(hp.n), W = pat::HostProblem::kEll;
    if (dr.ell_col.size() != N * W || dr.ell_val.size() != N * W || dr.bslot.size() != hp.bslot.size() ||
        dr.rspec.size() != N || dr.spec.size() % 2)
        return fail("sizes");
    if (dr.rdir.size() != (hp.n <= pat::kFewRows ? N : 0)) return fail("records by row");
    auto quad = [](size_t j) { return 4 * (j % 4) + j / 4; };  // place of slot j
    int32_t bnd = 0, nb = 0, most = 0, special = 0;
    for (size_t i = 0; i < N; ++i) {
        const std::string at = "row " + std::to_string(i) + ": ";
        const int32_t bo = hp.bsoff[i], x0 = hp.xptr[i], x1 = hp.xptr[i + 1], e0 = hp.injptr[i], e1 = hp.injptr[i + 1];
        for (size_t j = 0; j < W; ++j) {
            if (dr.ell_col[i * W + quad(j)] != hp.ell_col[i * W + j]) return fail(at + "column");
            if (dr.ell_val[i * W + quad(j)] != hp.ell_val[i * W + j]) return fail(at + "K value");
            if (bo >= 0 && dr.bslot[size_t(bo) + quad(j)] != hp.bslot[size_t(bo) + j]) return fail(at + "B value");
        }
        if (bo >= 0)
            for (size_t j = W; j < W + size_t(x1 - x0); ++j)
                if (dr.bslot[size_t(bo) + j] != hp.bslot[size_t(bo) + j]) return fail(at + "B value beyond the slots");
        const bool any = bo >= 0 || x1 > x0 || e1 > e0;
        if (any != (dr.rspec[i] != 0)) return fail(at + "record");
        const pat::Int4 zero{0, 0, 0, 0}, *r = any ? &dr.spec[2 * size_t(dr.rspec[i] - 1)] : nullptr;
        if (!dr.rdir.empty() && std::memcmp(&dr.rdir[i], any ? r : &zero, sizeof zero)) return fail(at + "record by row");
        if (!any) continue;
        if (dr.rspec[i] != ++special) return fail(at + "record order");
        if (r[0].x != (bo >= 0 ? bo : 0) || r[0].y != hp.bnum[i] || r[0].z != x0 || r[0].w != x1) return fail(at + "first half");
        if (r[1].x != e0 || r[1].y != e1 || r[1].z != bnd) return fail(at + "second half");
        bnd += bo >= 0;
        nb = std::max(nb, hp.bnum[i]);
        most = std::max(most, std::max(x1 - x0, e1 - e0));
    }
    if (dr.n_bnd != bnd || dr.max_nb != nb || dr.max_spec != most || dr.spec.size() != 2 * size_t(special))
        return fail("counts");
    // the order of the one-launch sweeps, only where they may run
    if (dr.order.size() != (hp.n <= pat::kSmallRows ? N : 0) || dr.pos.size() != dr.order.size()) return fail("order");
    auto kind = [&](size_t i) {
        return (hp.xptr[i + 1] > hp.xptr[i]) * 4 + (hp.bsoff[i] >= 0) * 2 + (hp.injptr[i + 1] > hp.injptr[i]);
    };
    for (size_t k = 0; k < dr.order.size(); ++k) {
        const size_t i = size_t(dr.order[k]);
        if (dr.pos[i] != int32_t(k)) return fail("order: inverse");
        if (k && kind(size_t(dr.order[k - 1])) < kind(i)) return fail("order: kinds");
    }
    // halo tiles: the metadata blocks lie one after another, 96 bytes a row and 80 a boundary row
    if (dt.desc.size() != size_t(ht.n_tiles)) return fail("tiles");
    int32_t rank = 0;
    for (size_t t = 0; t < dt.desc.size(); ++t) {
        const pat::Int4 d = dt.desc[t];
        const int32_t *D = &ht.desc[4 * t];
        const std::string at = "tile " + std::to_string(t) + ": ";
        if (d.x != D[0] || d.y != D[1] || d.w != D[3]) return fail(at + "descriptor");
        if (d.z != rank) return fail(at + "boundary rank");
        if (int64_t(D[2]) != int64_t(d.x) * 6 + int64_t(d.z) * 5) return fail(at + "metadata place");
        const int32_t nr = D[3] & ((1 << pat::HaloTiles::kNrBits) - 1);
        for (int32_t i = d.x; i < d.x + nr; ++i)
            if (hp.bsoff[size_t(i)] >= 0) {
                for (size_t j = 0; j < W; ++j)
                    if (dt.bw[size_t(rank) * W + j] != hp.bslot[size_t(hp.bsoff[size_t(i)]) + j])
                        return fail(at + "B value");
                ++rank;
            }
    }
    if (ht.n_tiles && (rank != bnd || dt.bw.size() != size_t(bnd) * W)) return fail("boundary rows of the tiles");
    std::printf("OK rows %d special %d boundary %d tiles %d\n", hp.n, special, bnd, ht.n_tiles);
    return 0;
}
