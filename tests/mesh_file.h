// Host problem of a mesh file as the host checks of the test suite read it: N (int32), E (int64),
// coordinates, tets, wave speeds, number of sensors (int32), sensor positions, dt, N_T (int32).
#pragma once

#include <cstdio>
#include <string>
#include <vector>

#include "pat_internal.h"

inline bool read_problem(const char *path, pat::HostProblem &hp, std::string &err) {
    FILE *f = std::fopen(path, "rb");
    if (!f) return err = "cannot open mesh", false;
    int32_t N = 0, nobs = 0, nsteps = 0;
    int64_t E = 0;
    double dt = 0;
    bool ok = std::fread(&N, 4, 1, f) == 1 && std::fread(&E, 8, 1, f) == 1;
    std::vector<double> coords(size_t(N) * 3), c(static_cast<size_t>(E));
    std::vector<int32_t> tets(size_t(E) * 4);
    ok = ok && std::fread(coords.data(), 8, coords.size(), f) == coords.size();
    ok = ok && std::fread(tets.data(), 4, tets.size(), f) == tets.size();
    ok = ok && std::fread(c.data(), 8, c.size(), f) == c.size();
    ok = ok && std::fread(&nobs, 4, 1, f) == 1;
    std::vector<double> sp(size_t(nobs) * 3);
    ok = ok && std::fread(sp.data(), 8, sp.size(), f) == sp.size();
    ok = ok && std::fread(&dt, 8, 1, f) == 1 && std::fread(&nsteps, 4, 1, f) == 1;
    std::fclose(f);
    if (!ok) return err = "short mesh file", false;
    pat_problem_desc d{};
    d.n_nodes = N; d.coords = coords.data(); d.n_tets = E; d.tets = tets.data(); d.c_tet = c.data();
    d.absorbing = 1; d.n_obs = nobs; d.sensor_pos = sp.data(); d.dt = dt; d.n_steps = nsteps;
    d.device = -1; d.check_dt = 0;
    return pat::build_host_problem(d, hp, err) == PAT_OK;
}
