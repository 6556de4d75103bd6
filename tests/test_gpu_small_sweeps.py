"""Resident sweeps of small meshes against the oracle, at the edges of what they take.

A mesh of up to 2048 nodes runs a whole sweep in one launch (Sec. 3 eq. (fully-discrete);
Sec. 5.1 eq. (adjoint-verlet)): one workgroup per right-hand side, one or two rows per
thread of 1024, the sensor data prefetched three sample times ahead.  The meshes sit on
both sides of one row per thread (1000, 1008 and 1056 nodes) and of the two-row limit (2028
and 2100), the sweeps have 1 to 8 steps, and the blocks take both orders of summation (one
right-hand side, and five).  Bars: rounding only, 1e-11 of the largest output in float64 and
2e-5 in float32.
"""
import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
pat = pytest.importorskip("paper_2607_21373_amd.pat")


@pytest.mark.parametrize("cells", [(2, 2, 2), (9, 9, 9), (13, 8, 7), (10, 11, 7), (12, 12, 11), (13, 14, 9)])
@pytest.mark.parametrize("n_steps", [1, 2, 3, 5, 8])
def test_small_sweeps(cells, n_steps):
    nx, ny, nz = cells
    h = 1.0 / nx
    coords, tets = W.box_mesh(nx, ny, nz, hi=(1.0, ny * h, nz * h), mirrored=True)
    rng = np.random.default_rng(nx + n_steps)
    n_obs = min(100, coords.shape[0] // 2)
    kw = dict(absorbing=True, dt=0.2 * h, n_steps=n_steps,
              sensor_nodes=rng.permutation(coords.shape[0])[:n_obs].astype(np.int32))
    O, G = oracle.Problem(coords, tets, **kw), pat.Problem(coords, tets, **kw)
    for R, dtype, tol in ((1, torch.float64, 1e-11), (5, torch.float64, 1e-11), (1, torch.float32, 2e-5),
                          (5, torch.float32, 2e-5)):
        print(f"small sweep {coords.shape[0]} nodes N_T={n_steps} R={R} {dtype}", flush=True)
        x = rng.standard_normal((R, G.n_nodes))
        yh = rng.standard_normal((R, n_steps, n_obs))
        y = pat.pat_forward(G, torch.as_tensor(x, dtype=dtype, device="cuda")).double().cpu().numpy()
        a = pat.pat_adjoint(G, torch.as_tensor(yh, dtype=dtype, device="cuda")).double().cpu().numpy()
        ry, ra = O.forward(x), O.adjoint(yh)
        assert np.abs(y - ry).max() < tol * np.abs(ry).max()
        assert np.abs(a - ra).max() < tol * np.abs(ra).max()
