"""Resident sweeps of small meshes with long rows, against the oracle.

A thread keeps the columns of the first twelve entries beyond the sixteen padded slots of its
first row in registers and reads the rest in turns of four: the meshes are Delaunay meshes of
random points with a hub (a node in a hollow ball, joined to everything around it), whose
rows have more than 28 entries, with one row per thread and with two.  Bars: rounding only, 1e-11 of the largest
output in float64 and 2e-5 in float32.
"""
import numpy as np
import pytest
from scipy.spatial import Delaunay

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
pat = pytest.importorskip("paper_2607_21373_amd.pat")


def hub_mesh(n, seed):
    rng = np.random.default_rng(seed)
    d = rng.standard_normal((n - 1, 3))
    r = rng.uniform(0.5 ** 3, 1.0, n - 1) ** (1 / 3)
    x = np.vstack([np.zeros((1, 3)), d / np.linalg.norm(d, axis=1)[:, None] * r[:, None]])
    t = Delaunay(x).simplices.astype(np.int64)
    e = x[t[:, 1:]] - x[t[:, :1]]
    vol = np.linalg.det(e)
    t[vol < 0] = t[vol < 0][:, [0, 2, 1, 3]]
    t = t[np.abs(vol) > 1e-9]
    used = np.unique(t)
    assert used.size == n
    return x, t.astype(np.int32)


@pytest.mark.parametrize("n", [200, 1000, 1030, 1500])
@pytest.mark.parametrize("n_steps", [1, 4])
def test_long_rows(n, n_steps):
    coords, tets = hub_mesh(n, n)
    rng = np.random.default_rng(n_steps)
    kw = dict(absorbing=True, dt=1e-4, n_steps=n_steps, sensor_nodes=rng.permutation(n)[:50].astype(np.int32))
    O, G = oracle.Problem(coords, tets, **kw), pat.Problem(coords, tets, **kw)
    rows = np.diff(O.csr("K")[0])
    assert rows.max() > 28 and (rows > 16).sum() > n // 6
    for R, dtype, tol in ((1, torch.float64, 1e-11), (5, torch.float64, 1e-11), (1, torch.float32, 2e-5),
                          (5, torch.float32, 2e-5)):
        print(f"long rows {n} nodes N_T={n_steps} R={R} {dtype}", flush=True)
        x = rng.standard_normal((R, n))
        yh = rng.standard_normal((R, n_steps, 50))
        y = pat.pat_forward(G, torch.as_tensor(x, dtype=dtype, device="cuda")).double().cpu().numpy()
        a = pat.pat_adjoint(G, torch.as_tensor(yh, dtype=dtype, device="cuda")).double().cpu().numpy()
        ry, ra = O.forward(x), O.adjoint(yh)
        assert np.abs(y - ry).max() < tol * np.abs(ry).max()
        assert np.abs(a - ra).max() < tol * np.abs(ra).max()
