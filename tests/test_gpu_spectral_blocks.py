"""The spectral prior's transforms at the edges of their workgroup shapes, against the oracle.

On grids of 64^3 and more a workgroup transforms 16 (line, right-hand side) pairs, several
lines of a block of up to 8 right-hand sides; on smaller grids and wider blocks one line.
Grids of 8 to 128 points (x passes of 4 to 64 points, with and without a last radix-2 or
radix-4 stage) and blocks of 1, 2, 8 and 16 take every shape; one right-hand side also skips
the layout change of the grid vectors.  Bar: 1e-12 of the largest output.
"""
import numpy as np
import pytest

import workloads as W
from oracle.spectral import SpectralPrior

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
pat = pytest.importorskip("paper_2607_21373_amd.pat")

LO, SIDE, ELL = -1.25, 2.5, 0.3


@pytest.mark.parametrize("n,R", [(8, 2), (16, 1), (16, 16), (32, 8), (64, 1), (64, 2), (64, 7), (64, 16), (128, 1),
                                 (128, 3)])
def test_transform_blocks(n, R):
    w = W.make_workload("ball16")
    G = pat.Problem.from_workload(w)
    prior = SpectralPrior(n, LO, SIDE, ELL, 3.0)
    I = prior.interp_matrix(w.coords)
    pat.spectral_prior_set(G, n, LO, SIDE, ELL, 3.0)
    rng = np.random.default_rng(n + R)
    x, v = rng.standard_normal((R, prior.size)), rng.standard_normal((R, w.n_nodes))
    print(f"spectral n={n} R={R}", flush=True)
    dev = lambda a: torch.as_tensor(a, device="cuda")  # noqa: E731
    y = pat.spectral_apply(G, dev(x)).cpu().numpy()
    g = pat.spectral_apply(G, dev(v), transpose=True).cpu().numpy()
    ry, rg = prior.apply(x, I), prior.apply_t(v, I)
    assert np.abs(y - ry).max() < 1e-12 * np.abs(ry).max()
    assert np.abs(g - rg).max() < 1e-12 * np.abs(rg).max()
