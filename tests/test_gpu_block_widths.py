"""Every block width of the step kernels against the oracle, on a mesh with remainders everywhere.

A block of R right-hand sides runs on lane groups of 1 to 64 lanes per row (Sec. 3
eq. (fully-discrete); Sec. 5.1 eq. (adjoint-verlet)), so tiles hold 256 down to a few
rows.  The mesh (18^3 nodes, no multiple of any tile) ends every launch in a partial
tile and has rows with more than the padded 16 entries, boundary rows and rows with
sensor weights.  Bars as for the short sweeps: rounding only, 1e-11 of the largest
output in float64 and 2e-5 in float32.
"""
import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
pat = pytest.importorskip("paper_2607_21373_amd.pat")

_CACHE = {}


def _problem(cells, n_steps):
    if (cells, n_steps) not in _CACHE:
        coords, tets = W.ball_mesh(cells)
        kw = dict(c_tet=W.wave_speed_bumps(coords, tets), absorbing=True, dt=0.2 * 2.0 / cells, n_steps=n_steps,
                  sensor_pos=W.fibonacci_sphere(70, 0.9))
        _CACHE[cells, n_steps] = (oracle.Problem(coords, tets, **kw), pat.Problem(coords, tets, **kw))
    return _CACHE[cells, n_steps]


def _check(O, G, R, dtype, tol):
    rng = np.random.default_rng(R)
    x = rng.standard_normal((R, G.n_nodes))
    yh = rng.standard_normal((R, G.n_steps, G.n_obs))
    y = pat.pat_forward(G, torch.as_tensor(x, dtype=dtype, device="cuda")).double().cpu().numpy()
    a = pat.pat_adjoint(G, torch.as_tensor(yh, dtype=dtype, device="cuda")).double().cpu().numpy()
    ry, ra = O.forward(x), O.adjoint(yh)
    assert np.abs(y - ry).max() < tol * np.abs(ry).max()
    assert np.abs(a - ra).max() < tol * np.abs(ra).max()


@pytest.mark.parametrize("dtype,tol", [(torch.float64, 1e-11), (torch.float32, 2e-5)])
@pytest.mark.parametrize("R", [1, 2, 4, 8, 16, 32])
def test_block_widths(R, dtype, tol):
    O, G = _problem(17, 6)
    print(f"block width {R} {dtype}", flush=True)
    _check(O, G, R, dtype, tol)


# Whole 256-byte chunks on a mesh with enough halo tiles (24,389 nodes) run the halo-tile
# kernels: one, two and four chunks per row.
@pytest.mark.parametrize("R,dtype,tol", [(32, torch.float64, 1e-11), (64, torch.float64, 1e-11),
                                         (64, torch.float32, 2e-5)])
def test_halo_widths(R, dtype, tol):
    O, G = _problem(28, 3)
    print(f"halo width {R} {dtype}", flush=True)
    _check(O, G, R, dtype, tol)
