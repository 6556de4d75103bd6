"""Step kernels beyond the launches with few waves, at every narrow block width.

Launches of at most 512 workgroups take a variant of their own, so a mesh of a few thousand nodes never
runs the others.  Here every width runs them: a 195,112-node ball (Sec. 3 eq. (fully-discrete); Sec. 5.1 eq.
(adjoint-verlet)) against the oracle, a Delaunay mesh of 9,000 nodes with rows of up to 89 entries and a boundary
row of 61 entries of B, also against the oracle, and the non-temporal variant on 753,571 nodes against the plain one,
bit for bit.  The kernels that ran are read from a trace.  Bars: rounding only, 1e-11 of the largest output
in float64 and 2e-5 in float32.
"""
import numpy as np
import pytest

import oracle
import workloads as W
from tests._kernels import kernels_of
from tests._meshes import hub_mesh

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
pat = pytest.importorskip("paper_2607_21373_amd.pat")

T32, T64 = ("float", torch.float32, 2e-5), ("double", torch.float64, 1e-11)
WIDTHS = [(R, *T32) for R in (1, 2, 4, 8, 16, 32)] + [(R, *T64) for R in (1, 2, 4, 8, 16)]


def _check(O, G, R, name, dtype, tol, want_f, want_a):
    print(f"{G.n_nodes} nodes R={R} {name}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(R)
    p = torch.randn((R, G.n_nodes), generator=g, dtype=dtype, device="cuda")
    yh = torch.randn((R, G.n_steps, G.n_obs), generator=g, dtype=dtype, device="cuda")
    (nf, y), (na, a) = kernels_of(lambda: pat.pat_forward(G, p)), kernels_of(lambda: pat.pat_adjoint(G, yh))
    assert want_f in nf, nf
    assert want_a in na, na
    k = sorted({0, R // 3, R - 1})
    ry, ra = O.forward(p[k].double().cpu().numpy()), O.adjoint(yh[k].double().cpu().numpy())
    assert np.abs(y[k].double().cpu().numpy() - ry).max() < tol * np.abs(ry).max()
    assert np.abs(a[k].double().cpu().numpy() - ra).max() < tol * np.abs(ra).max()


@pytest.fixture(scope="module")
def ball():
    w = W.make_workload("ball58_batched")
    return oracle.Problem.from_workload(w, n_steps=3), pat.Problem.from_workload(w, n_steps=3)


@pytest.mark.parametrize("R,name,dtype,tol", WIDTHS)
def test_large_mesh(ball, R, name, dtype, tol):
    if R * (4 if name == "float" else 8) < 16:
        want = f"k_fwd<{name}, {name}, {R}, false>", f"k_adj<{name}, {name}, {R}, false>"
    else:
        want = f"k_fwd_v<{name}, {name}, {R}, 0>", f"k_adj_v<{name}, {name}, {R}, 0, false>"
    _check(*ball, R, name, dtype, tol, *want)


@pytest.fixture(scope="module")
def hub():
    x, t = hub_mesh(9000, 0.2, 11)
    rng = np.random.default_rng(3)
    kw = dict(absorbing=True, dt=1e-4, n_steps=4, sensor_pos=x[t[rng.permutation(len(t))[:300]]].mean(1))
    O = oracle.Problem(x, t, **kw)
    rows = np.diff(O.csr("K")[0])
    assert rows.max() > 80 and (rows > 16).sum() > 3000
    return O, pat.Problem(x, t, **kw)


@pytest.mark.parametrize("R,name,dtype,tol", [(64, *T32), (32, *T64), (64, *T64)])
def test_long_rows(hub, R, name, dtype, tol):
    _check(*hub, R, name, dtype, tol, f"k_fwd_v<{name}, {name}, {R}, 0>", f"k_adj_v<{name}, {name}, {R}, 0, false>")


def test_beyond_the_cache():
    x, t = W.ball_mesh(90)
    G = pat.Problem(x, t, None, True, 0.2 * 2.0 / 90, 3, sensor_pos=W.fibonacci_sphere(100, 0.9), check_dt=False)
    print(f"{G.n_nodes} nodes, 32 float32 RHS", flush=True)
    g = torch.Generator(device="cuda").manual_seed(3)
    p = torch.randn((32, G.n_nodes), generator=g, device="cuda")
    yh = torch.randn((32, 3, G.n_obs), generator=g, device="cuda")
    (nf, y), (na, a) = kernels_of(lambda: pat.pat_forward(G, p)), kernels_of(lambda: pat.pat_adjoint(G, yh))
    assert "k_fwd_v<float, float, 32, 1>" in nf and "k_adj_v<float, float, 32, 1, false>" in na
    for c in (0, 16):
        nf, yn = kernels_of(lambda: pat.pat_forward(G, p[c:c + 16].contiguous()))
        na, an = kernels_of(lambda: pat.pat_adjoint(G, yh[c:c + 16].contiguous()))
        assert "k_fwd_v<float, float, 16, 0>" in nf and "k_adj_v<float, float, 16, 0, false>" in na
        assert torch.equal(y[c:c + 16], yn) and torch.equal(a[c:c + 16], an)
