"""Halo-tile step kernels where they run: against the oracle and, bit for bit, the vector-lane kernels.

Rows of one to four 256-byte chunks run on halo tiles on meshes of at least three tiles per compute
unit (Sec. 3 eq. (fully-discrete) row by row; Sec. 5.1 eq. (adjoint-verlet)).  The meshes have more:
a ragged box of 31,360 nodes (tiles full, cut by the boundary budget, and a last partial one) and a
Delaunay mesh of 22,000 nodes (tiles cut by the halo's size, rows of up to 92 entries, a boundary row
of 61 entries of B, sensors between nodes).  Sweeps have 1, 2 and 4 steps, so that the start, the
closing launch and the final samples follow the tiles directly.  The kernels that ran are read from a trace.

Both kernel families sum a column over a row's slots in the same order, so a block of 64 float32 (or
32 or 64 float64) columns equals the same columns in narrower blocks bit for bit.  128- and 256-wide
blocks exist in the sampler only: one solver iteration, whose sweeps are bitwise those of a
narrow block, leaves the order of the float64 dot products over at most 3e6 terms: 1e-13.
Bars against the oracle as for the other widths: rounding only, 1e-11 of the largest output in float64
and 2e-5 in float32.
"""
import numpy as np
import pytest

import oracle
import workloads as W
from tests._kernels import bases, kernels_of
from tests._meshes import hub_mesh

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
pat = pytest.importorskip("paper_2607_21373_amd.pat")

_MESH = {}


def _mesh(name):
    if name not in _MESH:
        rng = np.random.default_rng(9)
        if name == "box":
            x, t = W.box_mesh(31, 27, 34, hi=(1.0, 27 / 31, 34 / 31), mirrored=True)
            _MESH[name] = (x, t, dict(dt=0.2 / 31, sensor_nodes=rng.permutation(len(x))[:200].astype(np.int32)))
        else:
            x, t = hub_mesh(22000, 0.12, 4)
            _MESH[name] = (x, t, dict(dt=1e-4, sensor_pos=x[t[rng.permutation(len(t))[:200]]].mean(1)))
    return _MESH[name]


def _run(G, x, yh):
    (nf, y), (na, a) = kernels_of(lambda: pat.pat_forward(G, x)), kernels_of(lambda: pat.pat_adjoint(G, yh))
    return nf, na, y, a


@pytest.mark.parametrize("name", ["box", "hub"])
@pytest.mark.parametrize("n_steps", [1, 2, 4])
@pytest.mark.parametrize("prec,R,narrow,tol", [("float", 64, 32, 2e-5), ("double", 32, 16, 1e-11),
                                               ("double", 64, 16, 1e-11)])
def test_halo_equals_vector_lanes(name, n_steps, prec, R, narrow, tol):
    x, t, kw = _mesh(name)
    kw = dict(kw, absorbing=True, n_steps=n_steps)
    O, G = oracle.Problem(x, t, **kw), pat.Problem(x, t, **kw)
    print(f"halo {name} {G.n_nodes} nodes N_T={n_steps} {prec} R={R}", flush=True)
    dt = torch.float32 if prec == "float" else torch.float64
    g = torch.Generator(device="cuda").manual_seed(R + n_steps)
    p = torch.randn((R, G.n_nodes), generator=g, dtype=dt, device="cuda")
    yh = torch.randn((R, n_steps, G.n_obs), generator=g, dtype=dt, device="cuda")
    nf, na, y, a = _run(G, p, yh)
    assert f"k_halo<{prec}, {prec}, true, false, {R}, false>" in nf
    assert f"k_halo<{prec}, {prec}, false, true, {R}, false>" in na  # the closing launch
    assert n_steps == 1 or f"k_halo<{prec}, {prec}, false, false, {R}, false>" in na
    for c in range(0, R, narrow):
        nf, na, yn, an = _run(G, p[c:c + narrow].contiguous(), yh[c:c + narrow].contiguous())
        assert "k_halo" not in bases(nf | na) and bases(nf) >= {"k_fwd_v"} and bases(na) >= {"k_adj_v"}
        assert torch.equal(y[c:c + narrow], yn) and torch.equal(a[c:c + narrow], an)
    k = [0, R // 2 + 1, R - 1]
    ry, ra = O.forward(p[k].double().cpu().numpy()), O.adjoint(yh[k].double().cpu().numpy())
    assert np.abs(y[k].double().cpu().numpy() - ry).max() < tol * np.abs(ry).max()
    assert np.abs(a[k].double().cpu().numpy() - ra).max() < tol * np.abs(ra).max()


@pytest.mark.parametrize("name", ["box", "hub"])
@pytest.mark.parametrize("prec,R,narrow", [("f32", 128, 32), ("f32", 256, 32), ("f64", 64, 16), ("f64", 128, 16)])
def test_wide_halo_blocks(name, prec, R, narrow):
    x, t, kw = _mesh(name)
    G = pat.Problem(x, t, **dict(kw, absorbing=True, n_steps=5))
    print(f"halo blocks {name} {prec} R={R}", flush=True)
    yobs = torch.randn((5, G.n_obs), generator=torch.Generator(device="cuda").manual_seed(R), dtype=torch.float64,
                       device="cuda")

    def go(rb):
        return pat.rto_sample(G, yobs, None, None, 0.1, 0.01, 1, sweep_prec=prec, rhs_block=rb, n_samples=R, seed=2)

    names, wide = kernels_of(lambda: go(R))
    T = "float" if prec == "f32" else "double"
    for d in ("true, false", "false, false", "false, true"):
        assert f"k_halo<{T}, double, {d}, {R}, false>" in names
    names, ref = kernels_of(lambda: go(narrow))
    assert "k_halo" not in bases(names)
    d = torch.linalg.vector_norm(wide["samples"] - ref["samples"], dim=1) / torch.linalg.vector_norm(ref["samples"], dim=1)
    assert float(d.max()) < 1e-13


def test_halo_beyond_the_cache():
    """64 float64 RHS on 195,112 nodes: three states of 100 MB, own rows loaded and stored non-temporally."""
    w = W.make_workload("ball58_batched")
    G = pat.Problem.from_workload(w, n_steps=3)
    print("halo, 300 MB of states", flush=True)
    g = torch.Generator(device="cuda").manual_seed(1)
    p = torch.randn((64, G.n_nodes), generator=g, dtype=torch.float64, device="cuda")
    yh = torch.randn((64, 3, G.n_obs), generator=g, dtype=torch.float64, device="cuda")
    nf, na, y, a = _run(G, p, yh)
    assert "k_halo<double, double, true, false, 64, true>" in nf
    assert "k_halo<double, double, false, false, 64, true>" in na
    for c in range(0, 64, 16):
        nf, na, yn, an = _run(G, p[c:c + 16].contiguous(), yh[c:c + 16].contiguous())
        assert "k_halo" not in bases(nf | na)
        assert torch.equal(y[c:c + 16], yn) and torch.equal(a[c:c + 16], an)
