"""Meshes of up to 2,048 nodes that a one-launch sweep cannot hold run on step launches.

More than 1,024 sensors (one thread each), a boundary row with more than sixteen entries of B, or tables
beyond the 160 KiB of LDS (2,028 float64 nodes): forward and transposed sweeps (Sec. 3 eq.
(fully-discrete); Sec. 5.1 eq. (adjoint-verlet)) against the oracle, with the kernels read from a trace.
Bars: rounding only, 1e-11 of the largest output in float64 and 2e-5 in float32.
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


def _problem(case):
    if case == "boundary hub":
        x, t = hub_mesh(1500, 0.25, 5)
        kw = dict(dt=1e-4, sensor_nodes=np.arange(0, 1500, 31, dtype=np.int32))
    else:
        c = (10, 10, 10) if "sensors" in case else (12, 12, 11)
        x, t = W.box_mesh(*c, hi=(1.0, c[1] / c[0], c[2] / c[0]), mirrored=True)
        n_obs = int(case.split()[0]) if "sensors" in case else 60
        kw = dict(dt=0.2 / c[0], sensor_nodes=np.random.default_rng(1).permutation(len(x))[:n_obs].astype(np.int32))
    kw.update(absorbing=True, n_steps=4)
    return oracle.Problem(x, t, **kw), pat.Problem(x, t, **kw)


@pytest.mark.parametrize("case,resident", [("1024 sensors", "f32"), ("1025 sensors", ""), ("boundary hub", ""),
                                           ("2028 nodes", "f32")])
def test_refused(case, resident):
    O, G = _problem(case)
    for R, name, tol in ((1, "f64", 1e-11), (5, "f64", 1e-11), (1, "f32", 2e-5), (5, "f32", 2e-5)):
        print(f"small mesh, {case}: R={R} {name}", flush=True)
        dtype = torch.float64 if name == "f64" else torch.float32
        g = torch.Generator(device="cuda").manual_seed(R)
        p = torch.randn((R, G.n_nodes), generator=g, dtype=dtype, device="cuda")
        yh = torch.randn((R, 4, G.n_obs), generator=g, dtype=dtype, device="cuda")
        (nf, y), (na, a) = kernels_of(lambda: pat.pat_forward(G, p)), kernels_of(lambda: pat.pat_adjoint(G, yh))
        small = "k_fwd_small" in bases(nf)
        assert small == ("k_adj_small" in bases(na))
        if case != "1024 sensors" or name == "f32":
            assert small == (name == resident)
        ry, ra = O.forward(p.double().cpu().numpy()), O.adjoint(yh.double().cpu().numpy())
        assert np.abs(y.double().cpu().numpy() - ry).max() < tol * np.abs(ry).max()
        assert np.abs(a.double().cpu().numpy() - ra).max() < tol * np.abs(ra).max()
