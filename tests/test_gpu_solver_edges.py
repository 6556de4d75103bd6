"""CGLS and LSQR against the oracle at the edges of their reductions.

The basis products take eight vectors per pass and the Gram row one thread per (vector,
right-hand side): 1, 2, 8, 9, 16 and 18 iterations sit on both sides of one and two passes.
The norms and the scalar stages run on 256 / RB threads per right-hand side: blocks of 1, 4
and 64, on a mesh of fewer rows than the reductions have workgroups x threads.  Bar: the
float64 solver's 1e-10 (samples in relative L2, residual norms against the largest).
"""
import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
pat = pytest.importorskip("paper_2607_21373_amd.pat")


@pytest.fixture(scope="module")
def tiny():
    w = W.make_workload("cube8_tiny")
    return w, oracle.Problem.from_workload(w), pat.Problem.from_workload(w)


@pytest.mark.parametrize("solver", ["cgls", "lsqr"])
@pytest.mark.parametrize("n_iter,S,rb", [(1, 1, 1), (2, 3, 4), (8, 2, 1), (9, 5, 4), (16, 64, 64), (18, 1, 1)])
def test_reduction_edges(tiny, solver, n_iter, S, rb):
    w, O, G = tiny
    _, yobs, sigma = oracle.synthesize(O, w)
    eta, xi = W.rto_draws(S, w.n_steps, w.n_obs, w.n_nodes, w.rto_seed)
    ref, rres, rdg = O.rto(yobs, sigma, w.prior_a, n_iter, eta, xi, solver=solver, diag=True)
    print(f"{solver} n_iter={n_iter} S={S} rb={rb}", flush=True)
    dev = lambda a: torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")  # noqa: E731
    out = pat.rto_sample(G, dev(yobs), dev(eta), dev(xi), sigma, w.prior_a, n_iter, sweep_prec="f64", rhs_block=rb,
                         resid=True, solver=solver, diag=True)
    got = {k: out[k].cpu().numpy() for k in ("samples", "resid", "diag")}
    assert np.linalg.norm(got["samples"] - ref) < 1e-10 * np.linalg.norm(ref)
    assert np.abs(got["resid"] - rres).max() < 1e-10 * np.abs(rres).max()
    assert np.abs(got["diag"] - rdg).max() < 1e-10 * np.abs(rdg).max()
