"""The launch modes of a batch do what pat_batch_merge says, also with meshes whose sweeps run in one launch.

1 merges the steps of all meshes, 0 launches every mesh's step in turn, 2 runs each mesh's whole
sweep in turn, and only there a mesh of up to 2,048 nodes runs its sweep in one launch (Sec. 3 eq.
(fully-discrete); Sec. 5.1 eq. (adjoint-verlet)).  The kernels that ran are read from a trace.
Whatever the mode, the samples equal those of each mesh alone, bit for bit: float32 and float64
blocks, 128 and 256 wide ones, meshes with partial tiles on every side.
"""
import numpy as np
import pytest

import workloads as W
from tests._kernels import bases, kernels_of

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
pat = pytest.importorskip("paper_2607_21373_amd.pat")

STEPS = 6
SWEEPS = {"k_fwd", "k_adj", "k_fwd_v", "k_adj_v", "k_fwd_vm", "k_adj_vm", "k_fwd_small", "k_adj_small", "k_halo"}
MERGED, TURNS, WHOLE = {"k_fwd_vm", "k_adj_vm"}, {"k_fwd_v", "k_adj_v"}, {"k_fwd_small", "k_adj_small"}


def _box(nx, ny, nz):
    h = 1.0 / nx
    x, t = W.box_mesh(nx, ny, nz, hi=(1.0, ny * h, nz * h), mirrored=True)
    nodes = np.random.default_rng(nx).permutation(len(x))[:40].astype(np.int32)
    return pat.Problem(x, t, None, True, 0.2 * h, STEPS, sensor_nodes=nodes)


@pytest.fixture(scope="module")
def meshes():
    """Two meshes that run a sweep in one launch (729 and 864 nodes), three that do not (2,508, 4,913, 5,985)."""
    return {n: _box(*c) for n, c in dict(a=(8, 8, 8), b=(11, 11, 5), c=(10, 11, 18), d=(16, 16, 16),
                                         e=(18, 14, 20)).items()}


def _run(B, probs, prec, rb, S):
    g = torch.Generator(device="cuda").manual_seed(5)
    ys = [torch.randn((STEPS, p.n_obs), generator=g, device="cuda", dtype=torch.float64) for p in probs]
    kw = dict(sweep_prec=prec, rhs_block=rb)
    names, outs = kernels_of(lambda: pat.rto_sample_batch(B, ys, None, None, 0.1, 0.01, 3, n_samples=S,
                                                          seed=[1, 2, 3][:len(probs)], **kw))
    for m, (p, y) in enumerate(zip(probs, ys)):
        ref = pat.rto_sample(p, y, None, None, 0.1, 0.01, 3, n_samples=S[m], seed=m + 1, **kw)
        assert torch.equal(outs[m]["samples"], ref["samples"]), (prec, rb, m)
    return bases(names) & SWEEPS


@pytest.mark.parametrize("mode,expect", [(1, MERGED), (0, TURNS), (2, WHOLE | TURNS)])
@pytest.mark.parametrize("prec,rb", [("f32", 8), ("f64", 4)])
def test_forced_modes(meshes, mode, expect, prec, rb):
    probs = [meshes[n] for n in "acb"]
    print(f"batch mode {mode} {prec} rb={rb}", flush=True)
    B = pat.Batch(probs)
    B.merge(mode, mode)
    assert _run(B, probs, prec, rb, [5, 3, 2]) == expect


@pytest.mark.parametrize("prec,rb", [("f32", 4), ("f32", 32), ("f64", 8), ("f32", 128), ("f32", 256), ("f64", 128)])
def test_merged_blocks(meshes, prec, rb):
    """Merged launches of three meshes beyond the one-launch sweeps, up to the widest blocks."""
    probs = [meshes[n] for n in "dce"]
    print(f"merged {prec} rb={rb}", flush=True)
    B = pat.Batch(probs)
    B.merge(1, 1)
    assert _run(B, probs, prec, rb, [rb - 1, rb // 2 + 1, 3]) == MERGED


@pytest.mark.parametrize("names,prec,rb,expect", [
    ("acb", "f32", 8, MERGED),          # the small meshes' tiles ride along with the larger one's
    ("ab", "f32", 8, WHOLE),            # nothing to ride along with
    ("ad", "f32", 8, WHOLE | TURNS),    # one row per thread beside launches with few waves
    ("bc", "f64", 16, WHOLE | TURNS),
    ("acb", "f32", 2, WHOLE | {"k_fwd", "k_adj"}),  # too narrow to merge
    ("cd", "f32", 8, MERGED),
])
def test_untuned_modes(meshes, names, prec, rb, expect):
    probs = [meshes[n] for n in names]
    print(f"untuned {names} {prec} rb={rb}", flush=True)
    assert _run(pat.Batch(probs), probs, prec, rb, [rb, 1, 1][:len(probs)]) == expect


def test_untuned_with_halo_tiles():
    """A merged launch has no halo tiles: a mesh that has them and a small one take turns."""
    probs = [_box(8, 8, 8), _box(30, 30, 30)]
    print("untuned with halo tiles", flush=True)
    assert _run(pat.Batch(probs), probs, "f32", 64, [3, 2]) >= WHOLE | {"k_halo"}


def test_tuned_mode_runs(meshes):
    probs = [meshes[n] for n in "acb"]
    B = pat.Batch(probs)
    rb, us = B.autotune(8, "f32")
    print(f"tuned rb={rb} {us:.1f} us", flush=True)
    assert rb in (1, 2, 4, 8) and 0 < us < 1e6
    _run(B, probs, "f32", rb, [8, 5, 2])
