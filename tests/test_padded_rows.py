"""The padded row layout of the step kernels (host setup) against the assembled matrices.

The kernels hold a row of K and B (Sec. 3 eq. (discrete-wave-matrix), row by row) as sixteen padded
slots and the entries beyond, and load values four at a time.  A small checker, compiled against the
library's host setup, compares the layout with the CSR arrays on a structured box and on Delaunay
meshes whose boundary rows end at any count of entries.
"""
import os
import shutil
import subprocess

import numpy as np
import pytest
from scipy.spatial import Delaunay

import workloads as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2607_21373_amd", "csrc")


def delaunay_mesh(n, seed):
    """Random points in the unit ball: boundary rows of some 10 to 30 entries."""
    rng = np.random.default_rng(seed)
    d = rng.standard_normal((n, 3))
    x = d / np.linalg.norm(d, axis=1)[:, None] * rng.uniform(0.0, 1.0, n)[:, None] ** (1 / 3)
    t = Delaunay(x).simplices.astype(np.int64)
    vol = np.linalg.det(x[t[:, 1:]] - x[t[:, :1]])
    t[vol < 0] = t[vol < 0][:, [0, 2, 1, 3]]
    t = t[np.abs(vol) > 1e-9]
    assert np.unique(t).size == n
    return x, t.astype(np.int32)


def write_mesh(path, coords, tets, n_obs=20):
    c = np.ones(len(tets))
    sp = coords[tets[:: max(1, len(tets) // n_obs)][:n_obs]].mean(1)
    with open(path, "wb") as f:
        for a in (np.int32(len(coords)), np.int64(len(tets)), np.ascontiguousarray(coords, np.float64),
                  np.ascontiguousarray(tets, np.int32), c, np.int32(len(sp)), sp, np.float64(1e-4), np.int32(3)):
            f.write(a.tobytes())


def compile_check(tmp, name):
    if shutil.which("g++") is None:
        pytest.skip("no host C++ compiler")
    out = str(tmp / name)
    subprocess.run(["g++", "-O1", "-std=c++17", "-pthread", "-I", CSRC, "-I", os.path.join(ROOT, "include"),
                    os.path.join(ROOT, "tests", name + ".cpp"), os.path.join(CSRC, "pat_setup.cpp"), "-o", out],
                   check=True)
    return out


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    return compile_check(tmp_path_factory.mktemp("rows"), "padded_rows_check")


@pytest.mark.parametrize("mesh", ["box", 300, 1500])
def test_padded_rows(checker, tmp_path, mesh):
    coords, tets = W.box_mesh(7, 6, 5) if mesh == "box" else delaunay_mesh(mesh, mesh)
    path = str(tmp_path / "mesh.bin")
    write_mesh(path, coords, tets)
    r = subprocess.run([checker, path], capture_output=True, text=True)
    print(r.stdout.strip())
    assert r.returncode == 0 and r.stdout.startswith("OK"), r.stdout + r.stderr
    if mesh != "box":
        assert int(r.stdout.split()[-1]) > 10  # rows after which a running offset would be off
