"""The step kernels' tables as the device holds them (host setup) against the plain row layout.

Rows of K and B (Sec. 3 eq. (discrete-wave-matrix), row by row) go to the device with their slots in
quad order, a record for every row with more than its slots, and the halo tiles' descriptors and
float64 boundary values.  bench.py's stored memory traffic holds for one such layout: the files that
build it are in the hash that the stored counters carry.
"""
import os
import subprocess

import pytest

import bench
import workloads as W
from tests.test_padded_rows import CSRC, compile_check, delaunay_mesh, write_mesh


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    return compile_check(tmp_path_factory.mktemp("rows"), "device_rows_check")


@pytest.mark.parametrize("mesh", ["box", "ball", 300, 2500])
def test_device_rows(checker, tmp_path, mesh):
    coords, tets = (W.box_mesh(7, 6, 5) if mesh == "box" else W.ball_mesh(16) if mesh == "ball" else
                    delaunay_mesh(mesh, mesh))
    path = str(tmp_path / "mesh.bin")
    write_mesh(path, coords, tets, 100)
    r = subprocess.run([checker, path], capture_output=True, text=True)
    print(r.stdout.strip())
    assert r.returncode == 0 and r.stdout.startswith("OK"), r.stdout + r.stderr


def test_source_hash_covers_the_layout(monkeypatch):
    """Whichever file defines the layouts' builders, their types or the kernels: a change to it changes the hash."""
    names = ["build_padded_rows(HostProblem &hp) {", "build_halo_tiles(const HostProblem &hp, HaloTiles &ht) {",
             "build_device_rows(const HostProblem &hp, DeviceRows &dr) {",
             "build_device_tiles(const HostProblem &hp, const HaloTiles &ht, DeviceTiles &dt) {", "struct HaloTiles {",
             " k_halo(const HaloArgs<T> a) {", " k_fwd_v(const VFwdArgs<T> a) {", "int xcd_tile(int b, int nb) {",
             "T step_update("]
    files = {f: open(os.path.join(CSRC, f)).read() for f in os.listdir(CSRC)}
    before = bench.kernel_source_sha()
    real_open = open
    for name in names:
        (owner,) = [f for f, text in files.items() if name in text]

        def changed(path, *a, **k):
            import io
            if os.path.basename(str(path)) == owner:
                return io.StringIO(files[owner].replace(name, "int changed; " + name))
            return real_open(path, *a, **k)

        monkeypatch.setattr("builtins.open", changed)
        after = bench.kernel_source_sha()
        monkeypatch.undo()
        assert after != before, (name, owner)
