"""Meshes whose rows go beyond the step kernels' sixteen padded slots."""
import numpy as np
from scipy.spatial import Delaunay


def hub_mesh(n, hollow, seed, ring=60):
    """Delaunay mesh of n random points in the unit ball with two hubs: an interior node alone in a hollow
    of the given radius, and a boundary node on a spike over a ring of `ring` points, so that its row has
    ring + 1 entries of B."""
    rng = np.random.default_rng(seed)
    m = n - 2 - ring
    d = rng.standard_normal((m, 3))
    r = rng.uniform(hollow ** 3, 0.97 ** 3, m) ** (1 / 3)
    a, phi = 0.4, 2 * np.pi * np.arange(ring) / ring
    circle = np.stack([np.sin(a) * np.cos(phi), np.sin(a) * np.sin(phi), np.full(ring, np.cos(a))], 1)
    # the spike's cone touches the unit sphere along the ring
    x = np.vstack([np.zeros((1, 3)), [[0.0, 0.0, 1.0 / np.cos(a)]], circle,
                   d / np.linalg.norm(d, axis=1)[:, None] * r[:, None]])
    t = Delaunay(x).simplices.astype(np.int64)
    vol = np.linalg.det(x[t[:, 1:]] - x[t[:, :1]])
    t[vol < 0] = t[vol < 0][:, [0, 2, 1, 3]]
    t = t[np.abs(vol) > 1e-10]
    assert np.unique(t).size == n
    return x, t.astype(np.int32)
