"""Closest hits where the tree has one leaf or very many levels, where leaves
are full, where triangles coincide, at ray counts around a block, before and
after a refit."""
import os
import sys

import numpy as np
import pytest
import torch

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
from oracle import oracle as orc  # noqa: E402
from paper_2309_04581_amd import meshrf as M  # noqa: E402
from paper_2309_04581_amd import scenegen as sg  # noqa: E402

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()


@pytest.mark.parametrize("n_tri,n_rays", [(1, 1), (2, 127), (4, 128), (5, 129), (8, 257), (9, 63), (17, 2000)])
def test_closest_hit_of_small_meshes(n_tri, n_rays):
    mesh = sg.random_triangles(n_tri, seed=30 + n_tri)
    o, d = sg.random_rays(n_rays, seed=n_rays)
    G = M.Mesh(mesh)
    for scale in (1.0, 1.5):
        moved = sg.random_triangles(n_tri, seed=30 + n_tri)
        moved.vertices = (mesh.vertices * scale).astype(np.float32)
        if scale != 1.0:
            G.refit(dev(moved.vertices))
        t, tri = (x.cpu().numpy() for x in G.closest_hit(dev(o), dev(d), t_max=10.0))
        for i in range(n_rays):
            hid, want, _, tie = orc.closest_hit(moved, o[i], d[i], t_max=10.0)
            if not tie:
                assert tri[i] == hid and (hid < 0 or abs(t[i] - want) <= 1e-5 * want)


def _stack(z):
    """One wide triangle per height, all over the origin."""
    v = np.array([[[-8, -8, h], [8, -8, h], [0, 8, h]] for h in z], np.float32)
    m = sg.random_triangles(len(z), seed=1)
    m.vertices, m.indices = v.reshape(-1, 3), np.arange(3 * len(z), dtype=np.int32).reshape(-1, 3)
    return m


@pytest.mark.parametrize("z,first", [
    ([64.0 ** -k for k in range(20)], 19),   # every split takes one triangle off: a level each
    ([0.5] * 40, 0), ([0.5] * 3, 0)])        # coincident: the lowest id
def test_closest_hit_of_deep_and_coincident_triangles(z, first):
    G = M.Mesh(_stack(z))
    assert len(set(z)) == 1 or G.info()["depth"] >= 12   # leaves of at most 8
    # heights and origins are powers of two, so the order of the distances is exact
    o = np.zeros((130, 3), np.float32)
    o[:, 0] = np.linspace(-0.5, 0.5, 130)
    o[65:, 2] = 2.0
    d = np.zeros_like(o)
    d[:65, 2], d[65:, 2] = 1.0, -1.0
    for scale in (1.0, 0.5):
        if scale != 1.0:
            G.refit(dev(_stack([scale * h for h in z]).vertices))
        t, tri = (x.cpu().numpy() for x in G.closest_hit(dev(o), dev(d)))
        np.testing.assert_array_equal(tri, [first] * 65 + [0] * 65)
        want = np.array([scale * min(z)] * 65 + [2.0 - scale * max(z)] * 65)
        assert np.all(np.abs(t - want) <= 16 * 2.0 ** -24 * want)   # a quotient of sums of three products
