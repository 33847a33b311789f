"""The kernels that read a field's flat MLP weights (mr_field_params) follow
what a caller writes there: the occupancy grid, and the optical depth of the
light samples toward emitters."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2309_04581_amd import meshrf as M
from paper_2309_04581_amd import scenegen as sg

pytestmark = pytest.mark.gpu


def _fields(layout, offset, **box):
    """Fields of one table: with the first weights, with the second weights,
    and created with the first and given the second by a device copy."""
    make = sg.mid_field if layout == "mid" else sg.tiny_field
    a, b = make(6, 1.0, offset), make(6, 1.0, offset)
    b.mlp = make(7, 1.0, offset).mlp
    for f in (a, b):
        for k, v in box.items():
            setattr(f, k, v)
    A, B, W = M.Field(a), M.Field(b), M.Field(a)
    mlp, n = M.mr_field_params(W.handle)[1::2]
    new = torch.from_numpy(np.ascontiguousarray(b.mlp, np.float32)).cuda()
    assert new.numel() == n
    torch.cuda.synchronize()
    hip = ctypes.CDLL("libamdhip64.so.7")
    assert hip.hipMemcpy(ctypes.c_void_p(mlp), ctypes.c_void_p(new.data_ptr()), ctypes.c_size_t(4 * n), 3) == 0
    return A, B, W


# a group of 64 cells per block, and per wave
@pytest.mark.parametrize("layout,res", [("tiny", 9), ("tiny", 51), ("mid", 9), ("mid", 51)])
def test_occupancy_follows_written_weights(layout, res):
    old, want, got = (F.build_occupancy(res, 0.01, export=True) for F in _fields(layout, -5.0))
    assert torch.equal(got, want)
    assert not torch.equal(old, want)


# 70 000 light samples of 16 levels go one hash level at a time
@pytest.mark.parametrize("layout,n", [("tiny", 500), ("mid", 500), ("mid", 70000)])
def test_light_depth_follows_written_weights(layout, n):
    # rays straight down to a floor; the field lies out of reach of their
    # segments (length 1) but between the floor and the emitter
    pv, pf = sg.floor_plane(-0.6)
    ev, ef, em = sg.emitter_quad()
    mesh = M.Mesh(sg.merge_meshes([(pv, pf, 0), (ev, ef, 1)], [[sg.DIFFUSE, 1.0, 0.7, 0.7, 0.7], em]))
    rng = np.random.default_rng(3)
    o = rng.uniform(-0.4, 0.4, (n, 3)).astype(np.float32)
    o[:, 1] = -0.3
    d = np.tile(np.array([0, -1, 0], np.float32), (n, 1))
    o, d = torch.from_numpy(o).cuda(), torch.from_numpy(d).cuda()
    sc = sg.emitter_scene(8, 8)
    sc.t_near, sc.t_far, sc.n_samples = 0.0, 1.0, 64
    opts = M.make_opts(sc, sample_emitters=True)
    fields = _fields(layout, -1.0, aabb_min=np.float32([-1, 0.5, -1]), aabb_max=np.float32([1, 0.9, 1]))
    old, want, got = (M.Renderer(n, 2).render(F, mesh, o, d, sg.no_lights(), opts).radiance for F in fields)
    assert (want > 0).float().mean() > 0.9
    assert torch.equal(got, want)
    assert not torch.equal(old, want)
