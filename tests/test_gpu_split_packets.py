"""Camera packets split over a block's waves against one ray per wave, at the
queue lengths where the split begins and ends (512 resident blocks: 24 576
rays of 8 levels, 12 288 of 16)."""
import numpy as np
import pytest
import torch

from paper_2309_04581_amd import meshrf as M
from paper_2309_04581_amd import scenegen as sg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scene,w,h,n_samples,shadows", [
    ("tiny", 1, 1, 64, False), ("tiny", 5, 3, 3, False), ("tiny", 17, 1, 64, False), ("tiny", 33, 31, 61, False),
    ("tiny", 192, 128, 64, False), ("tiny", 193, 128, 64, False), ("mid", 3, 7, 33, False), ("mid", 65, 63, 96, True),
    ("mid", 128, 96, 96, False), ("mid", 129, 96, 96, False)])
def test_split_packets_match_per_ray(scene, w, h, n_samples, shadows):
    sc = (sg.tiny_scene if scene == "tiny" else sg.mid_scene)(width=w, height=h, table_amp=0.5)
    sc.n_samples, sc.max_bounces = n_samples, 1
    F, G = M.Field(sc.field), M.Mesh(sc.mesh)
    o, d, _ = M.camera_rays(sg.cameras_array(sc.cameras))
    got = []
    for packets in (1, -1):
        opts = M.make_opts(sc, shadow_mask=0.2 if shadows else None)
        opts.march_packets = packets
        R = M.Renderer(len(o), sc.max_bounces).render(F, G, o, d, sc.lights, opts)
        got.append([t.cpu().numpy() for t in (R.radiance, R.throughput, R.bounces, R.hit_ids, R.counters)])
    # one rounding per product or sum and step on either side, in another order
    tol = 4 * n_samples * 2.0 ** -24
    for a, b in zip(got[0][:2], got[1][:2]):
        np.testing.assert_allclose(a, b, rtol=tol, atol=tol * np.abs(b).max())
    for a, b in zip(got[0][2:], got[1][2:]):
        np.testing.assert_array_equal(a, b)
