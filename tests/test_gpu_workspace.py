"""Graph capture and the launch-shape search take the workspaces that
mr_render takes: the ray queues alone are enough."""
import pytest
import torch

from paper_2309_04581_amd import meshrf as M
from paper_2309_04581_amd import scenegen as sg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w,h", [(64, 48), (300, 230)])   # the larger has scratch beyond its queues
def test_queues_alone_are_a_workspace(w, h):
    sc = sg.mid_scene(width=w, height=h, n_samples=32)
    sc.max_bounces = 2
    F, G = M.Field(sc.field), M.Mesh(sc.mesh)
    o, d, _ = M.camera_rays(sg.cameras_array(sc.cameras))
    n, opts = w * h, M.make_opts(sc)
    R = M.Renderer(n, sc.max_bounces)
    queues = 4096 + 128 * ((n + 63) // 64 * 64)
    assert queues <= R.ws_bytes
    args = (F.handle, G.handle, n, o, d, sc.max_bounces, None, sc.lights, opts, R.out, R.workspace)
    M.mr_render(*args, queues)
    want = R.radiance.clone()
    g = M.mr_render_graph_create(*args, queues)
    for _ in range(3):
        R.radiance.fill_(-1.0)
        M.mr_graph_launch(g)
        torch.cuda.synchronize()
        assert torch.equal(R.radiance, want)
    M.mr_graph_destroy(g)
    R.radiance.fill_(-1.0)
    shape = M.mr_autotune_search(*args, queues)[0]
    if shape[5] == 0:   # packets on the same segments: the same bits
        assert torch.equal(R.radiance, want)
    for call in (M.mr_render, M.mr_render_graph_create, M.mr_autotune_search):
        with pytest.raises(M.MrError) as e:
            call(*args, queues - 1)
        assert e.value.status == M.MR_ERR_INVALID_ARG
