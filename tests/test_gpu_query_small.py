"""Point queries a tile of 16 points per wave: the same bits whatever else is in
the call, with and without directions."""
import pytest
import torch

from paper_2309_04581_amd import meshrf as M
from paper_2309_04581_amd import scenegen as sg

pytestmark = pytest.mark.gpu

# one tile of 16 points per wave and four waves per block, up to a second tile
# per wave (4 096 blocks)
@pytest.mark.parametrize("layout,half", [("tiny", False), ("tiny", True), ("mid", False), ("mid", True)])
@pytest.mark.parametrize("n", [1, 15, 17, 63, 65, 1000, 262145])
def test_small_queries_match_single_tiles(layout, half, n):
    f = (sg.mid_field if layout == "mid" else sg.tiny_field)(4, 0.5)
    f.pose = sg.pose_matrix(sg.rotation((0.3, 1.0, 0.2), 0.4), (0.1, -0.05, 0.15))
    F = M.Field(f, **(dict(table_dtype=M.MR_F16, mlp_dtype=M.MR_BF16) if half else {}))
    g = torch.Generator(device="cuda").manual_seed(n)
    x = torch.rand(n, 3, device="cuda", generator=g) * 2.2 - 1.1
    d = torch.nn.functional.normalize(torch.randn(n, 3, device="cuda", generator=g), dim=1)
    a = F.query(x, d, want_feat=True, want_raw=True)
    rows = torch.unique(torch.tensor([0, n // 3, n // 2, n - 1]))
    b = F.query(x[rows].contiguous(), d[rows].contiguous(), want_feat=True, want_raw=True)
    for k in a:
        assert torch.equal(a[k][rows], b[k]), k
    s = F.query(x, None, want_rgb=False)
    assert torch.equal(s["sigma"], a["sigma"])
