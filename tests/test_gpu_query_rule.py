"""Point queries on either side of the sizes from which they go level by level:
the same bits as the same points in small queries, for each pair of table and
MLP types."""
import pytest
import torch

from paper_2309_04581_amd import meshrf as M
from paper_2309_04581_amd import scenegen as sg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("half,bf16,log2_table,layers,n", [
    (False, False, 19, 2, 196607), (False, False, 19, 2, 196608), (True, False, 19, 1, 196608),
    (False, True, 19, 2, 196608), (True, True, 19, 2, 196607), (True, True, 19, 2, 196608), (True, True, 17, 2, 196608),
    (True, True, 17, 2, 262143), (True, True, 17, 2, 262144), (True, True, 19, 1, 262144), (False, False, 14, 2, 262144)])
def test_query_rule(half, bf16, log2_table, layers, n):
    f = sg.make_field(n_levels=16, feats=2, log2_table=log2_table, n_min=16, n_max=1024, d_hidden=64, d_out=16,
                      c_hidden=64, c_layers=layers, sh=16 if layers == 2 else 4, seed=3, table_amp=0.5)
    F = M.Field(f, table_dtype=M.MR_F16 if half else M.MR_F32, mlp_dtype=M.MR_BF16 if bf16 else M.MR_F32)
    g = torch.Generator(device="cuda").manual_seed(n)
    x = torch.rand(n, 3, device="cuda", generator=g) * 2.2 - 1.1
    d = torch.nn.functional.normalize(torch.randn(n, 3, device="cuda", generator=g), dim=1)
    a = F.query(x, d, want_feat=True, want_raw=True)
    parts = [F.query(p, q, want_feat=True, want_raw=True) for p, q in zip(x.split(50000), d.split(50000))]
    for k in a:
        assert torch.equal(a[k], torch.cat([p[k] for p in parts])), k
