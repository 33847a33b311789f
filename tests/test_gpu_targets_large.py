"""Proposal targets of more rays than a third of 2^31: ray offsets are 64 bits
wide (26 GB of device memory)."""
import pytest
import torch

from paper_2309_04581_amd import meshrf as M
from paper_2309_04581_amd import scenegen as sg

pytestmark = pytest.mark.gpu


def test_targets_beyond_a_third_of_2_31_rays():
    n, k = 715827883 + 200, 512
    F = M.Field(sg.mid_field(9, 0.5, -1.0))
    T = M.ProposalTrainer(M.Field(sg.make_proposal()), n_bins=1)
    os, ds = (torch.from_numpy(a).cuda() for a in sg.random_rays(k, seed=5))
    want = [t.cpu() for t in T.targets(F, os, ds, 0.05, 4.0, 64)]
    assert (want[0][:, 1] > 0).float().mean() > 0.5
    # rays that miss the box, but for k at either end of the array
    o = torch.full((n, 3), 5.0, device="cuda")
    d = torch.zeros((n, 3), device="cuda")
    d[:, 0] = 1.0
    for s in (slice(0, k), slice(n - k, n)):
        o[s], d[s] = os, ds
    got = T.targets(F, o, d, 0.05, 4.0, 64)
    torch.cuda.synchronize()
    for a, b in zip(got, want):
        assert torch.equal(a[:k].cpu(), b) and torch.equal(a[n - k:].cpu(), b)
        assert all(int(torch.count_nonzero(c)) == 0 for c in a[k:n - k].split(1 << 26))
    del o, d, got
    torch.cuda.empty_cache()
