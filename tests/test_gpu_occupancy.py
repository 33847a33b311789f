"""The occupancy grid against the FP64 oracle at the sizes where its kernel
changes shape: one cell, ragged groups of 64, a group per block and a group
per wave."""
import numpy as np
import pytest
import torch

from oracle import oracle as orc
from paper_2309_04581_amd import meshrf as M
from paper_2309_04581_amd import scenegen as sg

pytestmark = pytest.mark.gpu


# 50^3 cells are fewer groups of 64 than the device has waves, 51^3 are not
@pytest.mark.parametrize("layout,res,thresh,offset", [
    ("tiny", 1, 0.3, 0.0), ("tiny", 3, 0.3, 0.0), ("tiny", 9, 0.01, -5.0), ("tiny", 50, 0.01, -5.0),
    ("tiny", 51, 0.01, -5.0), ("tiny", 16, 0.0, -5.0), ("tiny", 16, -1.0, -5.0), ("tiny", 16, 1e9, -5.0),
    ("mid", 5, 0.01, -5.0), ("mid", 24, 0.01, -5.0), ("mid", 41, 0.01, -5.0)])
def test_occupancy_matches_oracle(layout, res, thresh, offset):
    f = (sg.mid_field if layout == "mid" else sg.tiny_field)(6, 1.0, offset)
    bits = M.Field(f).build_occupancy(res, thresh, export=True).cpu().numpy()
    ref, margin = orc.occupancy(f, res, thresh)
    certain = np.abs(margin) > 1e-5
    np.testing.assert_array_equal(bits[certain], ref[certain])
    assert certain.mean() > 0.98
    if res > 20 and thresh == 0.01:
        assert 0.02 < ref.mean() < 0.98
