"""GPU: scores far outside the range of ordinary attention, so that a later key tile of a block exceeds its first tile by more
than the exponents can hold against a fixed reference, and the kernels must fall back to a running maximum.  Tolerances of the
other parity tests."""
import numpy as np
import pytest

from paper_2505_17412_amd import inputs
from tests.test_gpu_parity import full_parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seed,hq,hkv,d,factor", [(501, 16, 2, 64, 60.0), (502, 8, 1, 32, 60.0), (503, 16, 2, 128, 60.0)])
def test_scores_of_hundreds(seed, hq, hkv, d, factor):
    # one-voxel compression blocks (their keys stay exact: a rounded mean would move such scores by 1) and every block selected
    wl = inputs.random_points_workload(seed, 16, (1500,), hq, hkv, d, (1, 8, 8), 8, "bf16")
    wl.q = inputs.round_to_bf16(wl.q * factor)
    s = np.einsum("nhd,mhd->hnm", wl.q[:64, ::hq // hkv], wl.k) / np.sqrt(d)
    assert np.ptp(s, axis=-1).min() > 200.0  # natural units: the largest exceeds any first tile by far for most rows
    full_parity(wl, backward=False)
