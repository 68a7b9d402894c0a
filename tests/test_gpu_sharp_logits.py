"""GPU: scores far outside the range of ordinary attention, so that a later key tile of a block exceeds its first tile by more
than the exponents can hold against a fixed reference, and the kernels must fall back to a running maximum.  Tolerances of the
other parity tests."""
import numpy as np
import pytest

from paper_2505_17412_amd import inputs
from tests import util
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


LONG = [
    (511, (1144, 300), 16, 2, 64, 286, 4),   # second segment of 30 keys: no full tile
    (512, (1144, 300), 8, 1, 32, 286, 4),
    (513, (1144, 300), 16, 2, 128, 286, 4),
    (514, (1700,), 8, 2, 64, 800, 3),        # four segments, the last of 32 keys
    (515, (1700,), 4, 2, 32, 800, 3),
    (516, (1700,), 16, 1, 128, 800, 3),
]


def long_blocks(seed, lens, hq, hkv, d, m_slc, topk):
    wl = inputs.make_sequence_workload(seed, lens, hq=hq, hkv=hkv, d=d, l=(1, m_slc, 70), topk=topk)
    place = np.concatenate([np.arange(n) for n in lens]) % m_slc
    wl.k = inputs.round_to_bf16(wl.k * np.array([0.02, 0.5, 0.1, 1.0])[np.minimum(place // 256, 3)][:, None, None])
    wl.q = inputs.round_to_bf16(wl.q * 60.0)
    return wl


@pytest.mark.parametrize("seed,lens,hq,hkv,d,m_slc,topk", LONG)
def test_later_segments_of_a_long_block_exceed_the_first(seed, lens, hq, hkv, d, m_slc, topk):
    """Blocks longer than the 256 keys held at a time: the partial result of the earlier segments is picked up again, and a later
    segment's scores exceed its reference.  Every block is selected, one-token compression blocks keep their keys exact."""
    wl = long_blocks(seed, lens, hq, hkv, d, m_slc, topk)
    # log2 units by which a block's largest score exceeds the largest of its first tile, over the first block's columns
    s = np.einsum("nhd,mhd->hnm", wl.q[:64, ::hq // hkv], wl.k[:m_slc]) / np.sqrt(d) * np.log2(np.e)
    excess = s.max(axis=-1) - s[..., :32].max(axis=-1)
    assert (excess > 60.0).mean() > 0.5  # their sums leave the range (2^60) and the running maximum has to take over
    full_parity(wl, backward=False)


@pytest.mark.parametrize("seed,lens,hq,hkv,d,m_slc,topk", LONG + [
    (517, (1701,), 16, 1, 64, 800, 3),       # chunks that end in a step of one token
    (518, (2501, 903), 2, 2, 64, 800, 4),    # 32 tokens per step
])
def test_long_blocks_are_deterministic(seed, lens, hq, hkv, d, m_slc, topk):
    """Columns past the end of a chunk share one row of partial results, which any workgroup may have written last: it decides
    nothing, and runs agree bit for bit."""
    wl = long_blocks(seed, lens, hq, hkv, d, m_slc, topk)
    blocks = util.build_blocks_gpu(wl)
    first = util.run_gpu(wl, blocks=blocks)
    for _ in range(3):
        again = util.run_gpu(wl, blocks=blocks)
        for name in ("out", "out_branch", "lse", "topk_idx", "dq", "dk", "dv", "dgates"):
            assert np.array_equal(getattr(again, name), getattr(first, name)), name
