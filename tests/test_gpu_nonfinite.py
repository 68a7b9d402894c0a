"""GPU: infinities and NaN in one batch item on the fp32-arithmetic path, and on the matrix path finite keys whose scores overflow.
The tiles hold query columns, keys and query rows of neighbouring items, so such a value must not reach a row through a weight of
zero.  The other items are compared with the oracle or a run on the untouched inputs, at the tolerances of the other parity tests."""
import copy

import numpy as np
import pytest

from oracle.ssa_oracle import oracle_for
from paper_2505_17412_amd import inputs
from tests import util

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), float("-inf")])
@pytest.mark.parametrize("seed,grid,n,hq,hkv,d,dtype", [
    (801, 16, (70, 65, 90), 4, 2, 32, "f32"),
    (802, 8, (21, 5, 33), 6, 2, 40, "f32"),    # 5 tokens per tile; an item inside one tile
    (803, 16, (45, 40, 51), 20, 1, 24, "bf16"),
    (804, 8, (17, 18, 19), 2, 2, 128, "f32"),
])
def test_other_items_keep_their_values(seed, grid, n, hq, hkv, d, dtype, bad):
    wl = inputs.random_points_workload(seed, grid, n, hq, hkv, d, (2, 4, 4), 3, dtype)
    orc = oracle_for(wl)
    clean = util.run_gpu(wl)
    ref = orc.forward(wl.q, wl.k, wl.v, wl.gates, topk_idx=clean.topk_idx)
    grad = orc.backward(wl.q, wl.k, wl.v, wl.gates, wl.dout, clean.topk_idx, out_branch=ref.out_branch)
    want = {"out": ref.out, "dq": grad.dq, "dk": grad.dk, "dv": grad.dv, "dgates": grad.dgates}
    others = np.r_[0:n[0], n[0] + n[1]:sum(n)]
    for what in ("q", "k", "v", "dout"):
        hit = copy.deepcopy(wl)
        getattr(hit, what)[n[0] + n[1] // 2, :, d // 3] = bad
        got = util.run_gpu(hit)
        assert not np.isfinite(getattr(got, "dk" if what == "dout" else "out")[n[0]:n[0] + n[1]]).all(), what
        assert np.array_equal(got.topk_idx[others], clean.topk_idx[others]), what
        for name, w in want.items():
            util.assert_close(getattr(got, name)[others], w[others], dtype, f"{what}: {name}")


def test_value_reaches_the_rows_that_attend_to_it():
    """A value row of infinities shows in exactly the output rows whose window or selected blocks (or item, pooled) hold it."""
    wl = inputs.random_points_workload(805, 16, (200,), 4, 2, 32, (2, 4, 4), 3, "f32")
    orc = oracle_for(wl)
    clean = util.run_gpu(wl, backward=False)
    wl.v[50, :, 7] = np.inf
    got = util.run_gpu(wl, backward=False)
    ref = orc.forward(wl.q, wl.k, wl.v, wl.gates, topk_idx=clean.topk_idx)
    for b in (1, 2):
        fine = np.isfinite(ref.out_branch[b])
        assert 0 < (~fine).sum() < fine[..., 7].size
        assert np.array_equal(np.isfinite(got.out_branch[b]), fine), b
        util.assert_close(got.out_branch[b][fine], ref.out_branch[b][fine], "f32", f"branch {b}")


@pytest.mark.parametrize("d", [24, 32, 72])
def test_keys_at_minus_infinity_have_no_weight(d):
    """Keys whose score is minus infinity for every query take no part, at head dimensions padded in the registers too."""
    wl = inputs.random_points_workload(806, 16, (150, 60), 4, 2, d, (2, 8, 16), 5, "f32")
    wl.q[..., 0] = np.abs(wl.q[..., 0]) + 0.5
    wl.k[30:60, :, 0] = -np.inf
    orc = oracle_for(wl)
    got = util.run_gpu(wl, backward=False)
    own = orc.forward(wl.q, wl.k, wl.v, wl.gates, want_scores=True)
    util.check_topk(got.topk_idx, own, orc, "f32")
    ref = orc.forward(wl.q, wl.k, wl.v, wl.gates, topk_idx=got.topk_idx)
    assert np.isfinite(ref.out).all()
    util.assert_close(got.out, ref.out, "f32", "out")


@pytest.mark.parametrize("seed,grid,n,hq,hkv,d", [
    (811, 16, (300, 270, 333), 16, 2, 64), (812, 16, (300, 270, 333), 8, 1, 32), (813, 16, (300, 270, 333), 16, 2, 128),
    (814, 16, (33, 21, 40), 4, 4, 64), (815, 16, (45, 9, 70), 2, 1, 64),
])
@pytest.mark.parametrize("far", [3e38, -3e38])
def test_scores_of_other_items_that_overflow_on_the_matrix_path(seed, grid, n, hq, hkv, d, far):
    """Finite keys of one item whose products with any query leave the range of the floats: tiles at the ends of the neighbouring
    items' key ranges hold them, and nothing of it reaches those items.  (To the tolerance of the type, not to the bit: columns of one
    wavefront raise their reference exponents together, and probabilities are rounded relative to the reference.)"""
    wl = inputs.random_points_workload(seed, grid, n, hq, hkv, d, (1, 4, 8), 4, "bf16")  # one-voxel blocks: the means stay finite
    clean = util.run_gpu(wl)
    others = np.r_[0:n[0], n[0] + n[1]:sum(n)]
    mine = slice(n[0], n[0] + n[1])
    wl.k[mine] = inputs.round_to_bf16(np.float32(far) * np.sign(wl.k[mine]))
    got = util.run_gpu(wl)
    assert np.array_equal(got.topk_idx[others], clean.topk_idx[others])
    for name in ("out", "dq", "dk", "dv", "dgates"):
        util.assert_close(getattr(got, name)[others], getattr(clean, name)[others], "bf16", name)
    util.assert_close(got.lse[:, others], clean.lse[:, others], "bf16", "lse")


@pytest.mark.parametrize("seed,lens,hq,hkv,d,l", [
    (821, (512, 200), 16, 2, 64, (1, 128, 128)), (822, (512, 200), 4, 4, 32, (1, 128, 128)),
    (823, (512, 200), 8, 1, 128, (1, 128, 128)), (824, (900, 200), 16, 2, 64, (1, 300, 300)),
])
def test_first_keys_at_the_lowest_value_have_no_weight_on_the_matrix_path(seed, lens, hq, hkv, d, l):
    """The first 40 keys carry the type's lowest value where every query is above one: their scores are minus infinity, no later
    tile may be measured against them, and the other keys keep their weights."""
    wl = inputs.make_sequence_workload(seed, lens, hq=hq, hkv=hkv, d=d, l=l, topk=2)
    wl.q[..., 0] = inputs.round_to_bf16(np.abs(wl.q[..., 0]) + 2.0)
    wl.k[0:40, :, 0] = -3.38e38
    wl.k = inputs.round_to_bf16(wl.k)
    assert np.isfinite(wl.k).all()
    orc = oracle_for(wl)
    got = util.run_gpu(wl, backward=False)
    ref = orc.forward(wl.q, wl.k, wl.v, wl.gates, topk_idx=got.topk_idx)
    assert np.isfinite(ref.out).all()
    for b in range(3):
        util.assert_close(got.out_branch[b], ref.out_branch[b], "bf16", f"branch {b}")
    util.assert_close(got.out, ref.out, "bf16", "out")
