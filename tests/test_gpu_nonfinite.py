"""GPU: infinities and NaN in one batch item on the fp32-arithmetic path.  Its tiles hold query columns, keys and query rows of
neighbouring items, so a value that is not finite must not reach a row through a weight of zero.  The other items are compared
with the oracle on the untouched inputs, at the tolerances of the other parity tests."""
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
