"""GPU: the profiling hook counts every part of a forward and a backward pass once (the preparation runs in both), wherever the
backward's selection index stands: beside its pre-pass and dQ kernel, its sums apart or not, or in launches of its own behind each other,
in the order of its chunks by falling length (up to 24576 tokens) or by classes."""
import pytest

from paper_2505_17412_amd import harness, inputs, ssa

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seed,n,hkv,l,topk,apart", [
    (801, 2000, 2, (16, 64, 64), 4, False),     # beside, sums by the last workgroup, by length: nothing apart
    (802, 24570, 2, (32, 64, 64), 3, True),     # beside, 768 lists: the sums apart
    (803, 26000, 1, (256, 512, 512), 2, True),  # beside, 51 lists: the order apart
    (804, 26000, 1, (64, 128, 128), 2, True),   # beside, 204 lists: sums and order apart
    (805, 26000, 4, (64, 128, 128), 2, True),   # 408 workgroups: on its own
    (806, 2000, 2, (16, 64, 64), 17, True),     # more entries a row than stand beside another kernel
])
def test_every_part_is_counted_once(seed, n, hkv, l, topk, apart):
    wl = inputs.make_sequence_workload(seed, (n,), hq=2 * hkv, hkv=hkv, d=32, l=l, topk=topk)
    harness.run_gpu(wl, backward=True)
    ssa.ssa_profile_enable(True)
    harness.run_gpu(wl, backward=True)
    counts = {name: launches for name, (ms, launches) in ssa.ssa_profile_get().items()}
    ssa.ssa_profile_enable(False)
    assert counts.pop("prep_sort_pool") == 2
    assert counts.pop("bwd_invert_selection", 0) == apart
    assert set(counts.values()) == {1}, counts
