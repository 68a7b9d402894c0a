"""GPU: the partition's sort at the edges of its tiles and digits, and memory kept from one handle to the next; compared bit
for bit with the oracle's block structure."""
import numpy as np
import pytest

from oracle.blocks import build_blocks_1d
from paper_2505_17412_amd import inputs
from tests import util
from tests.test_gpu_blocks import build_blocks, check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seed,grid,n,m,dup", [
    (61, 2, (8,), (1, 2, 2), False),                              # 3 key bits: one pass of the smallest digit
    (62, 64, (16384,), (4, 8, 8), False), (63, 64, (16385,), (4, 8, 8), False),   # one and two keys per thread
    (64, 128, (140000, 130000), (4, 8, 8), False),                # 16 keys per thread, several tiles
    (65, 512, (40000, 0, 9), (4, 8, 16), True),                   # three passes, duplicates
    # 2^20 tokens: the last size whose tiles every workgroup sums; then prefixes, of 2048 digits, of 8, of 16 tiles and more per segment
    (66, 128, (1048576,), (4, 8, 8), True), (67, 128, (1048577,), (4, 8, 8), True),
    (68, 2, (1100000,), (1, 2, 2), True), (69, 1024, (1500000, 0, 640001), (4, 8, 16), True),
])
def test_sort_tile_and_digit_edges(seed, grid, n, m, dup):
    check(inputs.random_points_workload(seed, grid, n, 2, 1, 8, m, 2, allow_duplicates=dup))


def test_long_sequences():
    """More tiles of tokens than the block arrays' workgroups sum up themselves."""
    wl = inputs.make_sequence_workload(60, (1000003, 48575, 17), hq=1, hkv=1, d=8, l=(3, 33, 70), topk=2, with_tensors=False)
    ref = build_blocks_1d(wl.batch_offsets, wl.m_cmp, wl.m_slc, wl.m_win)
    _, blk = util.build_blocks_gpu(wl)
    assert blk.counts() == (ref.n_blocks["cmp"], ref.n_blocks["slc"], ref.n_blocks["win"])
    for name, want in (("perm", ref.perm), ("cmp_start", ref.start["cmp"]), ("slc_start", ref.start["slc"]), ("win_start", ref.start["win"]),
                       ("slc_child_start", ref.slc_child_start), ("tok_win", ref.tok_win)):
        assert np.array_equal(blk.export(name).cpu().numpy(), want), name


def test_kept_memory_is_safe_across_handles():
    """Handles built and destroyed in turn (the memory of a destroyed one serves the next) hold their own arrays."""
    wls = [inputs.random_points_workload(70 + i, 32, (500 + 37 * i, 200), 2, 1, 8, (2, 4, 8), 2) for i in range(6)]
    alive = []
    for rep in range(3):
        for wl in wls:
            check(wl)
        alive = [util.build_blocks_gpu(wl)[1] for wl in wls[:3]]
    for wl, blk in zip(wls[:3], alive):
        ref = build_blocks(wl.coords, wl.batch_offsets, wl.grid, wl.m_cmp, wl.m_slc, wl.m_win)
        assert np.array_equal(blk.export("perm").cpu().numpy(), ref.perm)


def test_destroyed_handle_is_refused():
    """A destroyed handle reports no counts and exports nothing, whatever was asked of it before."""
    wl = inputs.random_points_workload(77, 16, (300,), 2, 1, 32, (4, 8, 8), 2, "f32")
    _, blk = util.build_blocks_gpu(wl)
    assert blk.counts()[0] > 0
    blk.export("perm")
    blk.destroy()
    with pytest.raises(Exception):
        blk.counts()
    with pytest.raises(Exception):
        blk.export("perm")
