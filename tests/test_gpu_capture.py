"""GPU: block handles are built and destroyed while a stream captures a graph.  In a relaxed capture, and beside a capture of another
thread, allocations and frees are allowed, so neither call may invalidate the graph."""
import threading

import numpy as np
import pytest

from oracle import blocks as oblocks
from paper_2505_17412_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode,other_thread", [("relaxed", False), ("relaxed", True), ("thread_local", True)])
def test_build_and_destroy_beside_a_capture(mode, other_thread):
    import torch
    from paper_2505_17412_amd import ssa
    from tests import util
    wl = inputs.random_points_workload(901, 16, (300, 217), 4, 2, 32, (2, 4, 8), 4, "f32")
    want = oblocks.build_blocks(wl.coords, wl.batch_offsets, wl.grid, wl.m_cmp, wl.m_slc, wl.m_win).perm
    p, first = util.build_blocks_gpu(wl)
    coords, offs = torch.from_numpy(wl.coords.reshape(-1, 3)).cuda(), torch.from_numpy(wl.batch_offsets).cuda()
    side, x = torch.cuda.Stream(), torch.arange(64, dtype=torch.float32, device="cuda")
    torch.cuda.synchronize()
    made = []

    def work():
        with torch.cuda.stream(side):
            first.destroy()
            made.append(ssa.ssa_build_blocks(p, coords, offs))

    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, capture_error_mode=mode):
        y = x * 2
        if other_thread:
            t = threading.Thread(target=work)
            t.start()
            t.join()
        else:
            work()
        z = y + 1
    for k in range(3):
        x.fill_(k)
        graph.replay()
        torch.cuda.synchronize()
        assert (z == 2 * k + 1).all()
    assert np.array_equal(util.to_np(made[0].export("perm")), want)
