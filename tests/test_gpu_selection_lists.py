"""GPU: the inverse selection index at the edges of its tiles, seen through forward and backward (the selection branch of
every gradient walks its lists): 256 sorted positions per tile, 16 / 32 / 64 list entries per token, 2048 selection blocks
per workgroup, work chunks of 32 to 256 tokens, 24576 tokens up to which chunks run by block length alone.  Tolerances of the
other parity tests."""
import numpy as np
import pytest

from paper_2505_17412_amd import inputs
from tests.test_gpu_parity import full_parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seed,grid,n,hq,hkv,d,m,topk", [
    (301, 16, (256,), 8, 1, 32, (2, 4, 4), 16),          # one full tile, a full round of entries
    (302, 16, (257,), 8, 1, 32, (2, 4, 4), 17),          # one position in a second tile, a second round
    (303, 32, (255, 0, 700), 16, 2, 64, (2, 4, 8), 33),  # more than two rounds; an empty item
    (304, 32, (600,), 8, 1, 64, (2, 4, 4), 64),          # the longest rows
    (305, 64, (2900,), 16, 1, 32, (1, 2, 8), 8),         # more than 2048 selection blocks
])
def test_lists_at_tile_edges(seed, grid, n, hq, hkv, d, m, topk):
    full_parity(inputs.random_points_workload(seed, grid, n, hq, hkv, d, m, topk, "bf16"))


@pytest.mark.parametrize("seed,lens", [(311, (24576,)), (312, (9000, 15577))])
def test_orders_of_the_work_chunks(seed, lens):
    wl = inputs.make_sequence_workload(seed, lens, hq=4, hkv=2, d=32, l=(32, 96, 64), topk=4)
    full_parity(wl, queries=np.arange(0, wl.n_tokens, 97, dtype=np.int32))
