"""GPU: the fp32-arithmetic kernels at the edges of their 16 x 16 tiles: head groupings that do not fill 16 columns or exceed
them, head dimensions that are no multiple of 16, an item of one token, ragged items, long selection rows, more than 256 pooled keys per
item (chunks of the score kernel), score rows that leave the kernel fewer tokens per workgroup."""
import numpy as np
import pytest

from paper_2505_17412_amd import inputs
from tests.test_gpu_parity import full_parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seed,grid,n,hq,hkv,d,m,topk,dtype", [
    (401, 16, (333, 1, 90), 6, 2, 40, (2, 4, 4), 3, "f32"),      # 3 heads per KV head: 5 tokens per tile, one unused column
    (402, 16, (130,), 20, 1, 96, (2, 4, 8), 5, "bf16"),          # 20 heads: two tiles per token
    (403, 8, (70,), 64, 1, 128, (2, 4, 4), 4, "f32"),            # 64 heads of 128
    # a partly filled tile, and an item of one token (a problem of one token alone has dQ = dK = 0 exactly: its softmaxes are
    # constant, and a relative error of rounding noise against zero has no bound)
    (404, 8, (1, 6), 2, 1, 8, (2, 4, 4), 2, "f32"),
    (405, 32, (1500, 800), 4, 4, 32, (2, 4, 8), 64, "f32"),      # one head per KV head, the longest rows, > 256 pooled keys
    (406, 64, (2600,), 2, 2, 16, (1, 2, 4), 4, "f32"),           # 2500 selection blocks: 5 tokens' scores do not fit
])
def test_generic_tile_edges(seed, grid, n, hq, hkv, d, m, topk, dtype):
    full_parity(inputs.random_points_workload(seed, grid, n, hq, hkv, d, m, topk, dtype))


def test_score_row_that_leaves_the_kernel_one_token_at_a_time():
    """15000 selection blocks in one item: a token's scores take most of the LDS, one token per workgroup."""
    wl = inputs.make_sequence_workload(408, (30000,), 2, 1, 8, (1, 2, 4), 4, "f32")
    full_parity(wl, queries=np.arange(5, 30000, 997, dtype=np.int32))


def test_one_long_block_among_many_short_ones():
    """Half of the tokens on one voxel, the rest alone in their blocks: (longest block's tiles) x (selection chunks) is more
    workgroups than one launch of the key-centric kernel can have."""
    wl = inputs.random_points_workload(407, 64, (18000,), 2, 2, 8, (1, 2, 2), 2, "f32")
    rng = np.random.default_rng(407)
    block = rng.choice(32 ** 3, size=9000, replace=False)
    wl.coords[:9000] = 2 * np.stack(np.unravel_index(block, (32, 32, 32)), axis=-1)
    wl.coords[9000:] = wl.coords[0]
    full_parity(wl, queries=np.arange(0, 18000, 41))
