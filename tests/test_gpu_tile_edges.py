"""GPU: the 32 x 32 tiles of the attention kernels at their edges, on sequences, where the lengths of the blocks can be set: key
ranges of one key to one key past a segment of 256, a last tile of 1, 31 or 32 keys, 2 to 32 tokens in a wavefront's 32 columns with
a remainder, token counts that leave the last workgroup or chunk a single token, every head grouping and head dimension; and each
form of the compression branch.  Tolerances of the other parity tests."""
import numpy as np
import pytest

from paper_2505_17412_amd import inputs
from tests.test_gpu_parity import full_parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seed,lens,hq,hkv,d,l,topk", [
    (901, (130,), 2, 2, 64, (1, 2, 3), 5),               # blocks of two keys; 32 tokens in 32 columns, 2 in the last step
    (902, (33, 1, 64), 4, 2, 32, (4, 32, 31), 2),        # one full tile; items of one token; windows of 31
    (903, (34, 99), 4, 1, 64, (3, 33, 33), 3),           # one key in the second tile
    (904, (200, 63), 8, 1, 128, (7, 63, 64), 2),         # 31 keys in the second tile; 4 tokens per step
    (905, (257,), 16, 1, 64, (8, 64, 65), 4),            # two tokens per step, a step of one; a last block of one key
    (906, (513, 255), 16, 2, 128, (17, 255, 257), 2),    # 31 keys in the eighth tile
    (907, (530,), 2, 1, 128, (16, 256, 256), 3),         # a whole segment, then blocks of 256 and 18
    (908, (771,), 8, 2, 64, (1, 257, 300), 3),           # one key in a second segment
    (909, (300, 129), 1, 1, 32, (2, 130, 96), 2),        # one head
    # windows of 500 tokens and more on average: 128 query rows per workgroup, some of several windows
    (930, (1001, 513, 1600), 4, 4, 64, (8, 64, 700), 2), (931, (1025, 530), 16, 1, 32, (16, 64, 1024), 3),
    (932, (998,), 8, 1, 128, (16, 64, 499), 3), (933, (1000,), 8, 1, 128, (16, 64, 500), 3),  # two windows on either side of the line
])
def test_tile_edges(seed, lens, hq, hkv, d, l, topk):
    full_parity(inputs.make_sequence_workload(seed, lens, hq=hq, hkv=hkv, d=d, l=l, topk=topk))


# Selection blocks of an item where the top-k search takes another form (1024, 2048, 4096), and where the score rows lead to each form of
# the compression branch (csrc/cmp_form.h; tests/test_cmp_form.py holds the last column to that rule).
MANY_BLOCKS = [
    (911, (8192, 40), 16, 2, 64, "tiles_in_lds"), (912, (8193,), 16, 2, 64, "tiles_in_lds"), (913, (40, 16385), 16, 2, 32, "own_tiles_4"),
    (914, (16384,), 8, 1, 64, "own_tiles_4"), (915, (32768,), 16, 1, 32, "own_tiles_4"), (916, (32777,), 16, 1, 32, "own_tiles_4"),
    (917, (6100,), 8, 1, 128, "tiles_in_lds"), (918, (4400, 300), 16, 2, 64, "one_kernel"), (919, (8192,), 16, 1, 32, "one_kernel"),
    (920, (33, 7201), 4, 2, 64, "own_tiles_8"), (921, (3500, 7), 2, 2, 32, "own_tiles_8"), (922, (14401,), 4, 1, 128, "own_tiles_8"),
    (923, (61, 59, 300), 3, 3, 64, "own_tiles_4"), (924, (45, 1, 75), 4, 1, 128, "tiles_in_lds"),
    (925, (999, 45), 8, 2, 64, "one_kernel"),
]


@pytest.mark.parametrize("seed,lens,hq,hkv,d,form", MANY_BLOCKS)
def test_many_selection_blocks(seed, lens, hq, hkv, d, form):
    wl = inputs.make_sequence_workload(seed, lens, hq=hq, hkv=hkv, d=d, l=(4, 8, 16), topk=8)
    full_parity(wl, queries=np.arange(0, wl.n_tokens, 211 if wl.n_tokens > 1000 else 1, dtype=np.int32))
