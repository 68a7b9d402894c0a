"""GPU: the selection backward at the edges of its workgroups, on sequences, where the lengths of the selection blocks can be set.
One pass: tiles of 16 keys, 128 keys for four wavefronts, 256 for eight, longer blocks in segments; 4 to 64 tokens per stage;
query lists shorter than a stage.  Two kernels (long blocks in a problem of 2^16 selections or more) on either side of the line
between the forms.  Tolerances of the other parity tests."""
import numpy as np
import pytest

from oracle import compare
from oracle.ssa_oracle import oracle_for
from paper_2505_17412_amd import harness, inputs
from tests.test_gpu_parity import full_parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seed,lens,hq,hkv,d,l,topk", [
    (501, (400, 37), 2, 2, 64, (4, 16, 32), 4),          # one tile of keys; one head, 64 tokens per stage
    (502, (700,), 4, 2, 32, (3, 33, 48), 3),             # three tiles, one key in the third
    (503, (1000, 130), 16, 1, 64, (8, 128, 64), 3),      # four full wavefronts; a block of 2 keys; 4 tokens per stage
    (504, (1032,), 8, 2, 64, (43, 129, 64), 4),          # one key in the ninth tile
    (505, (1300, 513), 8, 1, 32, (16, 256, 64), 2),      # eight full wavefronts, a block of one key
    (506, (1200,), 8, 1, 64, (26, 286, 128), 3),         # 30 keys in a second segment
    (507, (1700,), 4, 1, 32, (40, 800, 64), 2),          # four segments, the last of 32 keys; 16 tokens per stage
    (508, (1025,), 16, 1, 64, (32, 256, 64), 64),        # 65600 selections, no block beyond 256 keys: one pass
    (509, (1028,), 16, 1, 64, (1, 257, 64), 64),         # one key more: two kernels, the last key a segment of its own
    (510, (1025,), 8, 1, 32, (32, 128, 64), 64),         # head_dim 32, no block beyond 128 keys: one pass
    (511, (1032,), 8, 1, 32, (43, 129, 64), 64),         # one key more: two kernels
    (512, (1100, 30), 4, 2, 64, (40, 600, 64), 32),      # two kernels, blocks of 30, 500 and 600 keys
    (513, (1023,), 16, 1, 64, (40, 600, 64), 64),        # 65472 selections: one pass
])
def test_selection_backward_edges(seed, lens, hq, hkv, d, l, topk):
    full_parity(inputs.make_sequence_workload(seed, lens, hq=hq, hkv=hkv, d=d, l=l, topk=topk))


@pytest.mark.parametrize("seed,lens,hq,hkv,d,l,topk", [
    (531, (270, 20), 2, 2, 64, (10, 130, 64), 2),        # blocks of 130, 10 and 20 keys; 128 tokens per stage of the short ones
    (532, (386,), 16, 1, 64, (16, 128, 64), 4),          # the longest block just short enough for four wavefronts
    (533, (387, 3), 16, 1, 64, (3, 129, 64), 4),         # one key more: four tokens per group and stage, a list of three tokens
    (534, (900, 257, 61), 8, 2, 64, (20, 280, 64), 3),   # a second segment of 24 keys; blocks of 60, 61 and 257 in the same launch
    (535, (520, 90), 4, 1, 32, (65, 260, 64), 2),        # the same at head_dim 32
    (536, (212, 5), 8, 1, 32, (12, 144, 64), 2),         # nine tiles of keys beside five
    (537, (194, 193), 16, 2, 64, (1, 193, 64), 2),       # thirteen tiles, the last of one key; blocks of one key
])
def test_blocks_of_many_lengths_in_one_launch(seed, lens, hq, hkv, d, l, topk):
    full_parity(inputs.make_sequence_workload(seed, lens, hq=hq, hkv=hkv, d=d, l=l, topk=topk))


@pytest.mark.parametrize("seed,hq,hkv,d", [
    (541, 640, 40, 128),  # all LDS of a compute unit: the index has launches of its own
    (542, 636, 159, 128),  # 1 KB less: its count pass beside the pre-pass
    (543, 2560, 160, 32),
])
def test_dout_rows_that_fill_the_lds(seed, hq, hkv, d):
    full_parity(inputs.make_sequence_workload(seed, (19, 5), hq=hq, hkv=hkv, d=d, l=(2, 4, 8), topk=2))


@pytest.mark.parametrize("seed,lens,hq,hkv,d,l,topk", [
    (551, (1534, 2), 8, 8, 64, (2, 4, 8), 2),      # 768 blocks of 2 tokens, rows of 512: one wavefront, two passes over the columns
    (552, (3071, 1), 2, 1, 32, (4, 8, 16), 2),     # 769 of 4, one of them of one token, rows of 32: eight groups of threads in one wavefront
    (553, (3200,), 12, 6, 32, (4, 8, 16), 3),      # rows of 192 (48 pieces): a group of threads, the rest idle
    (554, (6144, 6145), 4, 2, 64, (16, 32, 64), 2),  # 769 of 16, rows of 128: two wavefronts
    (555, (3068,), 12, 6, 32, (4, 8, 16), 3),      # 767: four
])
def test_finish_by_one_to_four_wavefronts(seed, lens, hq, hkv, d, l, topk):
    """dK and dV for the sets the forward selected: with one or two heads per KV head and pooled keys of two to four tokens, the rounding of
    these keys moves a score by more than the margin check_topk leaves."""
    wl = inputs.make_sequence_workload(seed, lens, hq=hq, hkv=hkv, d=d, l=l, topk=topk)
    queries = np.arange(0, wl.n_tokens, 61, dtype=np.int32) if wl.n_tokens > 10000 else None
    dout = wl.dout.copy()
    if queries is not None:
        dout[np.setdiff1d(np.arange(wl.n_tokens), queries)] = 0
    g = harness.run_gpu(wl, dout=dout)
    orc = oracle_for(wl)
    ref = orc.forward(wl.q, wl.k, wl.v, wl.gates, topk_idx=g.topk_idx, queries=queries)
    rb = orc.backward(wl.q, wl.k, wl.v, wl.gates, dout, g.topk_idx, out_branch=ref.out_branch, queries=queries)
    compare.assert_close(g.dk, rb.dk, wl.dtype, "dk")
    compare.assert_close(g.dv, rb.dv, wl.dtype, "dv")


def test_one_long_block_among_many_short_ones():
    """Half of the tokens on one voxel, the rest alone in their blocks: the two kernels would launch 5 million workgroups."""
    wl = inputs.random_points_workload(520, 64, (18300,) + (300,) * 60, 16, 2, 64, (1, 2, 2), 2, "bf16")
    rng = np.random.default_rng(520)
    for a, b in zip(wl.batch_offsets[:-1], wl.batch_offsets[1:]):
        first = b - 300
        block = rng.choice(32 ** 3, size=300, replace=False)
        wl.coords[first:b] = 2 * np.stack(np.unravel_index(block, (32, 32, 32)), axis=-1)
        wl.coords[a:first] = wl.coords[first]
    full_parity(wl, queries=np.arange(0, wl.n_tokens, 41, dtype=np.int32))
