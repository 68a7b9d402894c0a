"""GPU: the inverse selection index at the edges of its tiles, seen through forward and backward (the selection branch of
every gradient walks its lists): 256 sorted positions per tile, 16 / 32 / 64 list entries per token, 2048 selection blocks
per workgroup, work chunks of 32 to 256 tokens, 24576 tokens up to which chunks run by block length alone, more KV heads than the order of
the chunks has buckets for at its usual fineness.  Tolerances of the other parity tests."""
import numpy as np
import pytest

from paper_2505_17412_amd import inputs
from tests import util
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


@pytest.mark.parametrize("seed,lens,hq,hkv,d,l,topk", [
    (331, (1020, 4), 2, 2, 32, (1, 2, 16), 16),          # 512 blocks: one part of blocks per workgroup, full rounds of entries
    (332, (1022, 4), 2, 2, 64, (1, 2, 16), 16),          # 513 blocks: a second part of one
    (333, (1023,), 4, 2, 128, (1, 2, 16), 5),            # two kernels' lists; a tile of 255 positions
    (334, (24576,), 4, 4, 32, (16, 32, 64), 2),          # 768 blocks, two parts: 768 workgroups, launches of its own
    (335, (24570,), 2, 2, 32, (32, 64, 64), 3),          # 384 blocks: 192 workgroups, sums by one kernel of their own
])
def test_lists_built_beside_the_backward_kernels(seed, lens, hq, hkv, d, l, topk):
    """The backward's index (csrc/sel_device.h: 512 blocks and 16 entries a row, 384 workgroups in all)."""
    wl = inputs.make_sequence_workload(seed, lens, hq=hq, hkv=hkv, d=d, l=l, topk=topk)
    full_parity(wl, queries=np.arange(0, wl.n_tokens, 97 if wl.n_tokens > 10000 else 1, dtype=np.int32))


@pytest.mark.parametrize("seed,lens,hq,hkv,d,l,topk", [
    (341, (1024,), 8, 1, 32, (1, 2, 16), 16),            # 512 lists, a thread each, in full tiles
    (342, (1026,), 8, 1, 32, (1, 2, 16), 16),            # 513: apart
    (343, (500, 0, 13, 258), 32, 2, 32, (4, 8, 32), 8),  # items of few blocks, an empty one, workgroups over several; two heads
    (344, (255,), 16, 2, 64, (2, 4, 16), 64),            # the longest rows, padded
    (345, (8192,), 8, 1, 64, (8, 16, 64), 17),          # 16384 counts
    (346, (8193,), 8, 1, 128, (8, 16, 64), 1),          # more: apart
])
def test_lists_counted_by_the_compression_kernel(seed, lens, hq, hkv, d, l, topk):
    """The forward's index (csrc/sel_index.hip: 512 lists and 16384 counts of 256 positions)."""
    wl = inputs.make_sequence_workload(seed, lens, hq=hq, hkv=hkv, d=d, l=l, topk=topk)
    full_parity(wl, queries=np.arange(0, wl.n_tokens, 97 if wl.n_tokens > 3000 else 1, dtype=np.int32))


@pytest.mark.parametrize("seed,lens", [(311, (24576,)), (312, (9000, 15577))])
def test_orders_of_the_work_chunks(seed, lens):
    wl = inputs.make_sequence_workload(seed, lens, hq=4, hkv=2, d=32, l=(32, 96, 64), topk=4)
    full_parity(wl, queries=np.arange(0, wl.n_tokens, 97, dtype=np.int32))


@pytest.mark.parametrize("topk", [3, 4, 8, 9])
def test_merge_of_rows_with_few_blocks(topk):
    """Rows of I with fewer blocks than top-k (items of 1 to 12): what the workspace held before, here NaNs, is in no result (the merge requests
    the partials of 4 to 8 blocks before it knows how many there are)."""
    import torch
    from paper_2505_17412_amd import ssa
    wl = inputs.make_sequence_workload(351, (5, 17, 90, 33, 1), hq=8, hkv=1, d=32, l=(4, 8, 16), topk=topk)
    p, blk = util.build_blocks_gpu(wl)
    q, k, v, g = (util.to_dev(t, "bf16") for t in (wl.q, wl.k, wl.v, wl.gates))
    n = wl.n_tokens

    def run(fill):
        out, branch = torch.empty_like(q), torch.empty((3, *q.shape), dtype=q.dtype, device="cuda")
        lse, idx = torch.empty((3, n, 8), device="cuda"), torch.empty((n, 1, topk), dtype=torch.int32, device="cuda")
        ws = torch.full((ssa.ssa_workspace_bytes(p, blk, False),), fill, dtype=torch.uint8, device="cuda")
        ssa.ssa_forward(p, blk, q, k, v, g, out, lse, idx, branch, workspace=ws)
        torch.cuda.synchronize()
        return out, lse, idx, branch

    a, b = run(0), run(255)
    assert (b[2] == -1).any() and torch.isfinite(b[0].float()).all()
    for x, y in zip(a, b):
        assert torch.equal(x, y)


@pytest.mark.parametrize("heads", [1025])
def test_more_kv_heads_than_buckets(heads):
    """Heads are independent: with more of them than 8192 buckets in eight classes of block length leave one each, the first, a middle
    and the last head come out as in a call of these three."""
    import torch
    from paper_2505_17412_amd import ssa
    n, d, topk, some = 24577, 32, 1, [0, heads // 2, heads - 1]
    offs = torch.tensor([0, n], dtype=torch.int32, device="cuda")
    gen = torch.Generator(device="cuda").manual_seed(321)
    x = {k: torch.randn((n, heads, d), generator=gen, device="cuda", dtype=torch.bfloat16) for k in ("q", "k", "v", "dout")}
    gates = torch.rand((n, heads, 3), generator=gen, device="cuda").to(torch.bfloat16)

    def run(hs):
        q, k, v, do, g = (t if hs is None else t[:, hs].contiguous() for t in (*x.values(), gates))
        h = q.shape[1]
        p = ssa.make_params(n, 1, 0, 512, 1024, 128, topk, h, h, d, "bf16")
        blk = ssa.ssa_build_blocks_1d(p, offs)
        out, dq, dk, dv, dg = (torch.full_like(t, float("nan")) for t in (q, q, k, v, g))
        branch = torch.empty((3, n, h, d), dtype=torch.bfloat16, device="cuda")
        lse, idx = torch.empty((3, n, h), device="cuda"), torch.empty((n, h, topk), dtype=torch.int32, device="cuda")
        ssa.ssa_forward(p, blk, q, k, v, g, out, lse, idx, branch)
        ssa.ssa_backward(p, blk, q, k, v, g, branch, lse, idx, do, dq, dk, dv, dg)
        torch.cuda.synchronize()
        return [t if hs is not None else t[:, some] for t in (idx, out, dq, dk, dv, dg)]

    few, many = run(some), run(None)
    assert torch.equal(few[0], many[0])
    for name, a, b in zip(("out", "dq", "dk", "dv", "dgates"), many[1:], few[1:]):
        util.assert_close(util.to_np(a), util.to_np(b), "bf16", name)
