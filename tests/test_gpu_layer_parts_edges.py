"""GPU: parts of a layer at the sizes where their kernels split the work differently: the gate predictor's contraction over four
wavefronts (fewer than four steps of 128, a number four does not divide) and 32-token workgroups, its data gradient in slices of
256 dims; the compression module's convolution where few offsets are in use; the projections by tiles of 256 x 256.  Oracles and tolerances of
the parts' own tests."""
import pytest

from paper_2505_17412_amd import inputs
from tests import util
from tests import test_gpu_cmp_module_edges, test_gpu_gate

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seed,n,hq,dm", [
    (71, 31, 16, 384), (72, 33, 5, 640), (73, 64, 21, 128),
    (76, 49152, 11, 128), (77, 49153, 16, 128), (78, 60001, 21, 256),   # the last split, a copy of 48 columns, whole contractions of four blocks
    (79, 66000, 16, 128), (80, 129, 5, 128),                            # split: the third round is nearly empty; whole with one block
    (81, 49152, 16, 128), (82, 114689, 8, 128), (83, 62229, 16, 128),   # 48 columns as they are; a copy of 24; of 48, whole contractions
])
def test_gate_splits(seed, n, hq, dm):
    test_gpu_gate.test_gate_forward_backward(seed, n, hq, dm)


# isolated tokens (the offset of the token itself alone), and more of them than one workgroup takes
@pytest.mark.parametrize("seed,n", [(74, (1,) * 70), (75, (2, 1, 3) * 30)])
def test_convolution_with_few_offsets(seed, n):
    test_gpu_cmp_module_edges.test_module_edges(seed, n, 2, 64)


@pytest.mark.parametrize("seed,n,hq,hkv,d,dm", [
    (82, 12400, 16, 2, 64, 1024),   # the data gradient over three contractions; q, k, v would take a second round and stay in tiles of 128
    (83, 32768, 1, 1, 128, 256),    # too short a contraction for them; gates alone (J = 3)
    (84, 12288, 16, 2, 64, 1024),   # three projections, 48 gates beside them
    (85, 12225, 8, 1, 128, 1024),   # 24 gates, the last of their workgroups with one token in its first half and none in its second
    (86, 32768, 1, 1, 128, 768),    # 384 features, the last tile half
])
def test_projections_in_wide_tiles(seed, n, hq, hkv, d, dm):
    """A layer's q, k, v and gates against float32 products of the same bf16 numbers, and its dx against those of what the library's attention
    and output projection return on the saved activations (dx is rounded twice, with the gates' part added behind)."""
    import torch
    from paper_2505_17412_amd import ssa
    wl = inputs.random_points_workload(seed, 64, (n,), hq, hkv, d, (4, 8, 8), 2, "bf16")
    p, blk = util.build_blocks_gpu(wl)
    cq, c = hq * d, hkv * d
    gen = torch.Generator(device="cuda").manual_seed(seed)
    draw = lambda *s, scale=1.0: (scale * torch.randn(s, generator=gen, device="cuda")).bfloat16()
    x, dy = draw(n, dm), draw(n, dm)
    w = {"wq": draw(cq, dm, scale=dm ** -0.5), "wk": draw(c, dm, scale=dm ** -0.5), "wv": draw(c, dm, scale=dm ** -0.5),
         "wg": draw(dm, 3 * hq, scale=dm ** -0.5), "bg": draw(3 * hq), "wo": draw(dm, cq, scale=cq ** -0.5), "bk": draw(c)}
    nbytes, offs = ssa.ssa_layer_saved_bytes(p)
    saved = torch.zeros(nbytes + 256, dtype=torch.uint8, device="cuda")
    y = torch.empty_like(x)
    ssa.ssa_layer_forward(p, blk, x, w, y, saved)
    base = (-saved.data_ptr()) % 256

    def view(name, dtype, *shape):
        nb = torch.Size(shape).numel() * torch.empty((), dtype=dtype).element_size()
        return saved[base + offs[name]: base + offs[name] + nb].view(dtype).view(*shape)

    b16 = torch.bfloat16
    q, k, v, g, o = (view(s, b16, n, *t) for s, t in (("q", (hq, d)), ("k", (hkv, d)), ("v", (hkv, d)), ("gates", (hq, 3)), ("o", (hq, d))))
    ob, lse, idx = view("out_branch", b16, 3, n, hq, d), view("lse", torch.float32, 3, n, hq), view("topk_idx", torch.int32, n, hkv, 2)
    f = {s: t.float() for s, t in w.items()}
    close = lambda got, want, name: util.assert_close(util.to_np(got), util.to_np(want), "bf16", name)
    close(q.reshape(n, cq), x.float() @ f["wq"].T, "q")
    close(k.reshape(n, c), x.float() @ f["wk"].T + f["bk"], "k")
    close(v.reshape(n, c), x.float() @ f["wv"].T, "v")
    close(g.reshape(n, 3 * hq), torch.sigmoid(x.float() @ f["wg"] + f["bg"]), "gates")
    close(y, o.reshape(n, cq).float() @ f["wo"].T, "y")
    grads = {"d" + s: torch.empty(t.shape, dtype=torch.float32, device="cuda") for s, t in w.items()}
    dx = torch.empty_like(x)
    ssa.ssa_layer_backward(p, blk, x, w, saved, dy, dx, grads)
    d_o = torch.empty_like(o)
    ssa.ssa_linear_backward(o.reshape(n, cq).contiguous(), w["wo"], dy, d_o.view(n, cq), torch.empty_like(grads["dwo"]))
    dq, dk, dv, dg = (torch.empty_like(t) for t in (q, k, v, g))
    ssa.ssa_backward(p, blk, q, k, v, g, ob, lse, idx, d_o, dq, dk, dv, dg)
    dz = (dg.float() * g.float() * (1 - g.float())).bfloat16().float().reshape(n, 3 * hq)
    close(d_o.reshape(n, cq), dy.float() @ f["wo"], "dO")
    for s, t in (("dwq", dq), ("dwk", dk), ("dwv", dv)):
        close(grads[s], t.reshape(n, -1).float().T @ x.float(), s)
    close(dx, dq.reshape(n, cq).float() @ f["wq"] + dk.reshape(n, c).float() @ f["wk"] + dv.reshape(n, c).float() @ f["wv"] + dz @ f["wg"].T, "dx")
