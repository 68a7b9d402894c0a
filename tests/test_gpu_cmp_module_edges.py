"""GPU: the learned compression module at the sizes where its kernels change shape: one tile of tokens less or more, the
1024-token segments of the weight gradient, the line between 64 and 128 tokens per convolution workgroup (16384), and the parts
that a tile's offsets are dealt out to (one tensor: three up to 170 tiles of 64 tokens, one up to 16384 tokens, then of 128 three up to 170
tiles, two up to 256).
Against the fp64 oracle, tolerances as in test_gpu_cmp_module.py."""
import numpy as np
import pytest

from paper_2505_17412_amd import inputs
from tests import util
from tests.test_gpu_cmp_module import draw_weights, gpu_module, module_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seed,n,hkv,d", [
    (61, (63,), 2, 64), (62, (65,), 2, 64), (63, (1024,), 2, 64), (64, (1, 1024), 2, 64), (65, (1100, 950), 1, 32),
    (66, (16384,), 2, 64), (67, (9000, 7401), 2, 64),
    (68, (1,), 2, 64), (69, (1, 1, 1), 2, 64), (70, (170 * 64,), 2, 64), (71, (170 * 64 + 1,), 2, 64), (72, (170 * 128 + 1,), 2, 64),
])
def test_module_edges(seed, n, hkv, d):
    m = (4, 8, 8)
    wl = inputs.random_points_workload(seed, 32, n, 2 * hkv, hkv, d, m, 2, "bf16")
    orc, mod = module_oracle(wl)
    c = hkv * d
    pe, w, bias = draw_weights(seed, m[0], c)
    x = wl.k.reshape(wl.n_tokens, c)
    rng = np.random.default_rng(seed + 7)
    dxc = rng.standard_normal((orc.blocks.n_blocks["cmp"], c)).astype(np.float32)
    dx0 = inputs.round_to_bf16(rng.standard_normal((wl.n_tokens, c)).astype(np.float32))
    p, blk = util.build_blocks_gpu(wl)
    got = gpu_module(wl, p, blk, wl.k, pe, w, bias, dxc, dx0.reshape(wl.k.shape))
    f, g = mod.forward(x, pe, w, bias), mod.backward(x, pe, w, bias, dxc)
    util.assert_close(got["x_cmp"].reshape(-1, c), f.x_cmp, "bf16", "x_cmp")
    util.assert_close(got["dx"].reshape(-1, c), dx0 + g.dx, "bf16", "dx")
    for name in ("dpe", "dw", "dbias"):
        util.assert_close(got[name], getattr(g, name), "bf16", name)
