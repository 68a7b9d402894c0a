"""GPU: parts of a layer at the sizes where their kernels split the work differently: the gate predictor's contraction over four
wavefronts (fewer than four steps of 128, a number four does not divide) and 32-token workgroups, its data gradient in slices of
256 dims; the compression module's convolution where few offsets are in use.  Oracles and tolerances of
the parts' own tests."""
import pytest

from tests import test_gpu_cmp_module_edges, test_gpu_gate

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seed,n,hq,dm", [
    (71, 31, 16, 384), (72, 33, 5, 640), (73, 64, 21, 128),
    (76, 49152, 11, 128), (77, 49153, 16, 128), (78, 60001, 21, 256),   # the last split, whole contractions in two rounds, four column blocks
    (79, 66000, 16, 128), (80, 129, 5, 128),                            # split again: the third round is nearly empty; whole with one block
])
def test_gate_splits(seed, n, hq, dm):
    test_gpu_gate.test_gate_forward_backward(seed, n, hq, dm)


# isolated tokens (the offset of the token itself alone), and more of them than one workgroup takes
@pytest.mark.parametrize("seed,n", [(74, (1,) * 70), (75, (2, 1, 3) * 30)])
def test_convolution_with_few_offsets(seed, n):
    test_gpu_cmp_module_edges.test_module_edges(seed, n, 2, 64)
