"""GPU: the one-pass selection backward at the edges of its workgroups, on sequences, where the lengths of the selection
blocks can be set: tiles of 16 keys, 128 keys for four wavefronts, 256 for eight, longer blocks in segments; 4 to 64 tokens
per stage; query lists shorter than a stage.  Tolerances of the other parity tests."""
import pytest

from paper_2505_17412_amd import inputs
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
])
def test_selection_backward_edges(seed, lens, hq, hkv, d, l, topk):
    full_parity(inputs.make_sequence_workload(seed, lens, hq=hq, hkv=hkv, d=d, l=l, topk=topk))
