"""GPU: matrices whose bf16 operands are padded to whole 32-wide panels (sizes, ranks and caller
addresses that are no multiple of anything, and no decomposition), against the oracle."""
import pytest

import workloads as WL
from tests.harness import Case
from tests.test_gpu_history import _grad, history_parity
from tests.test_gpu_parity import step_parity

pytestmark = pytest.mark.gpu

# one past and one short of a panel, a 128- and a 256-wide tile on either side; n odd; ranks 1, 4,
# 33, r = s; a LEFT row of more blocks (B = 4) than the transposed decomposition holds at once
SHAPES = [(33, 1001, WL.Q), (1001, 33, WL.GATE), (255, 257, WL.V), (257, 255, WL.UP), (127, 129, WL.K),
          (31, 703, WL.DOWN), (641, 130, WL.O)]
RANKS = [33, 4, 130, 127, 1, 31, 66]


@pytest.mark.parametrize("B,wdt,mom", [(64, "bf16", "bf16"), (128, "bf16", "f32"), (32, "f32", "bf16"),
                                       (4, "f32", "f32")])
def test_padded_operands_from_a_restored_state(B, wdt, mom):
    c = Case(shapes=SHAPES, ranks=RANKS, block_size=B, operand_dtype="bf16", weight_dtype=wdt, moment_dtype=mom,
             weight_std=1e-2 if wdt == "bf16" else 1e-5)
    history_parity(c, 3, 130 + B, _grad(c, 130 + B))


@pytest.mark.parametrize("misalign", [False, True])
@pytest.mark.parametrize("decompose", [False, True])
def test_padded_operands_and_unaligned_buffers(decompose, misalign):
    c = Case(shapes=SHAPES, ranks=RANKS, block_size=64, operand_dtype="bf16", weight_dtype="bf16", weight_std=0.02,
             decompose=decompose)
    step_parity(c, 2, misalign=misalign)
