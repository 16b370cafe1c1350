"""GPU: moara_state_bytes' first figure is what a state takes from the device."""
import pytest

import workloads as WL
from tests.harness import Case, gpu_state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("operand,decompose,ranks", [("bf16", True, (300, 1001, 200)), ("bf16", False, (300, 1001, 200)),
                                                     ("bf16", False, (100, 251, 200)), ("f32", True, (300, 1001, 200))])
def test_state_bytes_is_what_creating_a_state_allocates(operand, decompose, ranks):
    """Sizes and ranks that need padding, with and without the decomposition, on either side of the
    one-pass kernel's rank range. The state's descriptor arena and the allocator's granularity are
    the slack."""
    import torch
    from paper_2609_15037_amd import moara as M
    c = Case(shapes=[(4001, 8003, WL.Q), (8003, 4001, WL.GATE), (2048, 2048, WL.V)], ranks=list(ranks), block_size=64,
             operand_dtype=operand, decompose=decompose)
    gpu_state(Case(shapes=[(64, 64, WL.Q)], ranks=[8], block_size=64))   # the library's own first allocations
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    st = gpu_state(c)
    taken = before - torch.cuda.mem_get_info()[0]
    want, _ = M.moara_state_bytes(st.cfg, M.make_descs([(m, n, mod, r) for (m, n, mod), r in zip(c.shapes, c.ranks)]))
    assert -(4 << 20) <= taken - want <= 8 << 20, (taken, want)
