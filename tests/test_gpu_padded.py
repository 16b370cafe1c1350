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


def test_moments_beyond_two_gib_on_the_large_tile_path():
    """A tall matrix whose fp32 moments pass 2^31 bytes (its bf16 operands do not): one step's first
    moment and weights on rows from its start, middle and end against the oracle (a RIGHT matrix's
    rows are independent given P)."""
    import dataclasses
    import numpy as np
    import torch
    from oracle import moara_oracle as O
    from paper_2609_15037_amd import moara as M
    from tests.harness import TOL_BF16, compare, gpu_state, oracle_cfg, rng, to_np
    m, n, r = 530000, 1024, 1024
    c = Case(shapes=[(m, n, WL.UP)], ranks=[r], block_size=64, operand_dtype="bf16", weight_dtype="bf16")
    rows = torch.cat([torch.arange(400), torch.arange(m // 2, m // 2 + 300), torch.arange(m - 400, m)])
    gen = torch.Generator(device="cuda").manual_seed(3)
    G = torch.randn(m, n, device="cuda", generator=gen) * 1e-3
    W = (torch.randn(m, n, device="cuda", generator=gen) * 0.02).bfloat16()
    P = O.round_f32(np.linalg.qr(rng(8, 1).standard_normal((n, r)))[0])
    st = gpu_state(c)
    M.moara_set_tensor(st, 0, M.MOARA_T_P, P)
    Gs, Ws = to_np(G[rows.cuda()]), to_np(W[rows.cuda()])
    M.moara_step(st, [W], [G], lr=c.lr)
    torch.cuda.synchronize()
    ocfg = oracle_cfg(dataclasses.replace(c, shapes=[(len(rows), n, WL.UP)]), 0)
    ost = O.init_state(len(rows), n, ocfg)
    assert ost.side == O.RIGHT
    ost.P = P
    Wo = O.step(Ws, Gs, ost, ocfg, c.lr)
    report = {}
    compare("exp_avg", M.moara_get_tensor(st, 0, M.MOARA_T_EXP_AVG)[rows.numpy()], ost.exp_avg, TOL_BF16, report)
    compare("W", to_np(W[rows.cuda()]), Wo, TOL_BF16, report)


# the one-pass decomposition and projection: tiles of 64 (RIGHT) and 128 (LEFT) rows, K chunks of
# 128 and 64 and panels of 32, one past and one short of each; ranks at the edges of its 32-column
# blocks and of its range; unaligned rows (n % 4 != 0) beside aligned ones
FUSED = [(32, 128, WL.Q), (129, 32, WL.GATE), (96, 257, WL.K), (127, 128, WL.V), (260, 132, WL.UP), (191, 97, WL.O),
         (256, 1000, WL.DOWN), (640, 256, WL.GATE), (130, 384, WL.Q)]
FUSED_RANKS = [1, 31, 33, 64, 100, 97, 256, 255, 129]


# fewer rows or columns than a panel: the one-pass kernel down to four columns, below that (and at
# other block sizes) the 128-row kernels
THIN = [(16, 4096, WL.Q), (4096, 16, WL.GATE), (5, 700, WL.K), (700, 5, WL.UP), (3, 64, WL.V), (64, 3, WL.O),
        (1, 300, WL.DOWN), (300, 1, WL.GATE), (4, 4, WL.Q), (31, 129, WL.K), (65, 31, WL.UP)]
THIN_RANKS = [16, 9, 5, 3, 2, 3, 1, 1, 4, 31, 30]


@pytest.mark.parametrize("B,wdt,mom", [(32, "bf16", "bf16"), (64, "f32", "f32"), (128, "bf16", "f32"),
                                       (16, "f32", "bf16"), (256, "bf16", "f32")])
def test_thin_matrices_from_a_restored_state(B, wdt, mom):
    # bf16 moments are held to 99 % equal bits; sums of four products or fewer have so few bits that
    # 0.9 e + 0.1 R meets midpoints of bf16 exactly, which the library's fp32 beta1 breaks otherwise
    # than the oracle's fp64 one (3 x 64: 2 of 128 moments within 6e-15 of a midpoint)
    keep = [i for i, (m, n, _) in enumerate(THIN) if mom == "f32" or min(m, n) > 4]
    c = Case(shapes=[THIN[i] for i in keep], ranks=[THIN_RANKS[i] for i in keep], block_size=B, operand_dtype="bf16",
             weight_dtype=wdt, moment_dtype=mom, weight_std=1e-2 if wdt == "bf16" else 1e-5)
    history_parity(c, 2, 430 + B, _grad(c, 430 + B))


@pytest.mark.parametrize("misalign", [False, True])
def test_thin_matrices_without_the_decomposition(misalign):
    c = Case(shapes=THIN, ranks=THIN_RANKS, block_size=64, operand_dtype="bf16", weight_dtype="bf16", weight_std=0.02,
             decompose=False)
    step_parity(c, 2, misalign=misalign)


@pytest.mark.parametrize("B,wdt,mom", [(32, "bf16", "bf16"), (64, "f32", "f32"), (128, "bf16", "f32"),
                                       (128, "f32", "bf16")])
def test_one_pass_projection_from_a_restored_state(B, wdt, mom):
    c = Case(shapes=FUSED, ranks=FUSED_RANKS, block_size=B, operand_dtype="bf16", weight_dtype=wdt, moment_dtype=mom,
             weight_std=1e-2 if wdt == "bf16" else 1e-5)
    history_parity(c, 2, 230 + B, _grad(c, 230 + B))


@pytest.mark.parametrize("misalign", [False, True])
@pytest.mark.parametrize("mom", ["f32", "bf16"])
def test_one_pass_projection_without_the_decomposition(mom, misalign):
    c = Case(shapes=FUSED, ranks=FUSED_RANKS, block_size=1, operand_dtype="bf16", weight_dtype="bf16", weight_std=0.02,
             decompose=False, moment_dtype=mom)
    step_parity(c, 2, misalign=misalign)


# decomp_eps = 0, and one so small that 1 / eps overflows fp32: the padding rows of a LEFT matrix's
# last K panel are zero gradients, whose scale 1 / (0 + eps) is then infinite. m % 32 != 0, with
# m % 8 zero and not (the transposed decomposition stores groups of 8 rows)
LEFT_ROWS = [(33, 200, WL.Q), (129, 257, WL.V), (1000, 1032, WL.DOWN), (257, 33, WL.GATE)]
LEFT_RANKS = [20, 100, 250, 33]


@pytest.mark.parametrize("eps", [0.0, 1e-40])
@pytest.mark.parametrize("two_pass", [False, True])
def test_padding_stays_zero_when_the_decomposition_epsilon_is_zero(two_pass, eps):
    """Finite dense gradients give the oracle's finite results on either route (a rank above 256
    sends a short list through the two-pass kernels)."""
    c = Case(shapes=LEFT_ROWS + ([(300, 320, WL.K)] if two_pass else []), ranks=LEFT_RANKS + ([257] if two_pass else []),
             block_size=64, operand_dtype="bf16", weight_dtype="bf16", weight_std=1e-2, decomp_eps=eps)
    history_parity(c, 2, 330, _grad(c, 330))


@pytest.mark.parametrize("block,thin", [(64, False), (256, False), (64, True)])
def test_one_pass_and_two_pass_projection_are_bit_identical(block, thin):
    """A matrix whose rank exceeds the one-pass kernel's range sends a short list of matrices through
    the two-pass kernels, and its update through 256-column tiles: the same matrices give the same
    bits with and without it beside them. Blocks of 256 columns take the two-pass kernels either
    way, so there only the update's tiles differ."""
    import numpy as np
    import torch
    from paper_2609_15037_amd import moara as M
    from tests.harness import gpu_state, rng, to_dev
    shapes, ranks = (THIN, THIN_RANKS) if thin else (FUSED, FUSED_RANKS)
    big, rbig = (300, 320, WL.V), 257
    out = []
    for extra in (False, True):
        c = Case(shapes=shapes + ([big] if extra else []), ranks=ranks + ([rbig] if extra else []), block_size=block,
                 operand_dtype="bf16", weight_dtype="bf16", weight_std=0.02, moment_dtype="bf16")
        st = gpu_state(c)
        W, G = [], []
        for i, ((m, n, _), r) in enumerate(zip(c.shapes, c.ranks)):
            W.append(to_dev(0.02 * rng(5, 1, i).standard_normal((m, n)), "bf16"))
            G.append(to_dev(rng(5, 2, i).standard_normal((m, n)), "f32"))
            P = np.linalg.qr(rng(5, 3, i).standard_normal((min(m, n), r)))[0]
            M.moara_set_tensor(st, i, M.MOARA_T_P, P)
        for _ in range(3):
            M.moara_step(st, W, G, lr=1e-2)
        torch.cuda.synchronize()
        out.append([(W[i], *[M.moara_get_tensor(st, i, k) for k in
                             (M.MOARA_T_EXP_AVG, M.MOARA_T_EXP_AVG_SQ, M.MOARA_T_MAG_AVG, M.MOARA_T_MAG_AVG_SQ)])
                    for i in range(len(shapes))])
    for i, (a, b) in enumerate(zip(*out)):
        assert torch.equal(a[0], b[0]), f"matrix {i}: W differs"
        for x, y in zip(a[1:], b[1:]):
            assert np.array_equal(x, y), f"matrix {i}: a moment differs"


@pytest.mark.parametrize("two_pass", [False, True])
def test_refresh_in_the_step_without_the_decomposition(two_pass):
    """decompose = 0: a step whose refresh is due gives the bits of an explicit refresh and a step,
    with the projection in the one-pass kernel (a state that has no V) and in the two-pass ones."""
    import torch
    from paper_2609_15037_amd import moara as M
    from tests.harness import assert_same_state, explicit_refresh, gpu_state, rng, to_dev
    extra = [(300, 320, WL.V)] if two_pass else []
    c = Case(shapes=FUSED + extra, ranks=FUSED_RANKS + [257] * len(extra), block_size=64, operand_dtype="bf16",
             weight_dtype="bf16", decompose=False, refresh_iters=6)
    n = len(c.shapes)
    A, B = gpu_state(c, refresh_interval=2), gpu_state(c)
    WA, WB = [[to_dev(0.02 * rng(9, 1, i).standard_normal(s[:2]), "bf16") for i, s in enumerate(c.shapes)] for _ in "AB"]
    for t in range(3):
        G = [to_dev(rng(9, 2, t, i).standard_normal(s[:2]), "f32") for i, s in enumerate(c.shapes)]
        explicit_refresh(M, B, G, [t % 2 == 0] * n)
        M.moara_step(A, WA, G, lr=1e-2)
        M.moara_step(B, WB, G, lr=1e-2)
        torch.cuda.synchronize()
        assert_same_state(M, A, B, WA, WB, range(n), f"step {t}:")


@pytest.mark.parametrize("case", ["fused", "two_pass", "fp32_operands", "no_decompose", "refresh_due", "refresh_due_no_decompose",
                                  "misaligned", "fused-f32-32", "fused-f32-64", "fused-f32-128", "fused-bf16-32",
                                  "fused-bf16-128", "many"])
def test_bf16_gradients_step_as_their_fp32_copies(case):
    """moara_step_mixed on bf16 gradients gives the bits of moara_step on the converted ones, on every
    route: read by the one-pass kernel (n % 4 == 0 and 8-byte aligned; every moment type and block
    size), or converted first (other widths and alignments, larger ranks, fp32 operands, a due
    refresh; "many": more buffers than one conversion launch holds); inactive matrices stay."""
    import numpy as np
    import torch
    from paper_2609_15037_amd import moara as M
    from tests.harness import gpu_state, rng, to_dev
    shapes, ranks = list(FUSED), list(FUSED_RANKS)
    if case == "two_pass":
        shapes, ranks = shapes + [(300, 320, WL.V)], ranks + [257]
    if case == "many":   # 150 buffers, 64 to a launch; counts that are and are not multiples of 8
        shapes = [(33 + i % 7, 41 + i % 5, WL.Q) for i in range(188)]
        ranks = [8] * len(shapes)
    operand = "f32" if case in ("fp32_operands", "many") else "bf16"
    mom, block = case.split("-")[1:] if case.startswith("fused-") else ("bf16" if operand == "bf16" else "f32", 64)
    c = Case(shapes=shapes, ranks=ranks, block_size=int(block), operand_dtype=operand, weight_dtype="bf16",
             weight_std=0.02, moment_dtype=mom, decompose="no_decompose" not in case)
    active = [i != 3 for i in range(len(shapes))]
    out = []
    for mixed in (False, True):
        st = gpu_state(c, refresh_interval=2 if "refresh_due" in case else 0)
        W, G, B32 = [], [], []
        for i, ((m, n, _), r) in enumerate(zip(c.shapes, c.ranks)):
            W.append(to_dev(0.02 * rng(6, 1, i).standard_normal((m, n)), "bf16"))
            g = to_dev(rng(6, 2, i).standard_normal((m, n)), "bf16")
            if case == "misaligned":
                buf = torch.zeros(m * n + 1 + i % 4, dtype=torch.bfloat16, device="cuda")
                buf[1 + i % 4:] = g.flatten()
                g = buf[1 + i % 4:].view(m, n)
            # one in five is fp32 already
            G.append(g if mixed and i % 5 else g.float())
            B32.append(torch.full((m, n), float("nan"), device="cuda") if mixed and i % 5 else None)
            P = np.linalg.qr(rng(6, 3, i).standard_normal((min(m, n), r)))[0]
            M.moara_set_tensor(st, i, M.MOARA_T_P, P)
        for _ in range(3):
            if mixed:
                M.moara_step_mixed(st, W, G, B32, lr=1e-2, active=active)
            else:
                M.moara_step(st, W, G, lr=1e-2, active=active)
        torch.cuda.synchronize()
        out.append([(W[i], *[M.moara_get_tensor(st, i, k) for k in
                             (M.MOARA_T_P, M.MOARA_T_EXP_AVG, M.MOARA_T_EXP_AVG_SQ, M.MOARA_T_MAG_AVG,
                              M.MOARA_T_MAG_AVG_SQ)]) for i in range(len(shapes))])
        if mixed:
            with pytest.raises(ValueError):   # no buffer for the bf16 gradients
                M.moara_step_mixed(st, W, G, [None] * len(W), lr=1e-2)
    for i, (a, b) in enumerate(zip(*out)):
        assert torch.equal(a[0], b[0]), f"matrix {i}: W differs"
        for x, y in zip(a[1:], b[1:]):
            assert np.array_equal(x, y), f"matrix {i}: a moment or the projector differs"


@pytest.mark.parametrize("block,decompose", [(16, True), (64, True), (256, True), (64, False)])
def test_transposed_decomposition_split_by_columns_gives_the_same_bits(block, decompose):
    """A LEFT matrix's two-pass step alone, its decomposition split over column parts, and in a list
    of enough row groups to run without the split; rows of more blocks than the kernel holds at once
    (B = 16), widths that leave the last part short or empty."""
    import numpy as np
    import torch
    from paper_2609_15037_amd import moara as M
    from tests.harness import assert_same_state, gpu_state, rng, to_dev
    few = [(300, 5001, WL.Q), (259, 4096, WL.K), (257, 2305, WL.V), (289, 1025, WL.O)]
    shapes = few + [(320, 640, WL.DOWN)] * 76   # ten row groups of 32 each
    c = Case(shapes=shapes, ranks=[257] * len(shapes), block_size=block, operand_dtype="bf16", weight_dtype="bf16",
             moment_dtype="bf16", decompose=decompose)
    out = []
    for alone in (False, True):
        st = gpu_state(c)
        W = [to_dev(0.02 * rng(10, 1, i % 5).standard_normal(s[:2]), "bf16") for i, s in enumerate(shapes)]
        G = [to_dev(rng(10, 2, i % 5).standard_normal(s[:2]), "f32") for i, s in enumerate(shapes)]
        for i, (m, n, _) in enumerate(shapes):
            M.moara_set_tensor(st, i, M.MOARA_T_P, np.eye(m, 257, dtype=np.float32) + 0.01)
        for one in (range(len(few)) if alone else [None]):
            M.moara_step(st, W, G, lr=1e-2, active=None if one is None else [j == one for j in range(len(shapes))])
        torch.cuda.synchronize()
        out.append((st, W))
    (sa, Wa), (sb, Wb) = out
    assert_same_state(M, sa, sb, Wa, Wb, range(len(few)))


def test_fp32_tiles_of_either_size_give_the_same_bits():
    """fp32 operands: lists of more than 4096 tiles of 128 x 128 run on those, shorter ones on 64 x 64
    tiles. Matrices stepped all at once (both projections and the update past the line) and one by one."""
    import numpy as np
    import torch
    from paper_2609_15037_amd import moara as M
    from tests.harness import assert_same_state, gpu_state, rng, to_dev
    k = 66
    shapes, ranks = [(1000, 1024, WL.Q)] * k + [(1152, 1024, WL.GATE)] * k, [1000] * k + [1024] * k
    c = Case(shapes=shapes, ranks=ranks, block_size=64, weight_std=0.02)
    assert min(8 * 8, 9 * 8) * k > 4096
    gen = torch.Generator(device="cuda").manual_seed(5)
    G = [torch.randn(m, n, device="cuda", generator=gen) for m, n, _ in shapes]
    out = []
    for each in (False, True):
        st = gpu_state(c)
        gw = torch.Generator(device="cuda").manual_seed(6)
        W = [0.02 * torch.randn(m, n, device="cuda", generator=gw) for m, n, _ in shapes]
        for i in range(2 * k):   # any fixed P will do
            P = np.zeros((min(shapes[i][:2]), ranks[i]), dtype=np.float32)
            P[np.arange(ranks[i]), np.arange(ranks[i])[::-1]] = 0.75
            P[0] += 0.01
            M.moara_set_tensor(st, i, M.MOARA_T_P, P)
        for one in (range(2 * k) if each else [None]):
            M.moara_step(st, W, G, lr=1e-2, active=None if one is None else [j == one for j in range(2 * k)])
        torch.cuda.synchronize()
        out.append((st, W))
    (sa, Wa), (sb, Wb) = out
    assert_same_state(M, sa, sb, Wa, Wb, [0, 1, k - 1, k, 2 * k - 1])
    assert all(torch.equal(a, b) for a, b in zip(Wa, Wb))
