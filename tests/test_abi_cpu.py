"""C ABI checks that need no GPU: the library loads, exports every declared
symbol, and its host logic (Phase 3 rank rule, rank/side resolution, argument
validation, state sizing) is exact."""
import ctypes
import os
import re

import numpy as np
import pytest

from oracle import moara_oracle as O
from tests.conftest import ROOT, golden

M = pytest.importorskip("paper_2609_15037_amd.moara")


def _lib():
    if not os.path.exists(M.LIB_PATH):
        pytest.skip("libmoara.so not built")
    return M.lib()


def test_every_declared_symbol_is_exported():
    L = _lib()
    header = open(os.path.join(ROOT, "include", "moara.h")).read()
    names = set(re.findall(r"^\s*(?:int|void|const char\*)\s+(moara_\w+)\s*\(", header, re.M))
    assert names, "no declarations parsed"
    for n in sorted(names):
        assert hasattr(L, n), f"{n} declared but not exported"
    assert set(M.EXPORTED) == names


def test_allocate_ranks_matches_oracle_and_paper_row():
    _lib()
    gd = golden("rank_allocations.json")
    assert M.moara_allocate_ranks(256, range(7), [0, 1], [6], 128)[:7] == gd["ours_r256"]
    for rb, D, R, dr in [(512, [0, 1], [6], 256), (1024, [0, 1], [6], 512), (256, [0], [5, 6], 64),
                         (200, [2, 3], [4], 50), (128, [], [], 0), (64, [7], [8, 9], 32)]:
        types = list(range(10)) if max(D + R + [0]) > 6 else list(range(7))
        got = M.moara_allocate_ranks(rb, types, D, R, dr)
        ref = O.allocate_ranks(rb, types, D, R, dr)
        assert [got[t] for t in types] == [ref[t] for t in types]
        assert sum(got) == rb * len(types)
        assert all(got[t] == 0 for t in range(10) if t not in types)


@pytest.mark.parametrize("args", [
    (256, range(7), [0, 1, 2], [5, 6], 1),     # non-integer receiver share
    (100, range(7), [0, 1], [6], 100),          # donors fall to 0
])
def test_allocate_ranks_rank_errors(args):
    _lib()
    with pytest.raises(M.MoaraError) as e:
        M.moara_allocate_ranks(*args)
    assert e.value.status == M.MOARA_E_RANK
    with pytest.raises(ValueError):
        O.allocate_ranks(*args)


@pytest.mark.parametrize("args", [
    (256, range(7), [0, 1], [1], 8),            # overlap
    (256, range(7), [0, 1], [], 8),             # receivers missing
    (0, range(7), [0], [6], 0),                 # r_base < 1
    (256, range(3), [0], [6], 8),               # receiver outside types
    (256, [], [], [], 0),                       # empty types
])
def test_allocate_ranks_argument_errors(args):
    _lib()
    with pytest.raises(M.MoaraError) as e:
        M.moara_allocate_ranks(*args)
    assert e.value.status == M.MOARA_E_ARG


def test_resolve_matrix_side_and_rank_bit_exact():
    _lib()
    cfg = M.moara_default_config(rank_table=[512, 512, 1024, 1024, 768, 768, 768, 128, 128, 128])
    cases = [((4096, 4096, 0), 512, M.MOARA_SIDE_LEFT), ((11008, 4096, 4), 768, M.MOARA_SIDE_RIGHT),
             ((4096, 11008, 6), 768, M.MOARA_SIDE_LEFT), ((512, 3584, 1), 512, M.MOARA_SIDE_LEFT),
             ((1408, 2048, 7), 128, M.MOARA_SIDE_LEFT), ((2048, 1408, 9), 128, M.MOARA_SIDE_RIGHT),
             ((300, 200, 2, 17), 17, M.MOARA_SIDE_RIGHT), ((300, 200, 2, 17, M.MOARA_SIDE_LEFT), 17, M.MOARA_SIDE_LEFT)]
    for t, r, side in cases:
        d = M.make_descs([t])[0]
        assert M.moara_resolve_matrix(cfg, d) == (r, side)
        want = O.projection_side(t[0], t[1])
        if len(t) < 5:
            assert (side == M.MOARA_SIDE_LEFT) == (want == O.LEFT)


def test_resolve_matrix_errors():
    _lib()
    cfg = M.moara_default_config(rank_table=[8] * 10)
    for t, code in [((0, 5, 0), M.MOARA_E_SHAPE), ((4, 4, 11), M.MOARA_E_ARG), ((4, 4, 0), M.MOARA_E_RANK),
                    ((8, 8, 0, 9), M.MOARA_E_RANK), ((8, 8, 0, 0, 3), M.MOARA_E_ARG)]:
        with pytest.raises(M.MoaraError) as e:
            M.moara_resolve_matrix(cfg, M.make_descs([t])[0])
        assert e.value.status == code


@pytest.mark.parametrize("field,value,code", [
    ("block_size", 0, -1), ("beta1", 1.0, -1), ("beta2", -0.1, -1), ("adam_eps", 0.0, -1),
    ("weight_decay", 0.01, -4), ("grad_dtype", 1, -4), ("operand_dtype", 7, -1), ("refresh_iters", 0, -1),
    ("refresh_interval", -1, -1), ("zero_grad_mode", 2, -1), ("decompose", 2, -1), ("moment_dtype", 3, -1),
])
def test_create_state_validates_before_touching_the_gpu(field, value, code):
    _lib()
    cfg = M.moara_default_config(rank_table=[8] * 10, **{field: value})
    descs = M.make_descs([(64, 64, 0)])
    with pytest.raises(M.MoaraError) as e:
        M.moara_create_state(cfg, descs)
    assert e.value.status == code
    with pytest.raises(M.MoaraError) as e:
        M.moara_state_bytes(cfg, descs)
    assert e.value.status == code


def test_refresh_workspace_follows_the_chunk_budget(monkeypatch):
    """The refresh workspace is the whole batch's need unless the chunk budget
    (MOARA_REFRESH_CHUNK_MIB) is smaller; then it is that budget plus one matrix's share."""
    _lib()
    cfg = M.moara_default_config(rank_table=[64] * 10, block_size=64, operand_dtype=M.MOARA_BF16)
    descs = M.make_descs([(1024, 1024, 0)] * 4)
    monkeypatch.delenv("MOARA_REFRESH_CHUNK_MIB", raising=False)
    _, whole = M.moara_state_bytes(cfg, descs)
    monkeypatch.setenv("MOARA_REFRESH_CHUNK_MIB", "1")
    _, small = M.moara_state_bytes(cfg, descs)
    assert small == (1 << 20) + whole // 4 < whole
    for bad in ("0", "-3", "12x", ""):   # ignored: the default budget applies
        monkeypatch.setenv("MOARA_REFRESH_CHUNK_MIB", bad)
        assert M.moara_state_bytes(cfg, descs)[1] == whole


def test_default_chunk_budget_is_128_gib(monkeypatch):
    """A Llama-2-7B-shaped stack (224 matrices, ranks 512 / 1024 / 2048, p = r) needs more
    refresh workspace than one chunk holds: the default bound is 128 GiB."""
    _lib()
    ranks = M.moara_allocate_ranks(1024, range(7), [M.MOARA_Q, M.MOARA_K], [M.MOARA_DOWN], 512)
    cfg = M.moara_default_config(rank_table=ranks, block_size=128)
    d, f = 4096, 11008
    descs = M.make_descs([((d, d), 0), ((d, d), 1), ((d, d), 2), ((d, d), 3),
                          ((f, d), 4), ((f, d), 5), ((d, f), 6)] * 32)
    monkeypatch.setenv("MOARA_REFRESH_CHUNK_MIB", str(1 << 30))   # 1 PiB: no bound
    _, whole = M.moara_state_bytes(cfg, descs)
    monkeypatch.delenv("MOARA_REFRESH_CHUNK_MIB")
    _, capped = M.moara_state_bytes(cfg, descs)
    assert whole > (128 << 30)
    assert capped == (128 << 30) + whole // 224


def test_state_bytes_counts_fp32_moments_projector_copies_and_v_workspace():
    _lib()
    cfg = M.moara_default_config(rank_table=[64] * 10, block_size=64, operand_dtype=M.MOARA_BF16)
    shapes = [(256, 688), (688, 256), (250, 688)]
    descs = M.make_descs([(m, n, 4) for m, n in shapes])
    sb, rb = M.moara_state_bytes(cfg, descs)
    al = lambda x: (x + 255) // 256 * 256
    up = lambda x: -(-x // 32) * 32
    exp = 0
    for m, n in shapes:
        s, L, k, r = min(m, n), max(m, n), -(-n // 64), 64
        # the bf16 operands (N, the two projector copies, the direction workspace V of the
        # large-tile projection) are padded to 32 along their reduction length
        exp += 4 * al(4 * m * k) + 2 * al(4 * L * r) + al(2 * L * r) + al(4 * s * r) + al(2 * s * r) + al(2 * up(s) * r)
        exp += al(2 * L * up(s))
    exp += al(16 * len(shapes))   # one refresh record (four int32) per matrix
    assert sb == exp and rb > 0
    # fp32 operands never materialise V
    cfg32 = M.moara_default_config(rank_table=[64] * 10, block_size=64, operand_dtype=M.MOARA_F32)
    sb32, _ = M.moara_state_bytes(cfg32, descs)
    exp32 = 0
    for m, n in shapes:
        s, L, k, r = min(m, n), max(m, n), -(-n // 64), 64
        exp32 += 4 * al(4 * m * k) + 2 * al(4 * L * r) + al(4 * L * r) + al(4 * s * r) + 2 * al(4 * s * r)
    exp32 += al(16 * len(shapes))
    assert sb32 == exp32
    # bf16 direction moments (2-byte states) halve exp_avg / exp_avg_sq and nothing else
    cfgm = M.moara_default_config(rank_table=[64] * 10, block_size=64, operand_dtype=M.MOARA_BF16,
                                  moment_dtype=M.MOARA_BF16)
    sbm, rbm = M.moara_state_bytes(cfgm, descs)
    assert rbm == rb
    assert sbm == sb - sum(2 * al(4 * max(m, n) * 64) - 2 * al(2 * max(m, n) * 64) for m, n in shapes)


def test_no_v_workspace_without_the_decomposition_at_ranks_up_to_256():
    """decompose = 0 and every matrix in the one-pass kernel's range: nothing ever writes V."""
    _lib()
    al = lambda x: (x + 255) // 256 * 256
    for ranks, v in (((64, 256), False), ((64, 288), True)):
        cfg = M.moara_default_config(block_size=64, operand_dtype=M.MOARA_BF16, decompose=0)
        shapes = [(1024, 2048), (640, 512)]
        sb, _ = M.moara_state_bytes(cfg, M.make_descs([(m, n, 4, r) for (m, n), r in zip(shapes, ranks)]))
        exp = al(16 * 2)
        for (m, n), r in zip(shapes, ranks):
            s, L = min(m, n), max(m, n)
            exp += 4 * al(4 * m * (n // 64)) + 2 * al(4 * L * r) + al(2 * L * r) + al(4 * s * r) + 2 * al(2 * s * r)
            exp += al(2 * m * n) if v else 0
        assert sb == exp, (ranks, sb, exp)


def test_v_workspace_reaches_to_the_operands_own_extents():
    """V is kept up to 2^31 bytes per bf16 operand, whatever the moments' bytes (here 4 L r > 2^31)."""
    _lib()
    m, n, r = 530000, 1024, 1024
    cfg = M.moara_default_config(block_size=64, operand_dtype=M.MOARA_BF16)
    sb, _ = M.moara_state_bytes(cfg, M.make_descs([(m, n, M.MOARA_UP, r)]))
    al = lambda x: (x + 255) // 256 * 256
    assert 4 * m * r > 2 ** 31 > 2 * m * n
    assert sb == (4 * al(4 * m * (n // 64)) + 2 * al(4 * m * r) + al(2 * m * r) + al(4 * n * r) + 2 * al(2 * n * r) +
                  al(2 * m * n) + al(16))


def test_default_config_keeps_fp32_direction_moments():
    _lib()
    assert M.moara_default_config().moment_dtype == M.MOARA_F32


def test_alignment_rejects_bad_arguments_before_any_gpu_work():
    L = _lib()
    import ctypes
    out = (ctypes.c_double * 2)()
    assert L.moara_alignment(None, None, None, out, None) == M.MOARA_E_ARG
    assert b"state is NULL" in L.moara_last_error()


def test_nd_shapes_flatten_into_descriptors():
    assert M.flatten_shape((64, 8, 3, 3)) == (64, 72)
    d = M.make_descs([((64, 8, 3, 3), 0), (32, 48, 1), ((10, 7), 2, 5)])
    assert (d[0].rows, d[0].cols, d[0].module) == (64, 72, 0)
    assert (d[1].rows, d[1].cols) == (32, 48)
    assert (d[2].rows, d[2].cols, d[2].rank_override) == (10, 7, 5)
    with pytest.raises(ValueError):
        M.flatten_shape((5,))


def test_version_names_the_target():
    _lib()
    v = M.moara_version()
    assert re.fullmatch(r"moara-mi355x \d+\.\d+ \(gfx950\)", v), v


def test_last_error_is_per_thread():
    """moara_last_error is thread-local: an error raised in one thread does not replace the
    message another thread reads for its own last error."""
    import threading
    _lib()
    cfg = M.moara_default_config(rank_table=[8] * 10)
    gate, out = threading.Barrier(2), {}

    def bad_shape():
        try:
            M.moara_resolve_matrix(cfg, M.make_descs([(0, 5, 0)])[0])
        except M.MoaraError:
            pass
        gate.wait()   # the other thread fails while this one still holds its message
        gate.wait()
        out["shape"] = M.moara_last_error()

    def bad_rank():
        gate.wait()
        try:
            M.moara_allocate_ranks(256, range(7), [0, 1, 2], [5, 6], 1)
        except M.MoaraError:
            pass
        out["rank"] = M.moara_last_error()
        gate.wait()

    ts = [threading.Thread(target=bad_shape), threading.Thread(target=bad_rank)]
    for t in ts:
        t.start()
    for t in ts:
        t.join(timeout=30)
    assert "shape" in out["shape"] and "receiver share" not in out["shape"], out
    assert "receiver share" in out["rank"], out


def test_failed_calls_leave_outputs_as_documented():
    """On error moara_allocate_ranks leaves the caller's table unchanged and
    moara_create_state sets *out to NULL (both before any GPU work)."""
    L = _lib()
    tab = (ctypes.c_int32 * M.MOARA_NUM_MODULES)(*range(100, 110))
    rc = L.moara_allocate_ranks(256, 0x7F, 0x7, 0x60, 1, tab)    # share 1 * 3 / 2 is not an integer
    assert rc == M.MOARA_E_RANK and list(tab) == list(range(100, 110))
    cfg = M.moara_default_config(rank_table=[8] * 10, weight_decay=0.5)
    h = ctypes.c_void_p(0x1234)
    rc = L.moara_create_state(ctypes.byref(cfg), M.make_descs([(64, 64, 0)]), 1, None, ctypes.byref(h))
    assert rc == M.MOARA_E_UNSUPPORTED and not h.value
