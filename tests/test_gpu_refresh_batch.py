"""GPU: a refresh batch large enough for the left-looking Cholesky form (its matrices' cubed block
counts add up to over 1300 times the square of the largest) against the same matrices in chunks that
take the right-looking one, and against the oracle."""
import numpy as np
import pytest

import workloads as WL
from oracle import moara_oracle as O
from tests.harness import Case, gpu_state, oracle_projector, rng, to_dev

pytestmark = pytest.mark.gpu


def test_left_and_right_looking_factorisations_are_bit_identical(monkeypatch):
    import torch
    from paper_2609_15037_amd import moara as M
    # w = r + p of 200 and 80 columns: four 64-blocks (the last of 8 columns) and two (of 16)
    big, small = 330, 20
    c = Case(shapes=[(256, 288, WL.Q)] * big + [(300, 130, WL.UP)] * small, ranks=[100] * big + [40] * small,
             block_size=32)
    assert big * 4 ** 3 + small * 2 ** 3 > 1300 * 4 ** 2
    G = []
    for i, (m, n, _) in enumerate(c.shapes):
        g = rng(7, i)
        A, B = g.standard_normal((m, 120)), g.standard_normal((n, 120))
        G.append(((A * np.arange(1, 121) ** -1.0) @ B.T + 1e-3 * g.standard_normal((m, n))).astype(np.float32))
    Gd = [to_dev(g, "f32") for g in G]
    out = []
    for budget in (None, "64"):   # MiB: a few dozen matrices a chunk
        if budget:
            monkeypatch.setenv("MOARA_REFRESH_CHUNK_MIB", budget)
        else:
            monkeypatch.delenv("MOARA_REFRESH_CHUNK_MIB", raising=False)
        st = gpu_state(c)
        print(f"[refresh] {len(G)} matrices, chunk budget {budget or 'default'}", flush=True)
        M.moara_refresh_projector(st, Gd)
        torch.cuda.synchronize()
        out.append([M.moara_get_tensor(st, i, M.MOARA_T_P) for i in range(len(G))])
    assert M.moara_state_bytes(st.cfg, M.make_descs([(m, n, mod, r) for (m, n, mod), r in zip(c.shapes, c.ranks)]))[1] < (
        2 << 30)   # one chunk by default
    for i, (a, b) in enumerate(zip(*out)):
        assert np.array_equal(a, b), f"matrix {i}: the projector depends on the chunks"
    for i in (0, 77, big - 1, big, len(G) - 1):
        ang = O.max_principal_angle(out[0][i].astype(np.float64), oracle_projector(G[i], c, i))
        assert ang <= 1e-3, f"matrix {i}: principal angle {ang:.2e}"
