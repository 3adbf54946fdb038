"""The length of the in-place part of long rows, as reported: it accounts for the pieces of every plan, and rows of
lengths on either side of it match the oracle (default plans, whose estimate may put it past the default head, J = 32, or
at two chunks, J = 16).  The tolerance is that of the other passes."""
import numpy as np
import pytest

import oracle
import synth
from tests.gpu_common import delta_ok, to_np

DIMS = [20_000, 3_000, 300]


@pytest.fixture(scope="module")
def problem():
    c, _ = synth.coords(DIMS, 6_000_000, 1.1, seed=31)
    v = synth.values(c.shape[1], "int1to5", seed=31)
    return c, v, [np.bincount(c[m], minlength=DIMS[m]) for m in range(3)]


def _check(info, counts):
    n, chunk = info["in_place"], info["chunk"]
    long = counts[counts > n]
    assert info["heavy_rows"] == long.size
    assert info["light_rows"] == int(np.sum((counts > 0) & (counts <= n)))
    assert info["chunks"] == int(np.sum(1 + (long - n + chunk - 1) // chunk))


@pytest.mark.parametrize("J,kw", [(8, {}), (16, {}), (32, {}), (32, dict(head=2048)), (16, dict(chunk=256)),
                                  (16, dict(relaxed=True))])
def test_reported_length_accounts_for_the_pieces(problem, J, kw):
    import paper_2210_06014_amd as ft

    c, v, counts = problem
    plan = ft.Plan(DIMS, J, J, c, v, upload=False, **kw)
    for m in range(3):
        info = plan.mode_info(m)
        _check(info, counts[m])
        if J == 8 or kw:
            assert info["in_place"] == info["head"]
        elif J == 16:
            assert info["in_place"] == 1024  # thousands of chunks
        else:
            assert info["in_place"] >= info["head"]
    if J == 32 and not kw:
        assert any(plan.mode_info(m)["in_place"] > plan.mode_info(m)["head"] for m in range(3))


@pytest.mark.gpu
@pytest.mark.parametrize("J", [16, 32])
def test_rows_about_the_length(problem, J):
    import torch

    import paper_2210_06014_amd as ft

    c, v, counts = problem
    A, B = synth.init_params(DIMS, J, J, 0.1, seed=32)
    plan = ft.Plan(DIMS, J, J, c, v)
    prm = ft.Params(A, B)
    ft.refresh(plan, prm)
    lr, lam = 1e-3, 1e-2
    for m in range(3):
        n, chunk = plan.mode_info(m)["in_place"], plan.mode_info(m)["chunk"]
        near = [int(np.argmin(np.abs(counts[m] - t))) for t in (n, n - 1, n + 1, n + chunk, n + chunk + 1, n + 5 * chunk,
                                                                 1024, 1025, 17, 16)]
        rows = np.unique(near + [int(np.argmax(counts[m]))])
        print(f"\n[in place] J {J} mode {m}: {n} elements, rows of {counts[m][rows].tolist()}", flush=True)
        A_now, B_now = [to_np(a) for a in prm.A], [to_np(b) for b in prm.B]
        ft.factor_pass(plan, prm, m, lr, lam)
        torch.cuda.synchronize()
        sel = np.isin(c[m], rows)
        orc = oracle.Model(DIMS, [J] * 3, J, np.ascontiguousarray(c[:, sel]), v[sel].astype(np.float64), A_now, B_now)
        orc.factor_pass(m, lr, lam)
        got = to_np(prm.A[m])
        for i in rows:
            ok, err, bound = delta_ok(got[i], orc.A[m][i], A_now[m][i])
            assert ok, (m, int(i), int(counts[m][i]), err, bound)
        ft.refresh(plan, prm, m)
