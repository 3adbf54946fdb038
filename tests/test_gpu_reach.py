"""In-place part of long rows past the head (default chunk and head, J = 16 and 32).

200 x 3000 x 2000, 2M elements, Zipf 1.1: in mode 0 every row is longer than the head and the
plan's estimate updates about half of the rows in one piece (J = 32); the other rows keep chunk maps after a
longer in-place part.  Checked against the oracle, with the bound of the other passes, for the rows on either side of that
length, the longest and the shortest; a plan that states chunk or head keeps the pieces it states.
"""
import numpy as np
import pytest

import oracle
import synth
from tests.gpu_common import delta_ok, to_np

DIMS, NNZ = [200, 3000, 2000], 2_000_000


@pytest.fixture(scope="module")
def problem():
    c, _ = synth.coords(DIMS, NNZ, 1.1, seed=21)
    v = synth.values(NNZ, "int1to5", seed=21)
    return c, v, np.bincount(c[0], minlength=DIMS[0])


def _pieces(counts, head, chunk):
    long = counts[counts > head]
    return int(np.sum(1 + (long - head + chunk - 1) // chunk))


@pytest.mark.parametrize("kw", [dict(chunk=1024), dict(head=2048), dict(relaxed=True)])
def test_stated_pieces_stay(problem, kw):
    import paper_2210_06014_amd as ft

    c, v, counts = problem
    info = ft.Plan(DIMS, 32, 32, c, v, upload=False, **kw).mode_info(0)
    assert info["heavy_rows"] == int(np.sum(counts > info["head"]))
    assert info["chunks"] == _pieces(counts, info["head"], info["chunk"])


@pytest.mark.gpu
@pytest.mark.parametrize("J", [16, 32])
@pytest.mark.parametrize("fiber_share", [True, False])
def test_rows_about_the_reach(problem, fiber_share, J):
    import torch

    import paper_2210_06014_amd as ft

    c, v, counts = problem
    R = J
    A, B = synth.init_params(DIMS, J, R, 0.1, seed=22)
    plan = ft.Plan(DIMS, J, R, c, v, fiber_share=fiber_share)
    info = plan.mode_info(0)
    assert info["chunks"] < _pieces(counts, info["head"], info["chunk"])  # the estimate takes more in place
    order = np.argsort(counts, kind="stable")
    n = info["light_rows"]
    assert J == 16 or (8 < n < DIMS[0] - 8 and counts[order[n - 1]] > info["head"])  # (J = 16: every row keeps maps)
    rows = np.unique(order[np.clip([0, 1, n // 2, n - 2, n - 1, n, n + 1, n + 20, DIMS[0] - 1], 0, None)])
    prm = ft.Params(A, B)
    ft.refresh(plan, prm)
    print(f"\n[reach] rows {rows.tolist()} lengths {counts[rows].tolist()} J={J} fiber_share={fiber_share}", flush=True)
    lr, lam = 1e-3, 1e-2
    before = to_np(prm.A[0])
    ft.factor_pass(plan, prm, 0, lr, lam)
    torch.cuda.synchronize()
    sel = np.isin(c[0], rows)
    orc = oracle.Model(DIMS, [J] * 3, R, np.ascontiguousarray(c[:, sel]), v[sel].astype(np.float64),
                       [a.astype(np.float64) for a in A], [b.astype(np.float64) for b in B])
    orc.factor_pass(0, lr, lam)
    got = to_np(prm.A[0])
    for i in rows:
        ok, err, bound = delta_ok(got[i], orc.A[0][i], before[i])
        assert ok, (int(i), int(counts[i]), err, bound)
