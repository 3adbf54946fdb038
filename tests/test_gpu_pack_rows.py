"""Factor passes over many short rows, which share blocks of 16 slots: every row length around the edges (1 to 18)
in random order, with empty and longer rows between, rows of exactly 16, every compiled J, both storages, shared g, a
decay that shrinks blocks to single elements, and values that are not finite, which stay in their own row.

Against the oracle's serial pass from the same state; tolerance as in test_gpu_factor_blocks."""
import numpy as np
import pytest

from tests.gpu_common import delta_ok, gpu_setup, oracle_model, to_np

pytestmark = pytest.mark.gpu


def _problem(order, J, R, fibers, seed=12):
    rng = np.random.default_rng(seed)
    lens = rng.choice([0, 1, 2, 3, 5, 7, 8, 9, 15, 16, 17, 18, 40], size=700,
                      p=[.1, .12, .1, .1, .1, .1, .08, .08, .06, .06, .04, .03, .03])
    lens[:6] = [16, 16, 8, 8, 1, 15]
    lens[-3:] = [0, 2, 1]
    side = 6 if fibers else 30
    dims = [lens.size] + [side] * (order - 1)
    cells = side ** min(order - 1, 3)
    cols = []
    for i, L in enumerate(lens):
        k = rng.choice(cells, size=min(L, cells), replace=False)
        cols.append(np.stack([np.full(k.size, i)] + [k // side ** n % side if n < 3 else rng.integers(0, side, k.size)
                                                     for n in range(order - 1)]))
    c = np.concatenate(cols, axis=1).astype(np.int32)
    c = np.ascontiguousarray(c[:, rng.permutation(c.shape[1])])
    v = rng.integers(1, 6, c.shape[1]).astype(np.float32)
    A = [rng.normal(0, 0.3, (d, J)).astype(np.float32) for d in dims]
    B = [rng.normal(0, 0.3, (J, R)).astype(np.float32) for _ in dims]
    return dims, c, v, A, B


CONFIGS = [(3, 8, 8, False), (3, 16, 16, False), (3, 16, 16, True), (3, 32, 32, False), (3, 32, 32, True),
           (4, 8, 8, False), (4, 32, 32, False), (8, 8, 16, False)]


@pytest.mark.parametrize("order,J,R,fibers", CONFIGS)
@pytest.mark.parametrize("lr,lam", [(1e-2, 1e-2), (0.9, 0.9)])
def test_packed_rows(order, J, R, fibers, lr, lam):
    import paper_2210_06014_amd as ft

    dims, c, v, A, B = _problem(order, J, R, fibers)
    count = np.bincount(c[0], minlength=dims[0])
    for storage in ("f32", "bf16"):
        for kw in ({}, {"head": 8, "chunk": 5}, {"relaxed": True}):
            if storage == "bf16" and kw:
                continue
            plan, prm = gpu_setup(dims, J, R, c, v, A, B, storage=storage, **kw)
            orc = oracle_model(dims, J, R, c, v, A, B)
            if storage == "bf16":  # the pass reads B16 and C16 and updates the master: the same inputs for the oracle
                for n in range(order):
                    orc.C[n][:] = to_np(prm.C16[n].float())
                orc.B[0][:] = to_np(prm.B16[0].float())
            before = orc.A[0].copy()
            orc.factor_pass(0, lr, lam)
            if fibers:
                assert plan.mode_info(0)["fiber_shared"] == 1
            ft.factor_pass(plan, prm, 0, lr, lam)
            got = to_np(prm.A[0])
            assert np.array_equal(got[count == 0], before[count == 0])
            ok, err, bound = delta_ok(got, orc.A[0], before)
            assert ok, (storage, kw, err, bound)


@pytest.mark.parametrize("order,J,R,fibers", [c for c in CONFIGS if not c[3]])
@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
def test_values_that_are_not_finite_stay_in_their_row(order, J, R, fibers, bad):
    import paper_2210_06014_amd as ft

    dims, c, v, A, B = _problem(order, J, R, fibers)
    plan, prm = gpu_setup(dims, J, R, c, v, A, B)
    ft.factor_pass(plan, prm, 0, 1e-2, 1e-2)
    clean = to_np(prm.A[0])
    hit = np.unique(c[0][[0, 17, 500, c.shape[1] - 1]])
    vb = v.copy()
    vb[[0, 17, 500, c.shape[1] - 1]] = bad
    plan, prm = gpu_setup(dims, J, R, c, vb, A, B)
    ft.factor_pass(plan, prm, 0, 1e-2, 1e-2)
    got = to_np(prm.A[0])
    rest = np.setdiff1d(np.arange(dims[0]), hit)
    assert not np.isfinite(got[hit]).all(axis=1).any()
    ok, err, bound = delta_ok(got[rest], clean[rest], A[0][rest].astype(np.float64))
    assert ok, (err, bound)
