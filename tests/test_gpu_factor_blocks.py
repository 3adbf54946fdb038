"""The factor kernels take a row in blocks of 16 elements: rows around the edges of a block, of the head and of
a chunk, every compiled (J, R), both storages, shared and per-element g, and a decay so strong (lr lam above one
half) that blocks shrink to one element.  Against the oracle's serial pass from the same state.

Tolerance: delta_ok's 1e-3 of a row's step plus 1e-6 of the row (FP32 sums of at most J + 16 terms per step,
FP64 row state), BF16 as in its error model (4 (N + 1) 2^-8 of the step)."""
import numpy as np
import pytest

from tests.gpu_common import delta_ok, gpu_setup, oracle_model, to_np

pytestmark = pytest.mark.gpu

LENGTHS = [1, 2, 15, 16, 17, 31, 32, 33, 48, 63, 64, 65, 79, 80, 81, 95, 96, 97, 127, 128, 129, 200]


def _problem(order, J, R, seed, fibers):
    """A tensor whose mode-0 rows have LENGTHS elements (row 0 empty): one column of distinct other indices per
    element, drawn from few fibers when `fibers`."""
    rng = np.random.default_rng(seed)
    dims = [len(LENGTHS) + 1] + ([15] * (order - 1) if fibers else [23 + n for n in range(order - 1)])
    cells = int(np.prod(dims[1:], dtype=np.int64))
    cols = []
    for i, L in enumerate(LENGTHS):
        k = rng.choice(min(cells, 10_000), size=L, replace=False)
        c = [np.full(L, i + 1)]
        for d in dims[1:]:
            c.append(k % d)
            k = k // d
        cols.append(np.stack(c))
    c = np.ascontiguousarray(np.concatenate(cols, axis=1).astype(np.int32))
    c = np.ascontiguousarray(c[:, rng.permutation(c.shape[1])])
    v = rng.integers(1, 6, c.shape[1]).astype(np.float32)
    A = [rng.normal(0, 0.2, (d, J)).astype(np.float32) for d in dims]
    B = [rng.normal(0, 0.2, (J, R)).astype(np.float32) for _ in dims]
    return dims, c, v, A, B


@pytest.mark.parametrize("lr,lam", [(1e-2, 1e-2), (0.9, 0.9)])
@pytest.mark.parametrize("head", [16, 64, 1 << 30])
@pytest.mark.parametrize("order,J,R,fibers", [(3, 8, 8, False), (3, 16, 16, True), (3, 32, 32, True),
                                              (3, 32, 32, False), (4, 8, 8, False), (4, 32, 32, False),
                                              (8, 8, 16, False)])
def test_block_edges(order, J, R, fibers, head, lr, lam):
    import paper_2210_06014_amd as ft

    dims, c, v, A, B = _problem(order, J, R, 5, fibers)
    for storage in ("f32", "bf16"):
        plan, prm = gpu_setup(dims, J, R, c, v, A, B, storage=storage, chunk=33, head=head)
        orc = oracle_model(dims, J, R, c, v, A, B)
        before = orc.A[0].copy()
        ft.factor_pass(plan, prm, 0, lr, lam)
        orc.factor_pass(0, lr, lam)
        got = to_np(prm.A[0])
        if storage == "f32":
            ok, err, bound = delta_ok(got, orc.A[0], before)
            assert ok, (head, err, bound)
            assert np.array_equal(got[0], before[0])  # the empty row
        else:
            # decay acts on the FP32 master; the data part carries the BF16 rounding
            data = np.abs(orc.A[0] - before).max() + np.abs(before).max() * (1 if lr * lam > 0.5 else 0)
            assert np.abs(got - orc.A[0]).max() <= 4 * (order + 1) * 2.0 ** -8 * data + 1e-6
