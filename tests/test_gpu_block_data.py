"""Blocks of 16 elements where a wrong gradient shows: the problems of test_gpu_factor_blocks with C entries of order
one at every order (and larger values where the decay is above one half), so that the data part of a row's change is
not lost beside the decay (at order 8 it was a millionth of it), in both storages; the BF16 pass reads B16 and C16, which the oracle gets too.  Tolerance as there,
per row; the test asserts that a result which only decays misses it by a factor of twenty."""
import numpy as np
import pytest

from tests.gpu_common import delta_ok, gpu_setup, oracle_model, to_np
from tests.test_gpu_factor_blocks import LENGTHS, _problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("head", [16, 64, 1 << 30])
@pytest.mark.parametrize("lr,lam", [(1e-3, 1e-2), (2e-3, 260.0)])
@pytest.mark.parametrize("order,J,R,fibers", [(3, 8, 8, False), (3, 16, 16, True), (3, 32, 32, False), (4, 8, 8, False),
                                              (4, 32, 32, False), (6, 32, 32, False), (8, 8, 16, False)])
def test_data_part(order, J, R, fibers, head, lr, lam):
    import paper_2210_06014_amd as ft

    dims, c, v, A, B = _problem(order, J, R, 5, fibers)
    goal = 1.0 if order < 6 else 0.9
    v = v * np.float32(1.0 if lr * lam < 0.5 else 50.0)
    for n in range(order):
        s = np.sqrt(goal / np.sqrt(np.mean((A[n].astype(np.float64) @ B[n]) ** 2)))
        A[n], B[n] = (A[n] * s).astype(np.float32), (B[n] * s).astype(np.float32)
    lens = np.array([0] + LENGTHS)
    for storage in ("f32", "bf16"):
        plan, prm = gpu_setup(dims, J, R, c, v, A, B, storage=storage, chunk=33, head=head)
        orc = oracle_model(dims, J, R, c, v, A, B)
        if storage == "bf16":
            for n in range(order):
                orc.C[n][:] = to_np(prm.C16[n].float())
            orc.B[0][:] = to_np(prm.B16[0].float())
        before = orc.A[0].copy()
        ft.factor_pass(plan, prm, 0, lr, lam)
        orc.factor_pass(0, lr, lam)
        ok, err, bound = delta_ok(to_np(prm.A[0]), orc.A[0], before)
        assert ok, (storage, head, err, bound)
        decayed = before * ((1.0 - lr * lam) ** lens)[:, None]
        assert not delta_ok(decayed[1:], orc.A[0][1:], before[1:], rel=0.02)[0]
