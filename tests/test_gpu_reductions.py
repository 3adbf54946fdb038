"""The reductions of the loss and of the core gradient: regulariser sums of matrices that start off a 16-byte
boundary or end inside a 16-byte load, and core gradients from one workgroup's partial up to many.

Tolerances: the sums of squares run in FP64 over FP32 values, relative 1e-12; the gradient is an FP32 sum, held to
1e-5 of the sum of its terms' magnitudes."""
import numpy as np
import pytest

from tests.gpu_common import gpu_setup, make_problem, oracle_model, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [1, 5, 513, 70_001])
def test_regularisers_of_unaligned_matrices(rows):
    import torch

    import paper_2210_06014_amd as ft

    dims, J, R = [rows, 9, 8], 8, 8
    nnz = min(300, rows * 72)
    c, v, A, B = make_problem(dims, nnz, 0.0, J, R, seed=6)
    plan, prm = gpu_setup(dims, J, R, c, v, A, B)
    want = [3e-2 * sum(float((x.astype(np.float64) ** 2).sum()) for x in A),
            5e-2 * sum(float((x.astype(np.float64) ** 2).sum()) for x in B)]
    for off in (0, 1, 3):
        for n in range(3):
            flat = torch.zeros(A[n].size + off, dtype=torch.float32, device="cuda")
            flat[off:] = torch.from_numpy(A[n]).cuda().reshape(-1)
            prm.A[n] = flat[off:].reshape(A[n].shape)
        got = to_np(ft.loss(plan, prm, 3e-2, 5e-2))
        np.testing.assert_allclose(got[2:], want, rtol=1e-12)


@pytest.mark.parametrize("J,R,order", [(8, 8, 3), (16, 16, 3), (32, 32, 3), (8, 16, 8)])
@pytest.mark.parametrize("rows", [1, 3, 70, 1100, 9000])
def test_core_gradient_partials(J, R, order, rows):
    import paper_2210_06014_amd as ft

    dims = [rows] + [11] * (order - 1)
    nnz = min(3 * rows + 20, rows * 11 ** min(order - 1, 3) // 2)
    c, v, A, B = make_problem(dims, nnz, 0.0, J, R, seed=8)
    plan, prm = gpu_setup(dims, J, R, c, v, A, B)
    orc = oracle_model(dims, J, R, c, v, A, B)
    got, want = to_np(ft.core_grad(plan, prm, 0)), orc.core_grad(0)
    w = np.ones((nnz, R))
    for n in range(1, order):
        w = w * np.abs(orc.C[n][c[n]])
    e = np.abs(v - orc.predict(c))
    scale = np.abs(A[0].astype(np.float64)[c[0]]).T @ (e[:, None] * w)
    assert np.all(np.abs(got - want) <= 1e-5 * scale + 1e-12)
