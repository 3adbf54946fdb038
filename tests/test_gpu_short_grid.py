"""Core gradient of the smallest mode that lists its short rows apart (16384 of them), whose wavefronts take 8 to 64
rows each: the rows fill a part of the workgroups a segment per wavefront would ask for.  Tolerance as in
test_gpu_reductions: 1e-5 of the sum of the terms' magnitudes."""
import numpy as np
import pytest

from tests.gpu_common import gpu_setup, oracle_model, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("J,R,order", [(8, 8, 3), (16, 16, 3), (32, 32, 3), (8, 16, 8)])
@pytest.mark.parametrize("rows", [16384, 16385])
def test_core_gradient(J, R, order, rows):
    import paper_2210_06014_amd as ft

    rng = np.random.default_rng(rows + J)
    lens = rng.integers(1, 9, rows)
    nnz = int(lens.sum())
    dims = [rows] + [25] * (order - 1)
    c = np.stack([np.repeat(np.arange(rows), lens)] + [rng.integers(0, 25, nnz) for _ in range(order - 1)])
    c = np.ascontiguousarray(c[:, rng.permutation(nnz)].astype(np.int32))
    v = rng.integers(1, 6, nnz).astype(np.float32)
    A = [rng.normal(0, 0.4, (d, J)).astype(np.float32) for d in dims]
    B = [rng.normal(0, 0.4, (J, R)).astype(np.float32) for _ in dims]
    orc = oracle_model(dims, J, R, c, v, A, B)
    w = np.ones((nnz, R))
    for n in range(1, order):
        w = w * np.abs(orc.C[n][c[n]])
    scale = np.abs(A[0].astype(np.float64)[c[0]]).T @ (np.abs(v - orc.predict(c))[:, None] * w)
    plan, prm = gpu_setup(dims, J, R, c, v, A, B)
    got, want = to_np(ft.core_grad(plan, prm, 0)), orc.core_grad(0)
    assert np.all(np.abs(got - want) <= 1e-5 * scale + 1e-12)
