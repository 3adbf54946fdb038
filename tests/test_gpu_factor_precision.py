"""The factor pass is as exact as one step per element with an FP64 row: its error against the oracle, over rows of
16, 700 (a wavefront each) and 2000 elements (a workgroup each), is at most 1.05 times that of the plain algorithm

    g = B w (FP32),  e = x - a.g (FP32),  a <- a + (-lr lam) a + (lr e) g (FP64)

restated in numpy on the same elements, in a learning regime (lr = 1e-2).  Both start from the same FP32 A, B and C,
which the oracle takes too, so that only the pass itself is compared; the final rounding to FP32 is in both.  Root mean
squares over some thousand entries agree between repetitions to about 1 %, hence the 5 %.
"""
import numpy as np
import pytest

from tests.gpu_common import gpu_setup, oracle_model, to_np

pytestmark = pytest.mark.gpu

LR, LAM = 1e-2, 1e-2


@pytest.mark.parametrize("J", [8, 16, 32])
@pytest.mark.parametrize("length,rows", [(16, 3000), (700, 400), (2000, 200)])
def test_error_of_a_pass(J, length, rows):
    import paper_2210_06014_amd as ft

    rng = np.random.default_rng(J + length)
    dims = [rows, 400, 300]
    nnz = rows * length
    cell = np.concatenate([rng.choice(dims[1] * dims[2], size=length, replace=False) for _ in range(rows)])
    c = np.stack([np.repeat(np.arange(rows), length), cell // dims[2], cell % dims[2]]).astype(np.int32)
    v = rng.uniform(1, 5, nnz).astype(np.float32)
    A = [(rng.normal(0, 1, (d, J)) * 0.35 / np.sqrt(J / 8)).astype(np.float32) for d in dims]
    B = [(rng.normal(0, 1, (J, J)) * 0.4).astype(np.float32) for _ in dims]
    plan, prm = gpu_setup(dims, J, J, c, v, A, B, keep_host=True, head=1 << 20)
    C = [to_np(x).astype(np.float32) for x in prm.C]
    orc = oracle_model(dims, J, J, c, v, A, B)
    for n in range(3):
        orc.C[n][:] = C[n]
    orc.factor_pass(0, LR, LAM)
    ft.factor_pass(plan, prm, 0, LR, LAM)
    got = to_np(prm.A[0])
    # the plain algorithm, all rows a step at a time
    _, idx, x, _ = plan.host_csr(0)
    idx, x = idx.reshape(2, rows, length), x.reshape(rows, length)
    a = A[0].astype(np.float64)
    for t in range(length):
        g = (C[1][idx[0][:, t]] * C[2][idx[1][:, t]]) @ B[0].T
        e = x[:, t] - np.sum(a.astype(np.float32) * g, axis=1, dtype=np.float32)
        a += np.float64(np.float32(-LR * LAM)) * a
        a += (np.float32(LR) * e).astype(np.float64)[:, None] * g.astype(np.float64)
    plain = a.astype(np.float32).astype(np.float64)
    err, want = (np.sqrt(np.mean((y - orc.A[0]) ** 2)) for y in (got, plain))
    print(f"\n[precision] J {J} length {length}: error {err:.3e}, plain {want:.3e}, ratio {err / want:.3f}, "
          f"max |A| {np.abs(orc.A[0]).max():.2f}", flush=True)
    assert err <= 1.05 * want
