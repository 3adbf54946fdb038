"""Predictions in wavefronts of 64 queries, with the index range checked by the kernel: query counts around the
edges of a wavefront and a workgroup, and one index out of range (below, above) in each mode.

Tolerance: FP32 products of N values and a sum over R, |d| <= (N + R) 2^-24 sum_r prod_n |C(n)| (times 2 for the
rounding of C itself); BF16 reads exact widenings of C16, so the same bound holds against C16."""
import numpy as np
import pytest

from tests.gpu_common import abs_scale, gpu_setup, make_problem, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order,J,R", [(3, 8, 8), (3, 16, 16), (3, 32, 32), (4, 8, 8), (8, 8, 16)])
@pytest.mark.parametrize("storage", ["f32", "bf16"])
def test_query_counts_and_range(order, J, R, storage):
    import torch

    import paper_2210_06014_amd as ft

    dims = [37, 21, 18, 9, 8, 7, 6, 5][:order]
    c, v, A, B = make_problem(dims, 3000, 0.0, J, R, seed=3)
    plan, prm = gpu_setup(dims, J, R, c, v, A, B, storage=storage)
    C = [to_np(t.float()) for t in (prm.C if storage == "f32" else prm.C16)]
    rng = np.random.default_rng(4)
    for q in (0, 1, 7, 63, 64, 65, 255, 256, 257, 1000):
        x = np.stack([rng.integers(0, d, q) for d in dims]).astype(np.int32)
        if q:
            x[:, 0] = 0
            x[:, -1] = np.array(dims) - 1
        got = to_np(ft.predict(plan, prm, torch.from_numpy(x).cuda()))
        want = np.ones((q, R))
        for n in range(order):
            want = want * C[n][x[n]]
        assert got.shape == (q,)
        assert np.all(np.abs(got - want.sum(1)) <= 2 * (order + R) * 2.0 ** -24 * abs_scale(C, x) + 1e-30), q
    for n in range(order):
        for wrong in (-1, dims[n], 2**31 - 1, -(2**31)):
            for at in (0, 64, 129):
                x = np.zeros((order, 130), dtype=np.int32)
                x[n, at] = wrong
                with pytest.raises(ValueError, match=f"mode {n} out of range"):
                    ft.predict(plan, prm, torch.from_numpy(x).cuda())
    assert to_np(ft.predict(plan, prm, torch.zeros((order, 3), dtype=torch.int32, device="cuda"))).shape == (3,)
