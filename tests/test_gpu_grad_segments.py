"""Row gradients of rows of many segments: dA(m)[i] adds the row's segment sums, so its error must not grow with
their number.  Rows of 0, 1, 17, 128, 129 and some thousand segments, several long ones in one wavefront, at every
compiled J.

Every element of a row has the same upstream value, the same other indices and equal ranks, so that an FP32 chain over the
segments rounds alike at every step and its error adds up: the test asserts that such a chain would miss the bound.
Bound, relative to the sum (all terms positive): a segment's terms are N - 1 products and an FP32 sum over at most
512 / 8 additions and 3 tree steps of a wavefront, the product with B adds R terms: (N + 64 + 3 + R + 2) 2^-24.
"""
import numpy as np
import pytest

from tests.gpu_common import to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order,J,R", [(3, 8, 8), (3, 16, 16), (3, 32, 32), (4, 32, 32), (8, 8, 16)])
def test_rows_of_many_segments(order, J, R):
    import torch

    import paper_2210_06014_amd as ft

    nnz = 768_000
    seg = min(max(nnz // 4096 // 64 * 64, 64), 512)
    lens = np.zeros(37, dtype=np.int64)
    lens[[0, 1, 2, 3, 4, 6, 15, 16, 20, 36]] = [500_000, 128 * seg, 128 * seg + 1, 17 * seg, 1, 33 * seg - 1, 60_000,
                                                129 * seg, seg, seg + 1]
    lens[35] = nnz - lens.sum()
    assert lens[35] > 0
    row = np.repeat(np.arange(lens.size), lens)
    c = np.zeros((order, nnz), dtype=np.int32)
    c[0] = row
    rng = np.random.default_rng(order + J)
    c = np.ascontiguousarray(c[:, rng.permutation(nnz)])
    dims = [lens.size] + [2] * (order - 1)
    A = [np.tile(rng.uniform(0.2, 0.5, (1, J)).astype(np.float32), (d, 1)) for d in dims]
    B = [np.tile(rng.uniform(0.2, 0.5, (J, 1)).astype(np.float32), (1, R)) for _ in dims]  # every rank alike
    plan = ft.Plan(dims, J, R, c, np.ones(nnz, dtype=np.float32), with_perm=True)
    assert plan.mode_info(0)["segments"] == int(np.sum((lens + seg - 1) // seg))
    prm = ft.Params(A, B)
    ft.refresh(plan, prm)
    w = np.ones(R)
    for n in range(1, order):
        w = w * to_np(prm.C[n])[0]
    bound = (order + 64 + 3 + R + 2) * 2.0 ** -24
    # the upstream value (of a few) at which an FP32 chain over the segments of row 0 errs most
    nseg = int((lens[0] + seg - 1) // seg)
    ups = np.linspace(0.3, 0.9, 40).astype(np.float32)
    sums = (seg * w[0] * ups.astype(np.float64)).astype(np.float32)
    chain = np.cumsum(np.repeat(sums[None], nseg, axis=0), axis=0, dtype=np.float32)[-1].astype(np.float64)
    miss = np.abs(chain / (nseg * sums.astype(np.float64)) - 1)
    assert miss.max() > 2 * bound
    u = float(ups[np.argmax(miss)])
    up = torch.full((nnz,), u, dtype=torch.float32, device="cuda")
    gA, _ = ft.grad(plan, prm, up)
    got = to_np(gA[0])
    want = lens[:, None] * (B[0].astype(np.float64) @ (u * w))
    assert np.all(got[lens == 0] == 0)
    some = lens > 0
    err = np.abs(got[some] / want[some] - 1).max(axis=1)
    print(f"\n[grad segments] order {order} J {J} R {R}: {dict(zip(lens[some].tolist(), err.tolist()))}", flush=True)
    assert np.all(err <= bound), (err.max(), bound)
