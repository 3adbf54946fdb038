"""Folds of chunk maps: rows of one map, of as many as the last fold takes in sequence, of one more, and of the
same around the second and third level, at every compiled J.  Chunks of two elements and heads of four make a row of
4 + 2 k elements k maps.  Against the oracle's serial pass; tolerance as in test_gpu_factor_blocks."""
import numpy as np
import pytest

from tests.gpu_common import delta_ok, gpu_setup, oracle_model, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("J,R,order", [(8, 8, 3), (16, 16, 3), (32, 32, 3), (8, 16, 8), (32, 32, 5)])
@pytest.mark.parametrize("fanin", [0, 3])
def test_map_counts(J, R, order, fanin):
    import torch

    import paper_2210_06014_amd as ft

    counts = [1, 2, 3, 4, 8, 9, 10, 15, 16, 17, 27, 28, 31, 33, 255, 256, 257, 300]
    rng = np.random.default_rng(J + order)
    dims = [len(counts)] + [40] * (order - 1)
    cols = []
    for i, k in enumerate(counts):
        cell = rng.choice(40 ** min(order - 1, 3), size=4 + 2 * k - (i % 2), replace=False)  # odd rows: a last chunk of one
        cols.append(np.stack([np.full(cell.size, i)] + [cell // 40 ** n % 40 for n in range(order - 1)]))
    c = np.concatenate(cols, axis=1).astype(np.int32)
    c = np.ascontiguousarray(c[:, rng.permutation(c.shape[1])])
    v = rng.integers(1, 6, c.shape[1]).astype(np.float32)
    A = [rng.normal(0, 0.3, (d, J)).astype(np.float32) for d in dims]
    B = [rng.normal(0, 0.3, (J, R)).astype(np.float32) for _ in dims]
    plan, prm = gpu_setup(dims, J, R, c, v, A, B, chunk=2, head=4, fanin=fanin)
    orc = oracle_model(dims, J, R, c, v, A, B)
    before = orc.A[0].copy()
    ft.factor_pass(plan, prm, 0, 1e-2, 1e-2)
    orc.factor_pass(0, 1e-2, 1e-2)
    torch.cuda.synchronize()
    ok, err, bound = delta_ok(to_np(prm.A[0]), orc.A[0], before)
    assert ok, (err, bound)
