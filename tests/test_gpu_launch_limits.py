"""More work items than one grid dimension holds: 68.7M chunks of one element each (chunk = head = 1), a wavefront
or a 16-lane group per chunk, where a launch takes fewer than 2^32 threads along x.

1100 x 250 x 250 with every cell present, J = R = 8, relaxed passes (nine floats per chunk; the maps of an exact pass
would take 20 GB).  Sampled rows against the oracle's relaxed pass on their elements, tolerance of the other passes.
"""
import numpy as np
import pytest

import oracle
from tests.gpu_common import delta_ok, to_np

pytestmark = pytest.mark.gpu


def test_chunks_past_one_grid_dimension():
    import torch

    import paper_2210_06014_amd as ft

    dims, J, R = [1100, 250, 250], 8, 8
    print("\n[launch limits] building 68.75M chunks", flush=True)
    c = np.indices(dims, dtype=np.int32).reshape(3, -1)
    v = (1 + np.arange(c.shape[1]) % 5).astype(np.float32)
    rng = np.random.default_rng(4)
    A = [rng.normal(0, 0.3, (d, J)).astype(np.float32) for d in dims]
    B = [rng.normal(0, 0.3, (J, R)).astype(np.float32) for _ in dims]
    plan = ft.Plan(dims, J, R, c, v, chunk=1, head=1, relaxed=True)
    assert plan.mode_info(0)["chunks"] - dims[0] >= 2 ** 26
    prm = ft.Params(A, B)
    ft.refresh(plan, prm)
    ft.factor_pass(plan, prm, 0, 1e-3, 1e-2)
    torch.cuda.synchronize()
    rows = [0, 1, 549, 1073, 1074, 1099]  # the last rows' chunks lie past 2^26 of them
    print(f"[launch limits] pass done, oracle on rows {rows}", flush=True)
    sel = np.isin(c[0], rows)
    orc = oracle.Model(dims, [J] * 3, R, np.ascontiguousarray(c[:, sel]), v[sel].astype(np.float64),
                       [a.astype(np.float64) for a in A], [b.astype(np.float64) for b in B])
    orc.factor_pass_relaxed(0, 1e-3, 1e-2, 1, 1)
    got = to_np(prm.A[0])
    for i in rows:
        ok, err, bound = delta_ok(got[i], orc.A[0][i], A[0][i].astype(np.float64))
        assert ok, (i, err, bound)
