"""Core gradient, gradients and forward on a mode with many short rows, which a slot of a wavefront takes each:
rows of 1 to 33 elements (32 is the longest of them) beside empty and long ones, at every compiled J and both
storages, and row counts that leave the last wavefront's slots empty.

Tolerance: FP32 sums of n terms of N + 1 factors each, |d| <= (n + 16) 2^-23 sum of the terms' magnitudes for the row
gradients (n the row's elements), 1e-5 of it for the sums over the mode; BF16 through its storage bound, twice
(N + 1) 2^-8 of the same sums."""
import numpy as np
import pytest

from tests.gpu_common import gpu_setup, oracle_model, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order,J,R", [(3, 8, 8), (3, 16, 16), (3, 32, 32), (4, 8, 8), (4, 32, 32), (8, 8, 16)])
@pytest.mark.parametrize("rows", [18_000, 18_777])
def test_short_rows(order, J, R, rows):
    import torch

    import paper_2210_06014_amd as ft

    rng = np.random.default_rng(order + J)
    lens = rng.integers(0, 34, rows)
    lens[:4] = [700, 513, 33, 32]
    dims = [rows] + [30] * (order - 1)
    row = np.repeat(np.arange(rows), lens)
    nnz = row.size
    start = np.repeat(np.cumsum(lens) - lens, lens)
    cell = (np.arange(nnz) - start) * 7 + rng.integers(0, 7, nnz)  # distinct within a row
    c = np.stack([row] + [cell // 30 ** n % 30 if n < 3 else rng.integers(0, 30, nnz) for n in range(order - 1)])
    keep = cell < 30 ** min(order - 1, 3)
    c, nnz = c[:, keep], int(keep.sum())
    perm = rng.permutation(nnz)
    c = np.ascontiguousarray(c[:, perm].astype(np.int32))
    v = rng.integers(1, 6, nnz).astype(np.float32)
    A = [rng.normal(0, 0.3, (d, J)).astype(np.float32) for d in dims]
    B = [rng.normal(0, 0.3, (J, R)).astype(np.float32) for _ in dims]
    orc = oracle_model(dims, J, R, c, v, A, B)
    xh = orc.predict(c)
    w = np.ones((nnz, R))
    for n in range(1, order):
        w = w * orc.C[n][c[n]]
    S = [np.abs(a.astype(np.float64)) @ np.abs(b.astype(np.float64)) for a, b in zip(A, B)]
    wabs = np.ones((nnz, R))
    for n in range(1, order):
        wabs = wabs * S[n][c[n]]
    up = rng.normal(0, 1, nnz).astype(np.float32)
    count = np.bincount(c[0], minlength=rows)
    for storage in ("f32", "bf16"):
        plan, prm = gpu_setup(dims, J, R, c, v, A, B, storage=storage, with_perm=True)
        assert np.sum((count > 0) & (count <= 32)) >= 16384
        got_x = to_np(ft.forward(plan, prm))
        xs = (S[0][c[0]] * wabs).sum(1)
        eps = 1e-5 if storage == "f32" else 2 * (order + 1) * 2.0 ** -8
        assert np.all(np.abs(got_x - xh) <= eps * xs)
        for delta, kind in ((v - xh, "core"), (xh - v, "own"), (up.astype(np.float64), "up")):
            mag = np.abs(delta) + (0 if kind == "up" else eps * xs)
            t, tm = np.zeros((rows, R)), np.zeros((rows, R))
            np.add.at(t, c[0], delta[:, None] * w)
            np.add.at(tm, c[0], mag[:, None] * wabs)
            gB, gBm = A[0].astype(np.float64).T @ t, np.abs(A[0].astype(np.float64)).T @ tm
            if kind == "core":
                assert np.all(np.abs(to_np(ft.core_grad(plan, prm, 0)) - gB) <= 2 * eps * gBm)
                continue
            hA, hB = ft.grad(plan, prm, torch.from_numpy(up).cuda() if kind == "up" else None)
            gA = t @ B[0].astype(np.float64).T
            gAm = tm @ np.abs(B[0].astype(np.float64)).T
            assert np.all(np.abs(to_np(hA[0]) - gA) <= 2 * eps * gAm), kind
            assert np.all(np.abs(to_np(hB[0]) - gB) <= 2 * eps * gBm), kind
            assert np.all(to_np(hA[0])[count == 0] == 0)
