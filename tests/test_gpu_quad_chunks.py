"""Chunks and rows taken four to a wavefront (J <= 16, many of them): lengths around the edges of a block, last chunks
of one element, empty rows, counts that leave the last wavefront's rows of lanes empty, both storages, shared and
per-element g, no C cache, relaxed plans, and a decay above one half.

Against the oracle's pass from the same state (BF16: from the same C16 and B16); tolerance as in
test_gpu_factor_blocks.  The C entries are of order one at every order, so that the data part of a change is not lost
beside the decay: the test asserts that a result which only decays is off by more than 2 % of a row's change (twenty bounds).
"""
import numpy as np
import pytest

from tests.gpu_common import delta_ok, gpu_setup, oracle_model, to_np

pytestmark = pytest.mark.gpu

HEAD, CHUNK = 20, 17


def _problem(order, J, R, spare, seed=14):
    """Mode 0 of rows whose chunks number at least 60,000 plus `spare`."""
    rng = np.random.default_rng(seed + order)
    lens = rng.integers(HEAD + 1, 120, 19_000)
    lens[:40] = np.repeat([2000, HEAD + 1, HEAD + CHUNK, HEAD + CHUNK + 1, HEAD + 16, 1, 0, 3000], 5)
    lens[-1] = HEAD + 1 + spare * CHUNK
    side = 40
    dims = [lens.size] + [side] * (order - 1)
    nnz = int(lens.sum())
    c = np.stack([np.repeat(np.arange(lens.size), lens)] + [rng.integers(0, side, nnz) for _ in range(order - 1)])
    c = np.ascontiguousarray(c[:, rng.permutation(nnz)].astype(np.int32))
    v = rng.integers(1, 6, nnz).astype(np.float32)
    # C entries of about 0.7 at every order: the data part of a step then outweighs the decay
    A = [rng.normal(0, 1, (d, J)) / np.sqrt(J) for d in dims]
    B = [rng.normal(0, 1, (J, R)) * (1.0 if order < 8 else 0.85) for _ in dims]
    return dims, lens, c, v, [a.astype(np.float32) for a in A], [b.astype(np.float32) for b in B]


CASES = [(3, 8, 8, False), (3, 8, 8, True), (3, 16, 16, False), (3, 16, 16, True), (4, 8, 8, False), (8, 8, 16, False)]


@pytest.mark.parametrize("order,J,R,fibers", CASES)
@pytest.mark.parametrize("lr,lam,spare", [(1e-3, 1e-2, 1), (1e-3, 550.0, 2)])
def test_against_the_oracle(order, J, R, fibers, lr, lam, spare):
    import torch

    import paper_2210_06014_amd as ft

    dims, lens, c, v, A, B = _problem(order, J, R, spare)
    for storage, kw in (("f32", {}), ("bf16", {}), ("f32", {"relaxed": True}), ("f32", {"c_cache": False})):
        if "c_cache" in kw and (order, J, R) != (3, 16, 16):
            continue
        print(f"\n[quad] order {order} J {J} R {R} fibers {fibers} {storage} {kw} lr {lr} lam {lam}", flush=True)
        plan, prm = gpu_setup(dims, J, R, c, v, A, B, storage=storage, chunk=CHUNK, head=HEAD, fiber_share=fibers,
                              **kw)
        info = plan.mode_info(0)
        assert info["chunks"] - info["heavy_rows"] >= 60_000
        assert info["fiber_shared"] == int(fibers and "c_cache" not in kw)
        orc = oracle_model(dims, J, R, c, v, A, B)
        if storage == "bf16":
            for n in range(order):
                orc.C[n][:] = to_np(prm.C16[n].float())
            orc.B[0][:] = to_np(prm.B16[0].float())
        before = orc.A[0].copy()
        if kw.get("relaxed"):
            orc.factor_pass_relaxed(0, lr, lam, HEAD, CHUNK)
        else:
            orc.factor_pass(0, lr, lam)
        ft.factor_pass(plan, prm, 0, lr, lam)
        torch.cuda.synchronize()
        got = to_np(prm.A[0])
        ok, err, bound = delta_ok(got, orc.A[0], before)
        assert ok, (storage, kw, err, bound)
        decayed = before * ((1.0 - lr * lam) ** lens)[:, None]
        assert not delta_ok(decayed[lens > 0], orc.A[0][lens > 0], before[lens > 0], rel=0.02)[0]


@pytest.mark.parametrize("order,J,R", [(3, 8, 8), (3, 16, 16), (4, 8, 8)])
@pytest.mark.parametrize("relaxed", [False, True])
def test_rows(order, J, R, relaxed):
    """Rows in one piece of 17 to 1024 elements: 300 on average (four to a wavefront on their own), and beside chunks."""
    import torch

    import paper_2210_06014_amd as ft

    rng = np.random.default_rng(J)
    lens = np.concatenate([rng.integers(17, 600, 9000), [17, 18, 31, 32, 33, 1023, 1024, 1025, 5000, 0, 3]])
    rng.shuffle(lens)
    dims = [lens.size] + [60] * (order - 1)
    nnz = int(lens.sum())
    c = np.stack([np.repeat(np.arange(lens.size), lens)] + [rng.integers(0, 60, nnz) for _ in range(order - 1)])
    c = np.ascontiguousarray(c[:, rng.permutation(nnz)].astype(np.int32))
    v = rng.integers(1, 6, nnz).astype(np.float32)
    A = [(rng.normal(0, 1, (d, J)) / np.sqrt(J)).astype(np.float32) for d in dims]
    B = [rng.normal(0, 1, (J, R)).astype(np.float32) for _ in dims]
    for kw in (dict(head=1024), dict(head=300, chunk=40)):  # (the second: 60,000 chunks, heads beside shorter rows)
        print(f"\n[quad rows] order {order} J {J} relaxed {relaxed} {kw}", flush=True)
        plan, prm = gpu_setup(dims, J, R, c, v, A, B, relaxed=relaxed, **kw)
        orc = oracle_model(dims, J, R, c, v, A, B)
        before = orc.A[0].copy()
        if relaxed:
            orc.factor_pass_relaxed(0, 1e-3, 1e-2, kw["head"], kw.get("chunk", 512))
        else:
            orc.factor_pass(0, 1e-3, 1e-2)
        ft.factor_pass(plan, prm, 0, 1e-3, 1e-2)
        torch.cuda.synchronize()
        got = to_np(prm.A[0])
        assert np.array_equal(got[lens == 0], before[lens == 0])
        ok, err, bound = delta_ok(got, orc.A[0], before)
        assert ok, (kw, err, bound)


@pytest.mark.parametrize("order,J,R", [(3, 8, 8), (3, 16, 16)])
def test_same_bits(order, J, R):
    """Shared or per-element g, one launch or two."""
    import paper_2210_06014_amd as ft

    dims, lens, c, v, A, B = _problem(order, J, R, 1)
    got = []
    for kw in ({}, {"fiber_share": False}, {"fused": False}):
        plan, prm = gpu_setup(dims, J, R, c, v, A, B, chunk=CHUNK, head=HEAD, **kw)
        ft.factor_pass(plan, prm, 0, 1e-3, 1e-2)
        got.append(to_np(prm.A[0]))
    assert np.array_equal(got[0], got[1]) and np.array_equal(got[0], got[2])
