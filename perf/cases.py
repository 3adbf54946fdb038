"""Workloads for timing the framework through its public entry points.

Each case is one call pattern of a training or serving program: an iteration
of Algorithm 2 with its loss, a differentiable reconstruction with its
gradients, or a batch of predictions.  The tensors have the shapes, index
distributions, values, ranks and step sizes of the workloads in `synth`; the
element counts are smaller where those hold 50 to 200 million elements, so
that a plan is built in a few seconds.

`exact` restates the same mathematics in plain FP64 torch.
"""
from __future__ import annotations

import math

import torch

import paper_2210_06014_amd as ft

# Shapes and settings of the workloads: dimensions, Zipf exponent of the
# indices (0: uniform), kind of values, ranks, initial sigma, step size.
SHAPES = {
    "small": dict(dims=[1000] * 3, zipf=0.0, values="int", ranks=[(8, 8)], sigma=0.1, lr=1e-3, nnz=(20_000, 200_000)),
    "netflix": dict(dims=[480_000, 18_000, 2_200], zipf=1.1, values="int", ranks=[(16, 16), (32, 32)], sigma=0.1,
                    lr=1e-3, nnz=(200_000, 8_000_000)),
    "density": dict(dims=[1000] * 3, zipf=0.0, values="int", ranks=[(32, 32)], sigma=0.1, lr=1e-3,
                    nnz=(500_000, 8_000_000)),
    "planted": dict(dims=[100_000, 10_000, 1_000], zipf=1.1, values="planted", ranks=[(16, 16)], sigma=0.3, lr=1e-2,
                    nnz=(200_000, 4_000_000)),
    "order4": dict(dims=[1_000_000, 100_000, 10_000, 1_000], zipf=1.1, values="int", ranks=[(32, 32)], sigma=0.1,
                   lr=1e-3, nnz=(200_000, 3_000_000)),
    "order5": dict(dims=[10_000] * 5, zipf=0.0, values="int", ranks=[(32, 32)], sigma=0.1, lr=1e-3,
                   nnz=(50_000, 1_000_000)),
    "order6": dict(dims=[10_000] * 6, zipf=0.0, values="int", ranks=[(32, 32)], sigma=0.1, lr=1e-3,
                   nnz=(50_000, 1_000_000)),
    "order8": dict(dims=[10_000] * 8, zipf=1.05, values="normal", ranks=[(8, 16)], sigma=0.1, lr=1e-3,
                   nnz=(50_000, 1_000_000)),
    "order10": dict(dims=[10_000] * 10, zipf=0.0, values="int", ranks=[(32, 32)], sigma=0.1, lr=1e-3,
                    nnz=(50_000, 300_000)),
}
LAM = 1e-2  # weight decay of every workload


def _case(call, shape, J, R, nnz, storage="f32", relaxed=False, queries=0):
    return {"call": call, "shape": shape, "J": J, "R": R, "nnz": nnz, "storage": storage, "relaxed": relaxed,
            "queries": queries}


def listed():
    return [
        # a serving program asking for a handful of missing entries: launches and checks, no arithmetic to speak of
        dict(_case("predict", "small", 8, 8, 100_000, queries=1_000), name="predict_small_j8"),
        # held-out evaluation: predictions of a test set after training
        dict(_case("predict", "netflix", 32, 32, 200_000, queries=4_000_003), name="predict_netflix_j32"),
        # the smallest training problem, bound by launches and by the length of the rows' chains
        dict(_case("epoch", "small", 8, 8, 100_000), name="epoch_small_j8"),
        # the Netflix-shaped training iteration at the lower rank
        dict(_case("epoch", "netflix", 16, 16, 5_000_000), name="epoch_netflix_j16"),
        # the headline iteration: ranks 32, a few very long rows and many short ones, both storages
        dict(_case("epoch", "netflix", 32, 32, 8_000_000), name="epoch_netflix_j32"),
        dict(_case("epoch", "netflix", 32, 32, 8_000_000, storage="bf16"), name="epoch_netflix_j32_bf16"),
        # dense-ish tensor of few rows, 8000 elements each, with long fibers in every mode
        dict(_case("epoch", "density", 32, 32, 8_000_000), name="epoch_density_j32"),
        # higher orders: a very tall mode, uniform rows of a hundred elements, many gathered rows per element
        dict(_case("epoch", "order4", 32, 32, 3_000_000), name="epoch_order4_j32"),
        dict(_case("epoch", "order6", 32, 32, 999_999, storage="bf16"), name="epoch_order6_j32_bf16"),
        dict(_case("epoch", "order8", 8, 16, 1_000_000), name="epoch_order8_j8r16"),
        # relaxed factor passes in the learning regime (large steps)
        dict(_case("epoch", "planted", 16, 16, 4_000_000, relaxed=True), name="epoch_planted_relaxed_j16"),
        # the reconstruction inside a torch program: forward, loss, backward to A and B
        dict(_case("autograd", "planted", 16, 16, 1_000_003), name="autograd_planted_j16"),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: any shape, its ranks, an element count over its range, either storage."""
    call = rng.choice(["epoch", "epoch", "epoch", "autograd", "predict"])
    shape = rng.choice(sorted(SHAPES))
    s = SHAPES[shape]
    J, R = rng.choice(s["ranks"])
    storage = rng.choice(["f32", "bf16"])
    lo, hi = s["nnz"]
    if call == "predict":
        return _case(call, shape, J, R, _log_uniform(rng, lo, 4 * lo), storage,
                     queries=_log_uniform(rng, 1_000, 4_000_000 // (2 if len(s["dims"]) > 4 else 1)))
    if call == "autograd":
        return _case(call, shape, J, R, _log_uniform(rng, lo, min(hi, 1_500_000)), storage)
    relaxed = shape in ("netflix", "planted") and rng.random() < 0.25
    return _case(call, shape, J, R, _log_uniform(rng, lo, hi), storage, relaxed)


# --------------------------------------------------------------------------- inputs


def _columns(dims, zipf, count, gen, dev):
    """`count` random coordinates [order, count], each index Zipf(s) or uniform."""
    cols = []
    for d in dims:
        u = torch.rand(count, generator=gen, device=dev, dtype=torch.float64)
        if zipf:
            p = torch.arange(1, d + 1, dtype=torch.float64, device=dev).pow(-zipf)
            cols.append(torch.searchsorted(p.cumsum(0) / p.sum(), u).clamp_(max=d - 1))
        else:
            cols.append((u * d).long().clamp_(max=d - 1))
    return torch.stack(cols)


def _distinct(dims, zipf, count, gen, dev):
    """`count` distinct coordinates, int32 [order, count], in the order of the draws."""
    have = None
    while True:
        new = _columns(dims, zipf, int(1.1 * count) + 64, gen, dev)
        have = new if have is None else torch.cat([have, new], dim=1)
        # one 64-bit key per coordinate: the position in the tensor where that fits, else a mixed hash of it
        # (a coordinate that collides is dropped like a repeated one)
        key = torch.zeros(have.shape[1], dtype=torch.int64, device=dev)
        fits = math.prod(dims) < 2**62
        for n, d in enumerate(dims):
            key = key * d + have[n] if fits else (key ^ have[n]) * 0x1E3779B97F4A7C15 % (2**61) + (key >> 7)
        _, inv = torch.unique(key, return_inverse=True)
        first = torch.full((int(inv.max()) + 1,), have.shape[1], dtype=torch.int64, device=dev)
        first.scatter_reduce_(0, inv, torch.arange(have.shape[1], device=dev), "amin")
        have = have[:, first.sort().values]
        if have.shape[1] >= count:
            return have[:, :count].to(torch.int32)


def _inputs(case, seed, dev):
    """Coordinates (int32 [order, nnz]), values, initial A and B, and query coordinates, on the device."""
    s = SHAPES[case["shape"]]
    dims, J, R = s["dims"], case["J"], case["R"]
    gen = torch.Generator(device=dev).manual_seed(seed)
    coords = _distinct(dims, s["zipf"], case["nnz"], gen, dev)
    nnz = coords.shape[1]
    if s["values"] == "int":
        vals = torch.randint(1, 6, (nnz,), generator=gen, device=dev).float()
    else:
        noise = torch.randn(nnz, generator=gen, device=dev, dtype=torch.float64)
        if s["values"] == "normal":
            x = 3.0 + noise
        else:
            x = torch.full((nnz,), 4.0, dtype=torch.float64, device=dev)
            for n, d in enumerate(dims):
                u = 0.3 + 0.7 * torch.rand(d, generator=gen, device=dev, dtype=torch.float64)
                x = x * u[coords[n].long()]
            x = 1.0 + x + 0.25 * noise
        vals = x.clamp_(1.0, 5.0).float()
    A = [s["sigma"] * torch.randn(d, J, generator=gen, device=dev) for d in dims]
    B = [s["sigma"] * torch.randn(J, R, generator=gen, device=dev) for _ in dims]
    queries = None
    if case["queries"]:
        queries = _columns(dims, s["zipf"], case["queries"], gen, dev).to(torch.int32)
    return coords, vals, A, B, queries


def prepare(case, seed):
    """The uploaded plan, the parameter set with its C current, and the inputs of the call."""
    s = SHAPES[case["shape"]]
    coords, vals, A, B, queries = _inputs(case, seed, "cuda")
    auto = case["call"] == "autograd"
    plan = ft.Plan(s["dims"], case["J"], case["R"], coords.cpu().numpy(), vals.cpu().numpy(), with_perm=auto,
                   relaxed=case["relaxed"])
    st = {"case": case, "plan": plan, "lr": s["lr"]}
    if auto:
        st["A"] = [a.requires_grad_() for a in A]
        st["B"] = [b.requires_grad_() for b in B]
        st["vals"] = vals
        return st
    st["params"] = ft.Params(A, B, storage=case["storage"])
    ft.refresh(plan, st["params"])
    st["queries"] = queries
    st["loss"] = torch.empty(4, dtype=torch.float64, device="cuda")
    if case["call"] == "epoch":
        st["params"].ensure_scratch(plan.scratch_bytes)
    return st


def run(st):
    case, plan = st["case"], st["plan"]
    if case["call"] == "predict":
        return ft.predict(plan, st["params"], st["queries"])
    if case["call"] == "autograd":
        xhat = ft.reconstruct(plan, st["A"], st["B"], storage=case["storage"])
        loss = 0.5 * (xhat - st["vals"]).square().sum()
        grads = torch.autograd.grad(loss, st["A"] + st["B"])
        return {"xhat": xhat, "grads": list(grads)}
    p, lr = st["params"], st["lr"]
    ft.epoch(plan, p, lr, LAM, lr, LAM)
    ft.loss(plan, p, LAM, LAM, out=st["loss"])
    # the loss terms are FP64 sums over FP32 predictions; a training loop logs them in single precision
    return {"A": p.A, "B": p.B, "C": p.C if case["storage"] == "f32" else p.C16, "loss": st["loss"].float()}


def work(case):
    """Bytes and operations of one pass, each input read once and each output written once per pass of a mode."""
    s = SHAPES[case["shape"]]
    dims, J, R, nnz = s["dims"], case["J"], case["R"], case["nnz"]
    N, sp = len(dims), 4 if case["storage"] == "f32" else 2
    rows = [min(d, nnz) for d in dims]  # rows that elements can touch
    stream = nnz * (4 * (N - 1) + 4)
    if case["call"] == "predict":
        q = case["queries"]
        return {"bytes": q * (4 * N + 4) + sum(min(d, q) * R * sp for d in dims), "flops": q * N * R}
    refresh_b = sum(d * (J + R) * sp for d in dims)
    refresh_f = sum(2.0 * d * J * R for d in dims)
    bytes_, flops = 0.0, 0.0
    for m in range(N):
        others = sum(rows[n] * R * sp for n in range(N) if n != m)
        fibers = min(float(nnz), math.prod(float(dims[n]) for n in range(N) if n != m))
        if case["call"] == "epoch":
            # factor pass: w and g = B w once per fiber, then the dot product and the update per element
            bytes_ += stream + others + 2 * rows[m] * J * 4
            flops += fibers * ((N - 2) * R + 2 * J * R) + nnz * 5.0 * J
            # core pass: w, the residual, the row's sum, one outer product per row
            bytes_ += stream + others + rows[m] * (J + R) * sp
            flops += nnz * ((N - 2) * R + 4.0 * R) + rows[m] * 2.0 * J * R
        else:
            # gradient: delta_x w_x summed per row, then B t per row and A^T t per mode
            bytes_ += stream + others + rows[m] * J * sp + dims[m] * J * 4
            flops += nnz * ((N - 2) * R + 2.0 * R) + rows[m] * 4.0 * J * R
    passes = 2 if case["call"] == "epoch" else 1
    bytes_ += passes * refresh_b + stream + sum(r * R * sp for r in rows)  # refreshes; loss or forward
    flops += passes * refresh_f + nnz * N * R
    return {"bytes": int(bytes_), "flops": int(flops)}


# --------------------------------------------------------------------------- the same in FP64

HEAD, CHUNK = 1024, 512  # relaxed passes: in-place elements and piece length of a long row


def _w(C, coords, m, order):
    w = None
    for n in range(len(C)):
        if n != m:
            r = C[n][coords[n][order]]
            w = r if w is None else w * r
    return w


def _row_order(coords, m, N):
    """Positions sorted by (i_m, i_{m+1}, ..., i_{m-1})."""
    order = torch.arange(coords.shape[1], device=coords.device)
    for k in range(N - 1, -1, -1):
        order = order[coords[(m + k) % N][order].sort(stable=True).indices]
    return order


def _dealt(order, start, length):
    """Rows longer than HEAD in stride order: with Q = ceil(L / HEAD), positions 0, Q, 2Q, ..., 1, 1 + Q, ..."""
    row = torch.repeat_interleave(torch.arange(len(length), device=order.device), length)
    t = torch.arange(order.numel(), device=order.device) - start[row]
    Q = torch.where(length > HEAD, (length + HEAD - 1) // HEAD, torch.ones_like(length))[row]
    p = torch.arange(order.numel(), device=order.device)
    for k in (t // Q, t % Q, row):  # least significant key first
        p = p[k[p].sort(stable=True).indices]
    return order[p]


def _chains(a, g, x, start, length, lr, squares=False):
    """Serial SGD steps on every state a[k] over elements start[k] .. start[k] + length[k] - 1."""
    by = length.sort(descending=True).indices
    s, a = start[by], a[by].clone()
    left = length[by].cpu().numpy()
    gg = torch.zeros(len(a), dtype=a.dtype, device=a.device)
    for t in range(int(left[0]) if len(left) else 0):
        n = int((left > t).sum())
        gt, st = g[s[:n] + t], a[:n]
        e = x[s[:n] + t] - (st * gt).sum(1)
        a[:n] = st * (1 - lr * LAM) + (lr * e)[:, None] * gt
        if squares:
            gg[:n] += gt.square().sum(1)
    out, back = torch.empty_like(a), torch.empty_like(gg)
    out[by], back[by] = a, gg
    return (out, back) if squares else out


def _maps(g, x, start, length, lr):
    """The affine maps (M, v) of the serial steps of every piece: a -> M a + v."""
    J, rho = g.shape[1], 1 - lr * LAM
    by = length.sort(descending=True).indices
    s, left = start[by], length[by].cpu().numpy()
    M = torch.eye(J, dtype=g.dtype, device=g.device).repeat(len(left), 1, 1)
    v = torch.zeros(len(left), J, dtype=g.dtype, device=g.device)
    for t in range(int(left[0]) if len(left) else 0):
        n = int((left > t).sum())
        gt = g[s[:n] + t]
        gM = (gt[:, :, None] * M[:n]).sum(1)
        M[:n] = rho * M[:n] - lr * gt[:, :, None] * gM[:, None, :]
        e = x[s[:n] + t] - (v[:n] * gt).sum(1)
        v[:n] = v[:n] * rho + (lr * e)[:, None] * gt
    back = torch.empty_like(by)
    back[by] = torch.arange(len(by), device=by.device)
    return M[back], v[back]


def _factor_pass(A, B, C, coords, vals, m, lr, relaxed):
    N, rho = len(A), 1 - lr * LAM
    order = _row_order(coords, m, N)
    length = torch.bincount(coords[m], minlength=A[m].shape[0])
    start = length.cumsum(0) - length
    if relaxed:
        order = _dealt(order, start, length)
    g = _w(C, coords, m, order) @ B[m].T
    x = vals[order]
    head = HEAD if relaxed else CHUNK
    A[m] = _chains(A[m], g, x, start, length.clamp(max=head), lr)
    rows = (length > head).nonzero()[:, 0]
    if len(rows) == 0:
        return
    pieces = (length[rows] - head + CHUNK - 1) // CHUNK
    row = torch.repeat_interleave(torch.arange(len(rows), device=rows.device), pieces)
    k = torch.arange(len(row), device=rows.device) - (pieces.cumsum(0) - pieces)[row]
    ps = start[rows][row] + head + k * CHUNK
    end = (start + length)[rows][row]
    pl = torch.minimum(end - ps, torch.full_like(ps, CHUNK))
    if not relaxed:
        M, v = _maps(g, x, ps, pl, lr)
        first = pieces.cumsum(0) - pieces
        by = pieces.sort(descending=True).indices
        a, f, left = A[m][rows[by]], first[by], pieces[by].cpu().numpy()
        for t in range(int(left[0])):
            n = int((left > t).sum())
            a[:n] = (M[f[:n] + t] * a[:n, None, :]).sum(2) + v[f[:n] + t]
        A[m][rows[by]] = a
        return
    # relaxed: every piece runs from the row as its head left it; the increments beyond the decay are
    # weighted by the decay of the later elements and merged under the step guard
    aH = A[m][rows]
    b, gg = _chains(aH[row], g, x, ps, pl, lr, squares=True)
    d = (b - rho ** pl.double()[:, None] * aH[row]) * rho ** (end - ps - pl).double()[:, None]
    total = torch.zeros_like(aH).index_add_(0, row, d)
    G = torch.zeros(len(rows), dtype=aH.dtype, device=aH.device).index_add_(0, row, gg)
    omega = (1.0 / (lr * G)).clamp(max=1.0)
    decay = rho ** (length[rows] - head).double()
    A[m][rows] = aH + omega[:, None] * ((decay - 1.0)[:, None] * aH + total)


def exact(case, seed):
    """What `run` returns, in FP64 from the same inputs (no storage rounding)."""
    s = SHAPES[case["shape"]]
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    coords, vals, A, B, queries = _inputs(case, seed, dev)
    coords, vals = coords.long(), vals.double()
    A, B = [a.double() for a in A], [b.double() for b in B]
    N, lr, nnz = len(A), s["lr"], vals.numel()
    C = [a @ b for a, b in zip(A, B)]
    if case["call"] == "predict":
        return (_w(C, queries.long(), -1, slice(None))).sum(1)
    every = slice(None)
    if case["call"] == "autograd":
        xhat = _w(C, coords, -1, every).sum(1)
        gA, gB = [], []
        for m in range(N):
            t = torch.zeros_like(C[m]).index_add_(0, coords[m], _w(C, coords, m, every) * (xhat - vals)[:, None])
            gA.append(t @ B[m].T)
            gB.append(A[m].T @ t)
        return {"xhat": xhat, "grads": gA + gB}
    for m in range(N):
        _factor_pass(A, B, C, coords, vals, m, lr, case["relaxed"])
        C[m] = A[m] @ B[m]
    for m in range(N):
        w = _w(C, coords, m, every)
        e = vals - (w * C[m][coords[m]]).sum(1)
        t = torch.zeros_like(C[m]).index_add_(0, coords[m], w * e[:, None])
        B[m] = B[m] + lr * (A[m].T @ t / nnz - LAM * B[m])
        C[m] = A[m] @ B[m]
    sse = float((vals - _w(C, coords, -1, every).sum(1)).square().sum())
    reg = [LAM * float(sum(x.square().sum() for x in v)) for v in (A, B)]
    return {"A": A, "B": B, "C": C, "loss": torch.tensor([sse, math.sqrt(sse / nnz)] + reg, dtype=torch.float64)}
