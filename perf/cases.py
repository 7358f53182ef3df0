"""Workloads of the library as a user's program runs them, for timing and comparison.

A case is a dict of plain values:

  kind      "pass"  one all-mode spMTTKRP pass (mttkrp of every mode; with one
                    stored stream each call remaps it into the next mode's order)
            "als"   CP-ALS from given starting factors: `sweeps` sweeps with the fit
            "grad"  loss and gradient of the least-squares CP fit, through autograd
            "load"  a tensor that was not seen before: load with the device planner,
                    one CP-ALS sweep, free
  dims      mode sizes, "1000x800x600"
  nnz, rank
  zipf      exponent of the index distribution per mode (ids shuffled); 0 = uniform
  values    "uniform", "lognormal" or "planted" (a rank-`rank` model plus noise)
  dtype     "f32" or "bf16": how the factors of a pass are stored
  copies    0 = one stream, remapped from mode to mode; 1 = one stream per mode
  sweeps    CP-ALS sweeps ("als")

`listed()` holds the repository's own benchmark tensors and ordinary and small
sizes between them; `draw(rng)` spreads further cases over the same ranges.
"""
from __future__ import annotations

import math

import torch

from paper_2405_08470_amd import spmttkrp as S

RANKS = (8, 16, 32, 64, 128)


def _case(kind, dims, nnz, rank, zipf=0.0, values="uniform", dtype="f32", copies=0, sweeps=1, name=None):
    c = {"kind": kind, "dims": "x".join(str(int(d)) for d in dims), "nnz": int(nnz), "rank": int(rank),
         "zipf": float(zipf), "values": values, "dtype": dtype, "copies": int(copies), "sweeps": int(sweeps)}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest configuration: launches and host calls are what it costs
        _case("pass", (1000, 800, 600), 100_000, 16, name="pass3_1e5_r16"),
        # a whole small decomposition, five sweeps with their fits
        _case("als", (1000, 800, 600), 100_000, 16, sweeps=5, name="als3_1e5_r16"),
        # an ordinary tensor with ragged sizes, one stream per mode, at the smallest rank
        _case("pass", (6211, 1847, 733, 97), 1_250_003, 8, 1.1, copies=1, name="pass4_1e6_r8_copies"),
        # an ordinary skewed tensor at the largest rank
        _case("pass", (20011, 15013, 40009), 4_000_037, 128, 1.1, name="pass3_4e6_r128"),
        # an ordinary decomposition whose dense updates weigh as much as the tensor
        _case("als", (12007, 9001, 5003, 301), 2_000_003, 64, 0.8, name="als4_2e6_r64"),
        # the 3-mode benchmark tensor: one mode's factor is far larger than the caches
        _case("pass", (100_000, 80_000, 2_000_000), 80_000_000, 32, 1.1, name="pass3_8e7_r32"),
        # one CP-ALS sweep at its size: the dense update of two million rows (less
        # skew: a dominant row makes the normal equations too ill-conditioned for
        # two programs' roundings to be compared)
        _case("als", (100_000, 80_000, 2_000_000), 80_000_000, 32, 0.8, name="als3_8e7_r32"),
        # the 5-mode benchmark tensor: small modes, long runs
        _case("pass", (10_000, 10_000, 5_000, 200, 50), 50_000_000, 32, 1.2, "lognormal", name="pass5_5e7_r32"),
        # the 4-mode benchmark tensor, the largest, with FP32 and with BF16 factors
        _case("pass", (50_000, 50_000, 20_000, 1_000), 100_000_000, 64, 1.1, name="pass4_1e8_r64"),
        _case("pass", (50_000, 50_000, 20_000, 1_000), 100_000_000, 64, 1.1, dtype="bf16", name="pass4_1e8_r64_bf16"),
        # the gradient benchmark: forward and adjoint over uniform entries
        _case("grad", (20_000, 20_000, 10_000, 500), 50_000_000, 16, 0.0, "planted", name="grad4_5e7_r16"),
        # a new tensor from host arrays to its first sweep
        _case("load", (10_007, 8_009, 100_003), 10_000_019, 32, 0.8, name="load3_1e7_r32"),
    ]


def draw(rng):
    while True:
        kind = rng.choice(("pass", "pass", "pass", "als", "als", "grad", "load"))
        n = rng.choice((3, 3, 3, 4, 4, 5))
        rank = rng.choice(RANKS if kind == "pass" else RANKS[:4])
        nnz = int(round(10 ** rng.uniform(math.log10(5e4), 7.3 if kind == "load" else 8.0)))
        if n * nnz * rank > 4 * 100_000_000 * 64 // 2:
            continue
        lo = 64 if kind == "als" or kind == "load" else 40
        top = {3: 2e6, 4: 1e5, 5: 2e4}[n]
        dims = [int(round(10 ** rng.uniform(math.log10(lo), math.log10(top)))) for _ in range(n)]
        if math.prod(dims) < 20 * nnz:
            continue
        zipf = rng.choice((0.0, 0.5, 0.7, 0.8) if kind in ("als", "load") else (0.0, 1.05, 1.1, 1.15, 1.2))
        values = "planted" if kind == "grad" else rng.choice(("uniform", "lognormal"))
        dtype = "bf16" if kind == "pass" and rng.random() < 0.3 else "f32"
        copies = 1 if kind != "load" and rng.random() < 0.2 else 0
        return _case(kind, dims, nnz, rank, zipf, values, dtype, copies)


def _dims(case):
    return [int(d) for d in case["dims"].split("x")]


_CHUNK = 1 << 22


def _coordinates(case, g):
    """int32 [N, nnz] on the GPU: uniform, or Zipf over shuffled ids."""
    dims, nnz, s = _dims(case), case["nnz"], case["zipf"]
    idx = torch.empty((len(dims), nnz), dtype=torch.int32, device="cuda")
    for w, size in enumerate(dims):
        if s == 0.0:
            idx[w] = torch.randint(0, size, (nnz,), generator=g, device="cuda", dtype=torch.int32)
            continue
        cdf = torch.cumsum(torch.arange(1, size + 1, dtype=torch.float64, device="cuda") ** (-s), 0)
        cdf = cdf / cdf[-1]
        ids = torch.randperm(size, generator=g, device="cuda").to(torch.int32)
        for a in range(0, nnz, 4 * _CHUNK):
            b = min(nnz, a + 4 * _CHUNK)
            u = torch.rand(b - a, generator=g, device="cuda", dtype=torch.float64)
            idx[w, a:b] = ids[torch.searchsorted(cdf, u, right=True).clamp_(max=size - 1)]
    return idx


def _model(idx, factors, a, b):
    p = factors[0][idx[0, a:b].long()]
    for w in range(1, len(factors)):
        p = p * factors[w][idx[w, a:b].long()]
    return p


def _inputs(case, seed):
    """Coordinates, values and starting factors (FP32), on the GPU."""
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    dims, nnz, R = _dims(case), case["nnz"], case["rank"]
    idx = _coordinates(case, g)

    def randn(*shape):
        return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32)

    if case["values"] == "planted":
        scale = R ** (-1.0 / (2 * len(dims)))
        planted = [randn(d, R) * scale for d in dims]
        val = torch.empty(nnz, dtype=torch.float32, device="cuda")
        for a in range(0, nnz, _CHUNK):
            b = min(nnz, a + _CHUNK)
            val[a:b] = _model(idx, planted, a, b).sum(1)
        val += 0.01 * randn(nnz)
        factors = [p + 0.1 * randn(*p.shape) for p in planted]
    else:
        if case["values"] == "lognormal":
            val = torch.exp(randn(nnz))
        else:
            val = torch.rand(nnz, generator=g, device="cuda", dtype=torch.float32)
        factors = [randn(d, R) for d in dims]
    return idx, val, factors


def prepare(case, seed):
    idx, val, factors = _inputs(case, seed)
    dims, R = _dims(case), case["rank"]
    # the coordinate list as a program holds it, in host memory
    hidx, hval = idx.cpu().numpy(), val.cpu().numpy()
    del idx, val
    st = {"kind": case["kind"], "dims": dims, "copies": case["copies"], "sweeps": case["sweeps"],
          "rank": R}
    if case["kind"] == "load":
        st.update(idx=hidx, val=hval, factors=factors)
        return st
    st["t"] = S.tensor_load_coo(dims, hidx, hval, copies=case["copies"], prep="device")
    if case["kind"] == "pass":
        st["factors"] = [f.to(torch.bfloat16) for f in factors] if case["dtype"] == "bf16" else factors
        st["out"] = [torch.empty((d, R), dtype=torch.float32, device="cuda") for d in dims]
    elif case["kind"] == "grad":
        st["factors"] = [f.requires_grad_(True) for f in factors]
    else:
        st["factors"] = factors
    return st


def _als(st, t):
    factors = [f.clone() for f in st["factors"]]
    lam = torch.empty(st["rank"], dtype=torch.float64, device="cuda")
    fits = [S.cp_als_iter(t, factors, lam) for _ in range(st["sweeps"])]
    return {"factors": factors, "lambda": lam, "fits": fits}


def run(st):
    if st["kind"] == "pass":
        flags = 0 if st["copies"] else S.FUSE_REMAP_NEXT
        for d, out in enumerate(st["out"]):
            S.mttkrp(st["t"], d, st["factors"], out, flags=flags)
        return st["out"]
    if st["kind"] == "als":
        return _als(st, st["t"])
    if st["kind"] == "load":
        t = S.tensor_load_coo(st["dims"], st["idx"], st["val"], prep="device")
        r = _als(st, t)
        t.free()
        return r
    for f in st["factors"]:
        f.grad = None
    loss = S.cp_fit_loss(st["t"], st["factors"])
    loss.backward()
    return {"loss": loss.detach(), "grads": [f.grad for f in st["factors"]]}


def work(case):
    """Each nonzero (4-byte indices and value) and each factor read once per
    mode's product, each result written once; the remap between modes is not
    part of what the result needs."""
    dims, nnz, R = _dims(case), case["nnz"], case["rank"]
    N, rows = len(dims), sum(dims)
    fb = 2 if case["dtype"] == "bf16" else 4
    coo = nnz * 4 * (N + 1)
    one = {"bytes": N * coo + (N - 1) * rows * R * fb + rows * R * 4, "flops": N * nnz * R * (N + 1)}
    if case["kind"] == "pass":
        return one
    if case["kind"] == "grad":
        # the forward pass as well
        return {"bytes": one["bytes"] + coo + rows * R * 4, "flops": one["flops"] + nnz * R * N}
    # the update reads each product and writes each factor; Gram and solve
    sweep = {"bytes": one["bytes"] + 2 * rows * R * 4, "flops": one["flops"] + 4 * rows * R * R}
    s = case["sweeps"] if case["kind"] == "als" else 1
    extra = coo if case["kind"] == "load" else 0
    return {"bytes": s * sweep["bytes"] + extra, "flops": s * sweep["flops"]}


def _fold(rows, p):
    """Sums the terms of one row inside each block of 64 rows of `p` (rows in
    order): prefix sums of the block, read at the ends of each run."""
    n, R = p.shape
    head = torch.arange(n, device="cuda") % 64 == 0
    head[1:] |= rows[1:] != rows[:-1]
    start = torch.nonzero(head).squeeze(1)
    last = torch.cat([start[1:], torch.tensor([n], device="cuda")]) - 1
    c = torch.nn.functional.pad(p, (0, 0, 0, -n % 64)).view(-1, 64, R).cumsum(1).view(-1, R)
    before = torch.where((start % 64 == 0).unsqueeze(1), 0.0, c[(start - 1).clamp_(min=0)])
    return rows[start], c[last] - before


def _exact_mttkrp(idx, val, factors, d):
    """Mode d's product in FP64 (`factors` FP64): the terms ordered by output
    row and folded, so that few of a row are left to add up."""
    R, nnz = factors[0].shape[1], val.numel()
    out = torch.zeros((factors[d].shape[0], R), dtype=torch.float64, device="cuda")
    rows, order = torch.sort(idx[d])
    step = (1 << 27) // R
    for a in range(0, nnz, step):
        b = min(nnz, a + step)
        e = order[a:b]
        p = val[e].double().unsqueeze(1).expand(-1, R)
        for w in range(len(factors)):
            if w != d:
                p = p * factors[w][idx[w, e].long()]
        r = rows[a:b].long()
        for _ in range(4):
            r, p = _fold(r, p)
        out.index_add_(0, r, p)
    return out


def _norm_sq(dims, idx, val):
    """||X||^2 with repeated coordinates summed."""
    key = idx[0].long()
    for w in range(1, len(dims)):
        key = key * dims[w] + idx[w]
    key, order = torch.sort(key)
    run = torch.cumsum(torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda"),
                                  (key[1:] != key[:-1]).long()]), 0)
    s = torch.zeros(int(run[-1]) + 1, dtype=torch.float64, device="cuda").index_add_(0, run, val[order].double())
    return float(s.square().sum())


def exact(case, seed):
    idx, val, factors = _inputs(case, seed)
    dims, N = _dims(case), len(_dims(case))
    if case["kind"] == "pass":
        y = [(f.to(torch.bfloat16) if case["dtype"] == "bf16" else f).double() for f in factors]
        return [_exact_mttkrp(idx, val, y, d) for d in range(N)]
    if case["kind"] == "grad":
        y = [f.double() for f in factors]
        res = torch.empty(val.numel(), dtype=torch.float64, device="cuda")
        for a in range(0, val.numel(), _CHUNK):
            b = min(val.numel(), a + _CHUNK)
            res[a:b] = _model(idx, y, a, b).sum(1) - val[a:b].double()
        return {"loss": 0.5 * res.square().sum(), "grads": [_exact_mttkrp(idx, res, y, d) for d in range(N)]}
    y = [f.double() for f in factors]
    nsq = _norm_sq(dims, idx, val)
    fits = []
    for _ in range(case["sweeps"]):
        for d in range(N):
            m = _exact_mttkrp(idx, val, y, d)
            v = torch.ones((case["rank"], case["rank"]), dtype=torch.float64, device="cuda")
            for w in range(N):
                if w != d:
                    v = v * (y[w].T @ y[w])
            un = torch.linalg.solve(v.cpu(), m.T.cpu()).T.contiguous().cuda()
            lam = un.square().sum(0).sqrt()
            y[d] = torch.where(lam > 0, un / lam, torch.zeros_like(un))
        h = torch.outer(lam, lam)
        for w in range(N):
            h = h * (y[w].T @ y[w])
        res = max(0.0, nsq + float(h.sum()) - 2.0 * float((m * un).sum()))
        fits.append(1.0 - math.sqrt(res) / math.sqrt(nsq))
    return {"factors": y, "lambda": lam, "fits": fits}
