"""Performance cases of the BLCO library: the calls a user's program makes, over the range of
sizes they are made at.

Five kinds of work, each through the package's public entry points:

* ``mttkrp``: the MTTKRP of every mode of a tensor in device memory, one call per mode (what
  a CP solver of the user's own spends its time in);
* ``loss``: one training step of the sparse CP loss, forward and backward;
* ``als``: a few iterations of the CP-ALS driver from given initial factors;
* ``stream``: the MTTKRP of every mode of a tensor in pinned host memory, streamed;
* ``construct``: a new batch of coordinates becomes a tensor, and the model is evaluated at it.

A case's numbers: ``dims`` (mode lengths), ``nnz`` (distinct non-zeros), ``dist`` per mode
(``u``: uniform indices; ``z1.2``: power law with that exponent, frequent rows at small
indices as a sorted vocabulary has them; ``s1.2``: the same with the rows in random order),
``rank`` and ``dtype`` (storage of the factors).
"""
import math

import numpy as np
import torch

import paper_2201_12523_amd as blco

DEV = "cuda"


def _case(name, kind, dims, nnz, dist, rank, dtype="fp32", **more):
    return dict(name=name, kind=kind, dims="x".join(map(str, dims)), nnz=nnz, dist=dist, rank=rank,
                dtype=dtype, **more)


def listed():
    return [
        # a small tensor in the inner loop of a solver: launches and latency
        _case("mttkrp_20k", "mttkrp", (1000, 800, 600), 20_000, "u,u,u", 16),
        # a tensor of ordinary size with odd mode lengths, five modes and a rank that fills no
        # power of two, rows in no particular order
        _case("mttkrp_5mode", "mttkrp", (21_007, 9_001, 1_501, 367, 31), 3_000_001,
              "s1.1,s1.1,u,u,u", 35),
        # the 3-mode 50M-non-zero power-law tensor
        _case("mttkrp_zipf3", "mttkrp", (1 << 22, 1 << 21, 1 << 20), 50_000_000,
              "z1.1,z1.1,z1.1", 32),
        # the 4-mode 200M-non-zero tensor with a 76-bit index (blocked keys): the largest
        _case("mttkrp_zipf4", "mttkrp", (1 << 24, 1 << 22, 1 << 20, 1 << 10), 200_000_000,
              "z1.2,z1.2,u,u", 32),
        # its shape at a quarter of the non-zeros, the larger rank and bf16 factors
        _case("mttkrp_zipf4_r64_bf16", "mttkrp", (1 << 24, 1 << 22, 1 << 20, 1 << 10), 50_000_000,
              "z1.2,z1.2,u,u", 64, "bf16"),
        # two long modes and two shorter than the compute-unit count
        _case("mttkrp_short4", "mttkrp", (1 << 21, 1 << 17, 24, 168), 20_000_000,
              "z1.1,z1.1,u,u", 32),
        # a rank over 64, uniform indices (no row repeats much)
        _case("mttkrp_rank100", "mttkrp", (300_007, 200_003, 100_003), 4_000_000, "u,u,u", 100),
        # a training step at full size: loss and the gradient of every factor
        _case("loss_4mode", "loss", (1 << 20, 1 << 18, 1 << 16, 1 << 12), 40_000_000,
              "z1.1,z1.1,z1.1,z1.1", 32),
        # a training step on a small tensor, bf16 storage
        _case("loss_300k_bf16", "loss", (20_011, 5_003, 701), 300_000, "z1.1,z1.1,u", 10, "bf16"),
        # the CP-ALS driver on a tensor of moderate size
        _case("als_1m", "als", (30_011, 12_007, 4_001), 1_000_000, "z1.1,z1.1,u", 16, iters=5),
        # a tensor kept in host memory, streamed through the device
        _case("stream_20m", "stream", (1 << 20, 1 << 19, 1 << 17), 20_000_000, "z1.05,z1.05,z1.05",
              32, budget=8_000_000_000),
        # new data arrive: build the format on the GPU, evaluate the model at the new entries
        _case("construct_20m", "construct", (1 << 22, 1 << 21, 1 << 20), 20_000_000,
              "z1.1,z1.1,z1.1", 16),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["mttkrp"] * 5 + ["loss"] * 2 + ["als", "stream", "construct"])
    N = rng.choice([3, 3, 4, 4, 5])
    top = {"mttkrp": 40_000_000, "loss": 20_000_000, "als": 4_000_000, "stream": 20_000_000,
           "construct": 20_000_000}[kind]
    low = {"mttkrp": 5_000, "loss": 100_000, "als": 20_000, "stream": 500_000,
           "construct": 20_000}[kind]
    nnz = log_int(low, top)
    while True:
        dims = sorted((log_int(20, 1 << 21) for _ in range(N)), reverse=True)
        space = math.prod(dims)
        # a sparse tensor whose longest mode is no longer than its non-zeros
        if space >= 64 * nnz and dims[0] <= max(nnz, 1000) and space < 1 << 63:
            break
    dist = []
    for d in dims:
        skew = "%.2f" % rng.uniform(0.8, 1.2)
        dist.append("u" if d < 1000 else rng.choice(["u", "z" + skew, "s" + skew]))
    # enough cells must stay likely for the non-zeros to be distinct
    if nnz * 256 > space:
        dist = ["u"] * N
    rank = rng.choice([8, 10, 16, 24, 32, 48, 64, log_int(4, 64), log_int(4, 128)])
    if kind == "als":
        rank = min(rank, 64)
    dtype = "fp32" if kind == "als" else rng.choice(["fp32", "bf16"])
    more = {}
    if kind == "als":
        more["iters"] = rng.randint(1, 5)
    if kind == "stream":
        # what the factors and outputs take, and a share of the tensor for staging
        more["budget"] = (sum(dims) * rank * 8 + nnz * rng.choice([4, 8, 30]) + (64 << 20))
    c = _case("", kind, dims, nnz, ",".join(dist), rank, dtype, **more)
    del c["name"]
    return c


# ------------------------------------------------------------------ inputs

def _dims(case):
    return tuple(int(d) for d in case["dims"].split("x"))


def _dists(case):
    return case["dist"].split(",")


def _indices(d, n, dist, g):
    """n indices in [0, d) drawn from a mode's distribution."""
    if dist == "u":
        return torch.randint(0, d, (n,), generator=g, device=DEV)
    # whole-number weights: their running sums do not depend on the order of summation, so
    # a seed always gives the same indices
    w = torch.arange(1, d + 1, dtype=torch.float64, device=DEV).pow_(-float(dist[1:]))
    cdf = w.mul_(2.0 ** 44).round_().long().cumsum(0)
    u = torch.randint(0, int(cdf[-1]), (n,), generator=g, device=DEV)
    i = torch.searchsorted(cdf, u, right=True)
    if dist[0] == "s":
        i = torch.randperm(d, generator=g, device=DEV)[i]
    return i


def _coordinates(case, g):
    """nnz distinct coordinates in random order, one int32 tensor per mode."""
    dims, nnz = _dims(case), int(case["nnz"])
    got, n = None, int(nnz * 1.02) + 1000
    for _ in range(40):
        c = [_indices(d, n, s, g).to(torch.int32) for d, s in zip(dims, _dists(case))]
        if got is not None:
            c = [torch.cat([a, b]) for a, b in zip(got, c)]
        # one number per coordinate (a multiplicative hash where the index exceeds 63 bits)
        key = torch.zeros(c[0].numel(), dtype=torch.int64, device=DEV)
        wide = math.prod(dims) >= 1 << 63
        for x, d in zip(c, dims):
            key.mul_(6364136223846793005 if wide else d).add_(x)
            if wide:
                key.bitwise_xor_(key >> 29)
        s, at = key.sort(stable=True)
        del key
        keep = torch.ones(s.numel(), dtype=torch.bool, device=DEV)
        torch.ne(s[1:], s[:-1], out=keep[1:])
        del s
        at = at[keep]
        del keep
        if at.numel() >= nnz:
            at = at[torch.randperm(at.numel(), generator=g, device=DEV)[:nnz]]
            return [x[at] for x in c]
        got = [x[at] for x in c]
        n = int((nnz - at.numel()) * 2) + 1000
    raise ValueError("too few distinct coordinates: %r" % (case,))


_CHUNK = 1 << 21


def _model(coords, A):
    """sum_r prod_m A^(m)[i_m, r] at every coordinate, in A's type."""
    out = torch.empty(coords[0].numel(), dtype=A[0].dtype, device=DEV)
    for lo in range(0, out.numel(), _CHUNK):
        p = None
        for c, a in zip(coords, A):
            row = a[c[lo:lo + _CHUNK].long()]
            p = row if p is None else p.mul_(row)
        out[lo:lo + _CHUNK] = p.sum(1)
    return out


def _inputs(case, seed):
    """(coordinates, values, fp32 factors) of a case: the same for the same seed."""
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 1000003 + 12523)
    dims, nnz, R = _dims(case), int(case["nnz"]), int(case["rank"])
    coords = _coordinates(case, g)
    if case["kind"] in ("loss", "als", "construct"):
        # a planted rank-8 model plus noise: what a factorisation is run on
        truth = [torch.rand(d, 8, generator=g, device=DEV) for d in dims]
        values = _model(coords, truth)
        values += 0.01 * torch.randn(nnz, generator=g, device=DEV)
    else:
        values = torch.rand(nnz, generator=g, device=DEV)
    if case["kind"] == "als":
        A = [torch.rand(d, R, generator=g, device=DEV) for d in dims]
    else:
        A = [torch.randn(d, R, generator=g, device=DEV) for d in dims]
        if case["kind"] != "mttkrp" and case["kind"] != "stream":
            A = [a.mul_(R ** (-0.5 / len(dims))) for a in A]
    return coords, values, A


def _stored(case, A):
    return [a.to(torch.bfloat16) for a in A] if case["dtype"] == "bf16" else A


def prepare(case, seed):
    kind = case["kind"]
    coords, values, A = _inputs(case, seed)
    s = dict(kind=kind, dims=_dims(case))
    if kind == "construct":
        s.update(coords=coords, values=values, A=_stored(case, A))
        return s
    s["t"] = blco.build_device(coords, values, _dims(case),
                               placement="pinned" if kind == "stream" else "device")
    if kind == "loss":
        s.update(A=[a.requires_grad_() for a in A], storage=case["dtype"])
    elif kind == "als":
        s.update(A=A, iters=int(case["iters"]))
    else:
        s["A"] = _stored(case, A)
        if kind == "stream":
            s["budget"] = int(case["budget"])
    return s


def run(state):
    kind = state["kind"]
    if kind == "construct":
        t = blco.build_device(state["coords"], state["values"], state["dims"])
        loss, residual = blco.sampled_loss(t, state["A"])
        return dict(loss=loss, residual=residual)
    t, A = state["t"], state["A"]
    if kind == "mttkrp":
        return [blco.mttkrp(t, m, A) for m in range(len(A))]
    if kind == "stream":
        return blco.mttkrp_stream_all(t, A, device_budget=state["budget"])
    if kind == "loss":
        loss = blco.CPLoss.apply(t, state["storage"], *A)
        return dict(loss=loss, grads=torch.autograd.grad(loss, A))
    F = [a.clone() for a in A]
    fits, _ = blco.cp_als(t, F, max_iters=state["iters"], tol=-1e30)
    return dict(fits=fits, factors=F)


# ------------------------------------------------------------------ compulsory work

def _distinct(d, n, dist):
    """Expected number of distinct indices among n draws from a mode of length d."""
    if dist == "u":
        return d * -math.expm1(n * math.log1p(-1.0 / d)) if d > 1 else 1.0
    k = np.arange(1, d + 1, dtype=np.float64) ** -float(dist[1:])
    return float(-np.expm1(-n * k / k.sum()).sum())


def work(case):
    dims, n, R = _dims(case), int(case["nnz"]), int(case["rank"])
    N = len(dims)
    es = 2 if case["dtype"] == "bf16" else 4
    rows = [_distinct(d, n, s) * R * es for d, s in zip(dims, _dists(case))]
    # each mode's MTTKRP is a call of its own: the non-zeros and the other modes' touched
    # rows read, the output written
    one = [12 * n + sum(rows) - rows[m] + dims[m] * R * 4 for m in range(N)]
    kind = case["kind"]
    if kind == "mttkrp":
        return dict(bytes=sum(one), flops=N * N * n * R)
    if kind == "stream":   # one call for all modes: the non-zeros cross the link once
        return dict(bytes=12 * n + sum(rows) + 4 * R * sum(dims), flops=N * N * n * R)
    if kind == "loss":     # factors read, gradients written once
        return dict(bytes=12 * n + sum(rows) + 4 * R * sum(dims), flops=4 * N * n * R)
    if kind == "als":      # per update: the MTTKRP, M read and the factor written, its Gram
        it = int(case["iters"])
        return dict(bytes=it * (sum(one) + 2 * 4 * R * sum(dims)),
                    flops=it * (N * N * n * R + 4 * R * R * sum(dims)))
    # construct: coordinates and values read, keys and values written; then the loss
    return dict(bytes=n * (4 * N + 4 + 12) + 12 * n + sum(rows) + 4 * n, flops=N * n * R)


# ------------------------------------------------------------------ 64-bit results

def _order(coords, dims):
    """Permutation that puts the coordinates in ALTO order: index bits dealt round robin over
    the modes from the least significant, equal coordinates in input order."""
    bits = [max(0, (d - 1).bit_length()) for d in dims]
    key = torch.zeros(coords[0].numel(), dtype=torch.int64, device=DEV)
    at = 0
    for j in range(max(bits)):
        for c, b in zip(coords, bits):
            if j < b:
                key |= ((c.long() >> j) & 1) << at
                at += 1
    return key.sort(stable=True)[1] if at <= 63 else None


def _mttkrp64(coords, values, A, mode):
    """Mode-`mode` MTTKRP in 64 bits: the terms in order of their target row, summed by
    differences of running sums (no row is a serial chain of atomic additions)."""
    R = A[0].shape[1]
    rows = coords[mode].long()
    out = torch.zeros(A[mode].shape[0], R, dtype=torch.float64, device=DEV)
    order = rows.sort(stable=True)[1]
    B = 256
    step = max(B, (1 << 26) // R // B * B)
    for lo in range(0, order.numel(), step):
        at = order[lo:lo + step]
        p = values[at].double()[:, None]
        for m, a in enumerate(A):
            if m != mode:
                p = p * a[coords[m][at].long()]
        n = at.numel()
        if n % B:
            p = torch.cat([p, p.new_zeros(B - n % B, p.shape[1])])
        p = p.view(-1, B, p.shape[1]).cumsum(1)
        base = p[:, -1].t().contiguous().cumsum(1).t()
        p[1:] += base[:-1, None]
        p = p.reshape(-1, p.shape[2])[:n]
        r = rows[at]
        end = torch.ones(n, dtype=torch.bool, device=DEV)
        torch.ne(r[1:], r[:-1], out=end[:-1])
        p = p[end]
        p[1:] -= p[:-1].clone()
        out[r[end]] += p
    return out


def exact(case, seed):
    coords, values, A = _inputs(case, seed)
    dims, N, kind = _dims(case), len(_dims(case)), case["kind"]
    A = [a.double() for a in _stored(case, A)]
    if kind in ("mttkrp", "stream"):
        return [_mttkrp64(coords, values, A, m) for m in range(N)]
    if kind == "loss":
        e = values.double() - _model(coords, A)
        return dict(loss=0.5 * e.square().sum(),
                    grads=tuple(-_mttkrp64(coords, e, A, m) for m in range(N)))
    if kind == "construct":
        e = values.double() - _model(coords, A)
        order = _order(coords, dims)
        return dict(loss=0.5 * e.square().sum(), residual=None if order is None else e[order])
    fits, x2 = [], values.double().square().sum()
    for _ in range(int(case["iters"])):
        for n in range(N):
            V = torch.ones(A[0].shape[1], A[0].shape[1], dtype=torch.float64, device=DEV)
            for m in range(N):
                if m != n:
                    V = V * (A[m].t() @ A[m])
            M = _mttkrp64(coords, values, A, n)
            A[n] = M @ torch.linalg.pinv(V, hermitian=True)
        V = torch.ones_like(V)
        for a in A:
            V = V * (a.t() @ a)
        r2 = (x2 - 2 * (M * A[N - 1]).sum() + V.sum()).clamp(min=0)
        fits.append(1 - (r2.sqrt() / x2.sqrt()).item())
    return dict(fits=fits, factors=A)
