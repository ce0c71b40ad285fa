"""GPU parity of the window kernel's sizes, flushes and hot copies against the fp64 oracle.

Bounds: |M_gpu - M| <= 1e-5 * S per entry, S the sum of |terms| (each product has N - 1 fp32
multiplications, and an entry of n terms at most n additions, in any order: 1e-5 is
(N + 160) * 2^-24, and no entry here sums enough terms of one sign for its rounding to
reach it), and zeros exactly where no term lands.  bf16 against the oracle on rounded factors.
"""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import oracle  # noqa: E402
import paper_2201_12523_amd as blco  # noqa: E402

DEV = torch.device("cuda:0")
TOL = 1e-5


def make(dims, nnz, R, seed, dtype="fp32"):
    rng = np.random.default_rng(seed)
    coords = [rng.integers(0, d, size=nnz).astype(np.uint32) for d in dims]
    vals = rng.random(nnz).astype(np.float32)
    A = [rng.standard_normal((d, R)).astype(np.float32) for d in dims]
    F = [torch.from_numpy(a).to(DEV) for a in A]
    if dtype == "bf16":
        F = [blco.cast_bf16(f) for f in F]
        A = [oracle.bf16_round(a) for a in A]
    return coords, vals, A, F


def check(out, M, S, label):
    got = out.cpu().numpy().astype(np.float64)
    zero = S == 0
    assert np.all(got[zero] == 0.0), label
    assert float((np.abs(got - M)[~zero] / S[~zero]).max()) <= TOL, label


# windows of 256, 512, 1024 and 2048 non-zeros are taken up to 256 windows each (one per
# compute unit); part of a window, one window, a window and one, and either side of a change
@pytest.mark.parametrize("nnz", [1, 255, 256, 257, 65535, 65537, 131072, 131073, 262145])
@pytest.mark.parametrize("N,R,dtype", [(1, 16, "fp32"), (2, 33, "fp32"), (3, 8, "bf16"),
                                       (3, 48, "fp32"), (4, 31, "fp32"), (4, 64, "bf16"),
                                       (5, 50, "bf16"), (5, 64, "fp32")])
def test_window_sizes(nnz, N, R, dtype):
    dims = (3001, 300, 280, 270, 260)[:N]
    coords, vals, A, F = make(dims, nnz, R, nnz + 10 * N + R, dtype)
    t = blco.build(coords, vals, dims)
    t.set_resolution("register")
    for n in sorted({0, N - 1}):
        M, S = oracle.mttkrp(coords, vals, A, n)
        check(blco.mttkrp(t, n, F), M, S, f"nnz {nnz} N {N} R {R} {dtype} mode {n}")


# ranks whose rows start inside a 64-byte line, and outputs that do: the flush moves the sums
@pytest.mark.parametrize("R", [1, 7, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64])
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_flush_alignment(R, dtype):
    dims = (400, 300, 290)
    coords, vals, A, F = make(dims, 30_000, R, R, dtype)
    t = blco.build(coords, vals, dims)
    for n in range(3):
        M, S = oracle.mttkrp(coords, vals, A, n)
        for off in (0, 1, 13):
            buf = torch.full((dims[n] * R + 64,), 7.0, device=DEV)
            out = buf[off:off + dims[n] * R].view(dims[n], R)
            blco.mttkrp(t, n, F, out=out)
            check(out, M, S, f"R {R} {dtype} mode {n} offset {off}")
            assert bool((buf[:off] == 7).all()) and bool((buf[off + dims[n] * R:] == 7).all())


# frequent rows flushed to copies (more than 2048 windows), with a workspace and without one
# (the full stash), accumulating, and in the fused CP gradient
@pytest.mark.parametrize("N,R,dtype", [(3, 20, "fp32"), (4, 32, "bf16"), (5, 16, "fp32")])
def test_hot_copies(N, R, dtype):
    dims = (2000, 900, 700, 300, 280)[:N]
    nnz = 2049 * 2048 + 5
    rng = np.random.default_rng(N)
    coords, vals, A, F = make(dims, nnz, R, 100 + N, dtype)
    hot = rng.random(nnz) < 0.5          # half of the non-zeros on 40 rows, unevenly
    coords[0][hot] = (40 * rng.random(int(hot.sum())) ** 3).astype(np.uint32)
    t = blco.build(coords, vals, dims)
    assert t.workspace(0, R, dtype) > 0 and t.workspace(-1, R, dtype) >= t.workspace(0, R, dtype)
    M, S = oracle.mttkrp(coords, vals, A, 0)
    out = blco.mttkrp(t, 0, F)
    check(out, M, S, "copies")
    blco.mttkrp_acc(t, 0, F, out)
    check(out, 2 * M, S * 2, "accumulated")
    plain = torch.empty_like(out)        # no workspace
    fac = (ctypes.c_void_p * N)(*[f.data_ptr() for f in F])
    assert blco.lib().blco_mttkrp(t.handle, 0, fac, blco.BF16 if dtype == "bf16" else blco.F32, R,
                                  plain.data_ptr(), blco._stream()) == 0
    check(plain, M, S, "no workspace")
    # values replaced by the model's residual in the fused walk: gradient of mode 0 against
    # the MTTKRP of the residual it returns
    _, grads, e = blco.cp_grad(t, F)
    want = blco.mttkrp_v(t, 0, e, F, alpha=-1.0).cpu().numpy().astype(np.float64)
    bound = blco.mttkrp_v(t, 0, e.abs(), [f.abs() for f in F]).cpu().numpy().astype(np.float64)
    diff = np.abs(grads[0].cpu().numpy().astype(np.float64) - want)
    assert float((diff - 2 * TOL * bound).max()) <= 0


def test_workspace_errors():
    coords, vals, A, F = make((300, 280, 270), 1000, 16, 1)
    t = blco.build(coords, vals, (300, 280, 270))
    L, out = blco.lib(), torch.empty(300, 16, device=DEV)
    fac = (ctypes.c_void_p * 3)(*[f.data_ptr() for f in F])
    ws = torch.empty(4096, dtype=torch.uint8, device=DEV)
    args = lambda p, b: (t.handle, 0, None, fac, 0, 16, None, 1.0, 0, out.data_ptr(), p, b, None)
    assert L.blco_mttkrp_ws(*args(None, 512)) == -1
    assert L.blco_mttkrp_ws(*args(ws.data_ptr() + 4, 512)) == -1
    n = ctypes.c_size_t(7)
    assert L.blco_workspace(t.handle, 3, 16, 0, ctypes.byref(n)) == -1
    assert L.blco_workspace(t.handle, -1, 16, 0, ctypes.byref(n)) == 0 and n.value == 0
    assert L.blco_mttkrp_ws(*args(ws.data_ptr(), 4096)) == 0
    M, S = oracle.mttkrp(coords, vals, A, 0)
    check(out, M, S, "workspace")


def test_copies_keep_chains_short():
    # a frequent row's copies take at most 512 windows' sums each (the full stash took one per
    # workgroup, 512 to 2048), so that long launches stay as near 64 bits as with the stash
    g = torch.Generator(device=DEV)
    g.manual_seed(3)
    dims, nnz = (1 << 18, 1 << 17, 1 << 16), 6_000_000
    coords = []
    for d in dims:
        w = torch.arange(1, d + 1, dtype=torch.float64, device=DEV).pow(-1.1).cumsum(0)
        u = torch.rand(nnz, generator=g, device=DEV, dtype=torch.float64) * w[-1]
        coords.append(torch.searchsorted(w, u).clamp_(max=d - 1).to(torch.int32))
    t = blco.build_device(coords, torch.ones(nnz, device=DEV), dims)
    for m in range(3):
        for n in (5_000_000, 6_000_000, 16_000_000, 60_000_000, 200_000_000):
            p = t.plan(m, 32, nnz=n)
            windows = -(-n // p["window"])
            assert p["copies"] and (p["copies"] * 512 >= windows or p["copies"] == 64)
