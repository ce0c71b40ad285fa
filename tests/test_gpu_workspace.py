"""What a workspace adds to the MTTKRP (padded factors, grouped non-zeros, rank slices, hot
copies) against the same call without one, and against the fp64 oracle.

Bound: both calls sum the same fp32 products, each within 1e-5 of the sum S of |terms| of its
entry (the parity bound), so they differ by at most 2e-5 * S; S comes from the same call on
absolute values, itself good to 1e-5."""
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


def tensors(dims, nnz, seed, **kw):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    coords = [torch.randint(0, d, (nnz,), generator=g, device=DEV, dtype=torch.int32) for d in dims]
    vals = torch.randn(nnz, generator=g, device=DEV)
    return coords, vals, g, blco.build_device(coords, vals, dims, **kw)


def plain(t, mode, F, values=None):
    R = F[0].shape[1]
    out = torch.empty(t.dims[mode], R, device=DEV)
    fac = (ctypes.c_void_p * len(F))(*[f.data_ptr() for f in F])
    dt = blco.BF16 if F[0].dtype == torch.bfloat16 else blco.F32
    if values is None:
        rc = blco.lib().blco_mttkrp(t.handle, mode, fac, dt, R, out.data_ptr(), blco._stream())
    else:
        rc = blco.lib().blco_mttkrp_v(t.handle, mode, values.data_ptr(), fac, dt, R, None, 1.0,
                                      out.data_ptr(), blco._stream())
    assert rc == 0
    return out


def compare(t, vals, F, modes):
    for m in modes:
        a, b = blco.mttkrp(t, m, F), plain(t, m, F)
        S = plain(t, m, [f.abs() for f in F], values=vals.abs().max().expand(vals.numel()).contiguous())
        assert float(((a - b).abs() - 2.1e-5 * S).max()) <= 0, m


# padded factors: 2^18 non-zeros and at least eight per row; odd, even and 16-byte ranks, both
# types, three to six modes, a short mode (hierarchical), blocked keys
@pytest.mark.parametrize("dims,key_bits", [((3000, 2000, 900), 64), ((900, 700, 30, 600), 64),
                                           ((900, 800, 700, 600, 500), 64),
                                           ((400, 300, 280, 270, 260, 9), 64),
                                           ((3000, 2000, 900), 20)])
@pytest.mark.parametrize("R", [1, 10, 17, 35, 50, 63, 97])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_padded_factors(dims, key_bits, R, dtype):
    nnz = (1 << 18) + 77
    coords, vals, g, t = tensors(dims, nnz, R, key_bits=key_bits)
    F = [torch.randn(d, R, generator=g, device=DEV).to(dtype) for d in dims]
    assert t.workspace(0, R, "bf16" if dtype == torch.bfloat16 else "fp32") > 0
    compare(t, vals, F, range(len(dims)))


# grouped non-zeros and rank slices: flat long modes, ranks on both sides of 64, values
# replaced, one mode against the oracle
# (two short modes put more non-zeros of a window on a row: that case stays as it is)
@pytest.mark.parametrize("dims,R,dtype,moved", [
    ((60_001, 40_000, 30_011), 100, torch.float32, True),
    ((60_001, 40_000, 30_011), 129, torch.bfloat16, True),
    ((50_000, 20_011, 300, 40), 64, torch.float32, False),
    ((200_003, 100_000, 4096), 64, torch.float32, True),
    ((50_000, 20_011, 4096, 40), 101, torch.bfloat16, True)])
def test_grouped(dims, R, dtype, moved):
    nnz = (1 << 20) + 12_345
    coords, vals, g, t = tensors(dims, nnz, R)
    F = [torch.randn(d, R, generator=g, device=DEV).to(dtype) for d in dims]
    name = "bf16" if dtype == torch.bfloat16 else "fp32"
    assert (t.workspace(0, R, name) >= 12 * nnz) == moved
    compare(t, vals, F, range(len(dims)))
    keys, v, _, _ = t.export()                       # values in BLCO order, replaced by others
    w = torch.rand(nnz, generator=g, device=DEV)
    a = blco.mttkrp_v(t, 0, w, F)
    S = plain(t, 0, [f.abs() for f in F], values=w)
    assert float(((a - plain(t, 0, F, values=w)).abs() - 2.1e-5 * S).max()) <= 0
    host = [c.cpu().numpy().view(np.uint32) for c in coords]
    M, S = oracle.mttkrp(host, vals.cpu().numpy(), [f.float().cpu().numpy() for f in F], 1)
    got = blco.mttkrp(t, 1, F).cpu().numpy().astype(np.float64)
    assert np.all(got[S == 0] == 0)
    assert float((np.abs(got - M)[S > 0] / S[S > 0]).max()) <= 1e-5


def test_fused_gradient_with_padding():
    dims = (1500, 900, 400)
    coords, vals, g, t = tensors(dims, (1 << 18) + 5, 3)
    for R in (10, 33):
        F = [torch.randn(d, R, generator=g, device=DEV) for d in dims]
        loss, grads, e = blco.cp_grad(t, F)
        want_loss, want_e = blco.sampled_loss(t, F)
        # residuals of at most N R fp32 roundings of sum_r prod |a| either way
        mag = torch.zeros_like(e)
        _, neg = blco.sampled_loss(t, [f.abs() for f in F])
        keys_vals = torch.from_numpy(t.export()[1]).to(DEV)
        mag = keys_vals - neg
        assert float(((e - want_e).abs() - 2 * (3 + R) * 2.0 ** -24 * (mag.abs() + 10)).max()) <= 0
        for m in range(3):
            ref = plain(t, m, F, values=-e)
            S = plain(t, m, [f.abs() for f in F], values=e.abs())
            assert float(((grads[m] - ref).abs() - 2.1e-5 * S).max()) <= 0


def test_streams_and_graphs():
    # the workspace follows the call's stream, and a captured call replays on new inputs
    dims = (3000, 2000, 900)
    coords, vals, g, t = tensors(dims, (1 << 18) + 1, 9)
    F = [torch.randn(d, 17, generator=g, device=DEV) for d in dims]
    want = blco.mttkrp(t, 0, F).clone()
    S = plain(t, 0, [f.abs() for f in F], values=vals.abs().max().expand(vals.numel()).contiguous())
    outs = []
    for _ in range(4):
        s = torch.cuda.Stream()
        s.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(s):
            outs.append(blco.mttkrp(t, 0, F))
        outs.append(blco.mttkrp(t, 0, F, stream=s))
    torch.cuda.synchronize()
    for o in outs:
        assert float(((o - want).abs() - 2.1e-5 * S).max()) <= 0
    out = torch.empty_like(want)
    graph = torch.cuda.CUDAGraph()
    blco.mttkrp(t, 0, F, out=out)
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        blco.mttkrp(t, 0, F, out=out)
    for k in range(3):
        F[1].mul_(-1.0)
        want.mul_(-1.0)
        out.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert float(((out - want).abs() - 2.1e-5 * S).max()) <= 0, k


# added to an output, and into one that starts between 16-byte units
@pytest.mark.parametrize("R", [10, 16, 35, 97])
def test_added_and_misaligned_outputs(R):
    dims = (3000, 2000, 900)
    coords, vals, g, t = tensors(dims, (1 << 18) + 3, R)
    F = [torch.randn(d, R, generator=g, device=DEV) for d in dims]
    for m, d in enumerate(dims):
        want = plain(t, m, F)
        S = plain(t, m, [f.abs() for f in F], values=vals.abs().max().expand(vals.numel()).contiguous())
        first = torch.randn(d, R, generator=g, device=DEV)
        # one rounding of the sum either way
        eps = 2.0 ** -23 * (first.abs() + S)
        got = blco.mttkrp_acc(t, m, F, first.clone())
        assert float(((got - (first + want)).abs() - 2.1e-5 * S - eps).max()) <= 0
        for off in (1, 3):
            buf = torch.full((d * R + 8,), 7.0, device=DEV)
            out = buf[off:off + d * R].view(d, R)
            blco.mttkrp(t, m, F, out=out)
            assert float(((out - want).abs() - 2.1e-5 * S).max()) <= 0
            assert bool((buf[:off] == 7).all()) and bool((buf[off + d * R:] == 7).all())
