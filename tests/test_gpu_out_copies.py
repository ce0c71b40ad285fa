"""Copies of the whole output (windows of 2048 at 33-64 ranks on modes every window holds much of),
against the same call without a workspace, which takes windows of 4096.

Bound: both sum the same fp32 products, each within 1e-5 of the sum S of |terms| of its entry (the
parity bound), so they differ by at most 2e-5 * S, and S from the call on absolute values is good to
1e-5 itself."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2201_12523_amd as blco  # noqa: E402

DEV = torch.device("cuda:0")


def plain(t, mode, F, values):
    R = F[0].shape[1]
    out = torch.empty(t.dims[mode], R, device=DEV)
    fac = (ctypes.c_void_p * len(F))(*[f.data_ptr() for f in F])
    dt = blco.BF16 if F[0].dtype == torch.bfloat16 else blco.F32
    assert blco.lib().blco_mttkrp_v(t.handle, mode, values.data_ptr(), fac, dt, R, None, 1.0,
                                    out.data_ptr(), blco._stream()) == 0
    return out


@pytest.mark.parametrize("dims,key_bits", [((3000, 2000, 900), 64), ((3000, 1501, 367, 290), 64),
                                           ((2001, 1501, 367, 301, 290), 64), ((3000, 2000, 900), 25)])
@pytest.mark.parametrize("R", [33, 35, 48, 50, 64])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_out_copies(dims, key_bits, R, dtype):
    nnz = 1_500_001
    g = torch.Generator(device=DEV)
    g.manual_seed(R)
    coords = [torch.randint(0, d, (nnz,), generator=g, device=DEV, dtype=torch.int32) for d in dims]
    t = blco.build_device(coords, torch.randn(nnz, generator=g, device=DEV), dims, key_bits=key_bits)
    vals = torch.from_numpy(t.export()[1]).to(DEV)
    F = [torch.randn(d, R, generator=g, device=DEV).to(dtype) for d in dims]
    name = "bf16" if dtype == torch.bfloat16 else "fp32"
    taken = 0
    for m, d in enumerate(dims):
        p, q = t.plan(m, R, name), t.plan(m, R, name, workspace=0)
        if p["out_copies"] > 1:
            taken += 1
            assert p["window"] == 2048 and p["out_stride"] % 16 == 0 and q["window"] == 4096
            assert 256 * d <= nnz and p["out_copies"] * d * 128 <= nnz
        want = plain(t, m, F, vals)
        S = plain(t, m, [f.abs() for f in F], vals.abs())
        for add in (False, True):
            first = torch.randn(d, R, generator=g, device=DEV)
            got = blco.mttkrp_acc(t, m, F, first.clone()) if add else blco.mttkrp(t, m, F)
            # where it is added to something, one more rounding of the sum
            ref, eps = (first + want, 2.0 ** -23 * (first.abs() + S)) if add else (want, 0)
            assert float(((got - ref).abs() - 2.1e-5 * S - eps).max()) <= 0, (m, add)
        w = torch.rand(nnz, generator=g, device=DEV)
        S = plain(t, m, [f.abs() for f in F], w)
        assert float(((blco.mttkrp_v(t, m, w, F) - plain(t, m, F, w)).abs() - 2.1e-5 * S).max()) <= 0
    assert taken
