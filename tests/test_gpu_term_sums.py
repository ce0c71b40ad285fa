"""The workspace's routes against the call without one, by the sums of |terms| of the tensor's own
values, and with factors that are not finite.

Bound: as in test_gpu_workspace.py, 2e-5 * S, with S from the call on the absolute values in BLCO
order (t.export) and absolute factors, good to 1e-5 itself."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2201_12523_amd as blco  # noqa: E402

DEV = torch.device("cuda:0")


def tensor(dims, nnz, seed, skew=0.0, **kw):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    coords = []
    for k, d in enumerate(dims):
        if skew and k < 2:
            w = torch.arange(1, d + 1, dtype=torch.float64, device=DEV).pow(-skew).cumsum(0)
            u = torch.rand(nnz, generator=g, device=DEV, dtype=torch.float64) * w[-1]
            coords.append(torch.searchsorted(w, u).clamp_(max=d - 1).to(torch.int32))
        else:
            coords.append(torch.randint(0, d, (nnz,), generator=g, device=DEV, dtype=torch.int32))
    t = blco.build_device(coords, torch.randn(nnz, generator=g, device=DEV), dims, **kw)
    return t, torch.from_numpy(t.export()[1]).to(DEV), g


def plain(t, mode, F, values):
    R = F[0].shape[1]
    out = torch.empty(t.dims[mode], R, device=DEV)
    fac = (ctypes.c_void_p * len(F))(*[f.data_ptr() for f in F])
    dt = blco.BF16 if F[0].dtype == torch.bfloat16 else blco.F32
    assert blco.lib().blco_mttkrp_v(t.handle, mode, values.data_ptr(), fac, dt, R, None, 1.0,
                                    out.data_ptr(), blco._stream()) == 0
    return out


SHAPES = [((3000, 2000, 900), (1 << 18) + 77, 0.0), ((60_001, 40_000, 30_011), (1 << 20) + 9, 0.0),
          ((1 << 17, 1 << 16, 900), 5_000_000, 1.1), ((900, 700, 30, 600), 1_200_000, 0.0)]


@pytest.mark.parametrize("dims,nnz,skew", SHAPES)
@pytest.mark.parametrize("R", [10, 17, 35, 64, 100])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_sums_of_terms(dims, nnz, skew, R, dtype):
    t, vals, g = tensor(dims, nnz, R, skew)
    F = [torch.randn(d, R, generator=g, device=DEV).to(dtype) for d in dims]
    for m in range(len(dims)):
        S = plain(t, m, [f.abs() for f in F], vals.abs())
        a, b = blco.mttkrp(t, m, F), plain(t, m, F, vals)
        assert float(((a - b).abs() - 2.1e-5 * S).max()) <= 0, m


# an explicit threshold keeps the full LDS stash, beside padded factors and output rows
@pytest.mark.parametrize("R", [10, 17, 35, 50, 100])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_stash_and_padding(R, dtype):
    dims = (3000, 2000, 900)
    t, vals, g = tensor(dims, 400_001, R, 1.1, hot_min_count=50)
    F = [torch.randn(d, R, generator=g, device=DEV).to(dtype) for d in dims]
    name = "bf16" if dtype == torch.bfloat16 else "fp32"
    for m in range(3):
        p = t.plan(m, R, name)
        assert p["stash_rows"] > 0 and p["copies"] == 0 and p["factor_stride"] != R
        S = plain(t, m, [f.abs() for f in F], vals.abs())
        a, b = blco.mttkrp(t, m, F), plain(t, m, F, vals)
        assert float(((a - b).abs() - 2.1e-5 * S).max()) <= 0, m


@pytest.mark.parametrize("dims,nnz,skew", SHAPES)
@pytest.mark.parametrize("R", [10, 35, 100])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_not_finite(dims, nnz, skew, R, dtype):
    # an infinity or a NaN in a factor reaches the rows and ranks it is a term of, and no others:
    # padding multiplies zeros by whatever the values are, in ranks that nobody sees
    t, vals, g = tensor(dims, nnz, R, skew)
    vals = vals.clone()
    vals[5], vals[6] = float("inf"), float("nan")
    F = [torch.randn(d, R, generator=g, device=DEV).to(dtype) for d in dims]
    F[0][3, R - 1], F[1][2, 0], F[2][7, R // 2] = float("inf"), float("nan"), float("-inf")
    for m in range(len(dims)):
        a, b = blco.mttkrp_v(t, m, vals, F), plain(t, m, F, vals)
        assert torch.equal(torch.isnan(a), torch.isnan(b))
        inf = torch.isinf(b)
        assert torch.equal(torch.isinf(a), inf) and torch.equal(a[inf], b[inf])
        ok = torch.isfinite(b)
        assert bool(ok.any()) and not bool(ok.all())
        S = plain(t, m, [f.abs().float().nan_to_num(0, 0, 0).to(dtype) for f in F],
                  vals.abs().nan_to_num(0, 0, 0))
        assert float(((a - b).abs() - 2.1e-5 * S)[ok].max()) <= 0
