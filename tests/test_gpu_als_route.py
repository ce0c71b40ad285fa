"""CP-ALS multiplies its MTTKRPs by V^+, which carries their last bits into the factors' fifth
digit: its updates keep one summation order (the full LDS stash over windows of 1024 for a mode
with frequent rows, windows of 2048 or 4096 in LDS order otherwise, no copies, no grouping),
whatever the other calls on the tensor take."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2201_12523_amd as blco  # noqa: E402

DEV = torch.device("cuda:0")


def power_law(d, n, s, g):
    w = torch.arange(1, d + 1, dtype=torch.float64, device=DEV).pow(-s).cumsum(0)
    u = torch.rand(n, generator=g, device=DEV, dtype=torch.float64) * w[-1]
    return torch.searchsorted(w, u).clamp_(max=d - 1).to(torch.int32)


def tensor(dims, nnz, skew, seed=1):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    coords = [power_law(d, nnz, s, g) if s else
              torch.randint(0, d, (nnz,), generator=g, device=DEV, dtype=torch.int32)
              for d, s in zip(dims, skew)]
    return coords, torch.rand(nnz, generator=g, device=DEV), g


@pytest.mark.parametrize("R", [10, 16, 40, 64])
@pytest.mark.parametrize("nnz", [30_000, 300_000, 1_000_000, 3_000_000])
def test_als_route(R, nnz):
    dims = (30_011, 12_007, 4_001)
    coords, vals, g = tensor(dims, nnz, (1.1, 1.1, 0))
    t = blco.build_device(coords, vals, dims)
    for m in range(3):
        p = t.plan(m, R, use="als")
        assert p["copies"] == 0 and not p["grouped"] and p["out_stride"] == R
        windows = -(-nnz // p["window"])
        assert p["stash_rows"] > 0 or m == 2 or nnz < 300_000   # 30k: too few to stand out
        if p["stash_rows"]:
            assert p["window"] == 1024
            assert p["workgroups"] == min(windows, 2048)   # 4 rounds of 2 per compute unit
        else:
            assert p["window"] == (4096 if R > 32 else 2048)
            assert p["workgroups"] == windows
    # grouped for an MTTKRP call, as it lies for CP-ALS
    flat = blco.build_device(*tensor((200_003, 100_003, 50_021), 1 << 20, (0, 0, 0))[:2],
                             (200_003, 100_003, 50_021))
    assert flat.plan(0, 64)["grouped"] and not flat.plan(0, 64, use="als")["grouped"]

