"""Calls that add to one output from several streams at the same time lose nothing, whichever kernel
adds last: the window kernel, the frequent rows' copies, padded rows or copies of the output."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2201_12523_amd as blco  # noqa: E402

DEV = torch.device("cuda:0")


def tensor(dims, nnz, skew, g):
    coords = []
    for d in dims:
        if skew:
            w = torch.arange(1, d + 1, dtype=torch.float64, device=DEV).pow(-skew).cumsum(0)
            u = torch.rand(nnz, generator=g, device=DEV, dtype=torch.float64) * w[-1]
            coords.append(torch.searchsorted(w, u).clamp_(max=d - 1).to(torch.int32))
        else:
            coords.append(torch.randint(0, d, (nnz,), generator=g, device=DEV, dtype=torch.int32))
    return blco.build_device(coords, torch.rand(nnz, generator=g, device=DEV), dims)


@pytest.mark.parametrize("dims,nnz,skew,R,what", [
    ((3000, 2000, 900), (1 << 18) + 3, 0, 10, "padded"),
    ((3000, 2000, 900), 1_500_001, 0, 48, "copies of the output"),
    ((1 << 18, 1 << 17, 1 << 16), 5_000_000, 1.1, 16, "frequent rows"),
    ((1000, 800, 600), 20_000, 0, 16, "plain")])
def test_two_streams(dims, nnz, skew, R, what):
    g = torch.Generator(device=DEV)
    g.manual_seed(R)
    t = tensor(dims, nnz, skew, g)
    F = [torch.rand(d, R, generator=g, device=DEV) for d in dims]
    p = t.plan(0, R)
    assert {"padded": p["out_stride"] != R, "copies of the output": p["out_copies"] > 1,
            "frequent rows": p["copies"] > 0, "plain": True}[what]
    want = blco.mttkrp(t, 0, F).double()
    out = torch.zeros(dims[0], R, device=DEV)
    streams = [torch.cuda.Stream() for _ in range(4)]
    torch.cuda.synchronize()
    k = 0
    for _ in range(6):
        for s in streams:
            blco.mttkrp_acc(t, 0, F, out, stream=s)
            k += 1
    torch.cuda.synchronize()
    # positive terms: each call within 1e-5 of its sum, and a rounding of the total per addition
    assert float(((out.double() - k * want).abs() - (2.1e-5 + k * 2.0 ** -23) * k * want).max()) <= 0
