"""Row flushes counted at construction: the device builder's counts are the host builder's, and
grouping follows them, not what the mode lengths suggest."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2201_12523_amd as blco  # noqa: E402

DEV = torch.device("cuda:0")


@pytest.mark.parametrize("dims,nnz,key_bits", [((300, 200, 70), 1, 64), ((300, 200, 70), 524_287, 64),
                                               ((300, 200, 70), 524_288, 64),
                                               ((3000, 2000, 900, 5), 600_000, 64),
                                               ((30_011, 12_007, 4_001), 700_001, 30),
                                               ((1 << 24, 1 << 22, 1 << 20, 1 << 10), 800_000, 64)])
def test_counts(dims, nnz, key_bits):
    rng = np.random.default_rng(nnz)
    coords = [np.minimum(rng.zipf(1.3, nnz) - 1, d - 1).astype(np.uint32) if m == 0 else
              rng.integers(0, d, nnz).astype(np.uint32) for m, d in enumerate(dims)]
    vals = np.ones(nnz, np.float32)
    cd = [torch.from_numpy(c.view(np.int32)).to(DEV) for c in coords]
    vd = torch.from_numpy(vals).to(DEV)
    for place in ("device", "pinned"):
        a = blco.build(coords, vals, dims, key_bits=key_bits, placement=place)
        b = blco.build_device(cd, vd, dims, key_bits=key_bits, placement=place)
        for m in range(len(dims)):
            assert a.plan(m, 32)["flushes"] == b.plan(m, 32)["flushes"], m


def test_grouping_follows_the_counts():
    # a uniform long mode beside two power-law ones: the hot cells keep its windows on few rows
    # (0.16 flushes per non-zero where spread-out indices would make 0.5), and moving the
    # non-zeros costs more than it saves at R = 32
    n, dims = 30_000_000, (50_000, 30_000, 20_000)
    g = torch.Generator(device=DEV)
    g.manual_seed(1)
    coords = []
    for d in dims[:2]:
        w = torch.arange(1, d + 1, dtype=torch.float64, device=DEV).pow(-1.1).cumsum(0)
        u = torch.rand(n, generator=g, device=DEV, dtype=torch.float64) * w[-1]
        coords.append(torch.searchsorted(w, u).clamp_(max=d - 1).to(torch.int32))
    u3 = torch.randint(0, dims[2], (n,), generator=g, device=DEV, dtype=torch.int32)
    vals = torch.ones(n, device=DEV)
    t = blco.build_device(coords + [u3], vals, dims)
    p = t.plan(2, 32)
    assert p["flushes"][0] < 0.25 and not p["grouped"]
    assert t.plan(2, 128)["grouped"]
    flat = blco.build_device([torch.randint(0, d, (n,), generator=g, device=DEV, dtype=torch.int32)
                              for d in dims], vals, dims)
    p = flat.plan(2, 32)
    assert p["flushes"][0] > 0.4 and p["grouped"]
