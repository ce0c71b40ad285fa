"""Element-wise launches over several arrays: bytes equal to one call per array."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2201_12523_amd as blco  # noqa: E402

DEV = torch.device("cuda:0")


@pytest.mark.parametrize("sizes", [(1,), (0, 257, 3), (5_000_001, 0, 0, 1), (1, 2, 3, 4, 5, 6, 7, 8)])
def test_scale_and_cast(sizes):
    g = torch.Generator(device=DEV)
    g.manual_seed(sum(sizes))
    xs = [torch.randn(n, generator=g, device=DEV) for n in sizes]
    xs[-1].view(-1)[0] = float("nan")
    c = torch.tensor([0.37], dtype=torch.float64, device=DEV)
    cast = blco._cast_all(xs)
    want = [blco.cast_bf16(x) if x.numel() else x.bfloat16() for x in xs]
    assert all(torch.equal(a.view(torch.int16), b.view(torch.int16)) for a, b in zip(cast, want))
    want = [x * float(torch.tensor(0.37).float()) for x in xs]
    blco._scale_all(xs, c)
    assert all(torch.equal(a.view(torch.int32), b.view(torch.int32)) for a, b in zip(xs, want))


def test_errors():
    L = blco.lib()
    x = torch.zeros(4, device=DEV)
    p, n = (ctypes.c_void_p * 9)(*[x.data_ptr()] * 9), (ctypes.c_int64 * 9)(*[4] * 9)
    assert L.blco_scale_all(9, p, n, None, 1.0, None) == -1
    assert L.blco_scale_all(-1, p, n, None, 1.0, None) == -1
    assert L.blco_scale_all(0, None, None, None, 1.0, None) == 0
    assert L.blco_cast_bf16_all(1, p, (ctypes.c_void_p * 1)(), n, None) == -1
    n[0] = -1
    assert L.blco_scale_all(1, p, n, None, 1.0, None) == -1
