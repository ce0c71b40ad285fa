"""Any object with a `cuda_stream` handle is a stream, in every call that takes one."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2201_12523_amd as blco  # noqa: E402

DEV = torch.device("cuda:0")


class Handle:
    def __init__(self, s):
        self.cuda_stream = s.cuda_stream


@pytest.mark.parametrize("R", [10, 16])
def test_stream_objects(R):
    dims, nnz = (3000, 2000, 900), (1 << 18) + 7
    g = torch.Generator(device=DEV)
    g.manual_seed(R)
    coords = [torch.randint(0, d, (nnz,), generator=g, device=DEV, dtype=torch.int32) for d in dims]
    vals = torch.rand(nnz, generator=g, device=DEV)
    F = [torch.rand(d, R, generator=g, device=DEV) for d in dims]
    want = blco.mttkrp(blco.build_device(coords, vals, dims), 1, F)
    own = torch.cuda.Stream()
    torch.cuda.synchronize()
    for s in (own, Handle(own), torch.cuda.ExternalStream(own.cuda_stream),
              Handle(torch.cuda.default_stream())):
        t = blco.build_device(coords, vals, dims, stream=s)
        p = blco.build_device(coords, vals, dims, placement="pinned", stream=s)
        zero, A = torch.zeros_like(want), [f.clone() for f in F]
        torch.cuda.synchronize()       # made on this stream, used on another
        got = [blco.mttkrp(t, 1, F, stream=s), blco.mttkrp_stream(p, 1, F, stream=s),
               blco.mttkrp_stream_all(p, F, stream=s)[1],
               blco.mttkrp_acc(t, 1, F, zero, stream=s)]
        loss, grads, e = blco.cp_grad(t, F, stream=s)
        blco.cp_als(t, A, max_iters=1, stream=s)
        torch.cuda.synchronize()
        for x in got:
            assert float(((x - want).abs() - 2.1e-5 * want).max()) <= 0
        assert bool(torch.isfinite(loss)) and all(bool(torch.isfinite(x).all()) for x in grads)
        # another stream than the one the tensor's memory was made on
        other = Handle(torch.cuda.Stream())
        x = blco.mttkrp(t, 1, F, stream=other)
        torch.cuda.synchronize()
        assert float(((x - want).abs() - 2.1e-5 * want).max()) <= 0
