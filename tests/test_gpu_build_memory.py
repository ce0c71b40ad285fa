"""blco_build_device_in: the GPU builder in memory the caller provides, against the host
builder, bit for bit (keys, values, blocks), on an MI355X."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2201_12523_amd as blco  # noqa: E402

DEV = torch.device("cuda:0")


@pytest.mark.parametrize("short", [0, 1])
def test_build_in_given_memory(short):
    # storage and workspace of the sizes the library asks for, and blocks with room for only
    # some of the arrays (the rest is allocated); a blocked tensor's run tables and tile
    # table; the storage may be read through the tensor until it is dropped
    rng = np.random.default_rng(11 + short)
    dims = (1000, 300, 77, 6)
    coords = [rng.integers(0, n, size=30_000).astype(np.uint32) for n in dims]
    vals = rng.random(30_000).astype(np.float32)
    L = blco.lib()
    cd = [torch.from_numpy(c.view(np.int32)).to(DEV) for c in coords]
    v = torch.from_numpy(vals).to(DEV)
    d = np.asarray(dims, dtype=np.uint64)
    arr = (ctypes.c_void_p * 4)(*[c.data_ptr() for c in cd])
    for key_bits in (64, 14):
        opts = blco._Opts(key_bits, 1 << 27, 0, 0)
        ns, nw = ctypes.c_size_t(), ctypes.c_size_t()
        assert L.blco_build_device_sizes(4, d.ctypes.data, 30_000, ctypes.byref(opts),
                                         ctypes.byref(ns), ctypes.byref(nw)) == 0
        sizes = (300_000, 500_000) if short else (ns.value, nw.value)
        st, ws = (torch.full((n,), 255, dtype=torch.uint8, device=DEV) for n in sizes)
        h = ctypes.c_void_p()
        assert L.blco_build_device_in(4, d.ctypes.data, 30_000, arr, v.data_ptr(),
                                      ctypes.byref(opts), st.data_ptr(), sizes[0], ws.data_ptr(),
                                      sizes[1], None, ctypes.byref(h)) == 0
        t = blco.BLCOTensor(h.value, dims, st, 0)
        ref = blco.build(coords, vals, dims, key_bits=key_bits)
        for a, b in zip(t.export(), ref.export()):
            assert np.array_equal(a, b)
        F = [torch.rand(n, 16, device=DEV) for n in dims]
        a, b = blco.mttkrp(t, 0, F), blco.mttkrp(ref, 0, F)
        assert float((a - b).abs().max() / b.abs().max()) <= 1e-5
        t.free()
    assert L.blco_build_device_in(4, d.ctypes.data, 30_000, arr, v.data_ptr(), ctypes.byref(opts),
                                  st.data_ptr() + 8, 1000, None, 0, None, ctypes.byref(h)) == -1
