"""CP-ALS in memory of the caller, too little of it, and none: the same fits.

Bound: a fit of fp32 MTTKRP outputs is good to about 1e-4 (stated with blco_cp_als)."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2201_12523_amd as blco  # noqa: E402

DEV = torch.device("cuda:0")


# ranks around the solve's one wave, four waves and largest workgroup
@pytest.mark.parametrize("R", [1, 8, 9, 16, 17, 32, 33, 64])
@pytest.mark.parametrize("storage", ["fp32", "bf16"])
def test_memory_of_the_caller(R, storage):
    g = torch.Generator(device=DEV)
    g.manual_seed(R)
    dims, nnz = (300, 280, 20), 30_001
    coords = [torch.randint(0, d, (nnz,), generator=g, device=DEV, dtype=torch.int32) for d in dims]
    t = blco.build_device(coords, torch.rand(nnz, generator=g, device=DEV), dims)
    A = [torch.rand(d, R, generator=g, device=DEV) for d in dims]
    dt = blco.BF16 if storage == "bf16" else blco.F32
    L, need = blco.lib(), ctypes.c_size_t()
    assert L.blco_cp_als_size(t.handle, R, dt, ctypes.byref(need)) == 0
    ws = torch.empty(need.value + 256, dtype=torch.uint8, device=DEV)

    def run(wp, wb):
        F = [a.clone() for a in A]
        fits, rep = np.zeros(3), blco._CPALSReport()
        rc = L.blco_cp_als_in(t.handle, (ctypes.c_void_p * 3)(*[f.data_ptr() for f in F]), R,
                              ctypes.byref(blco._CPALSOpts(3, -1e30, dt)), fits.ctypes.data,
                              ctypes.byref(rep), wp, wb, blco._stream())
        return rc, fits

    rc, none = run(None, 0)
    assert rc == 0
    for wp, wb in ((ws.data_ptr(), need.value), (ws.data_ptr(), need.value - 1)):
        rc, fits = run(wp, wb)
        assert rc == 0 and np.abs(fits - none).max() <= 1e-4
    assert run(ws.data_ptr() + 8, need.value)[0] == -1
    F = [a.clone() for a in A]
    fits, _ = blco.cp_als(t, F, max_iters=3, tol=-1e30, storage=storage)
    assert np.abs(np.array(fits) - none).max() <= 1e-4
    assert L.blco_cp_als_size(t.handle, 65, dt, ctypes.byref(need)) == -1
