"""A call that finds no device memory is made again once torch has given its cached blocks back;
one whose budget is too small, or that fails otherwise, is not."""
import ctypes

import numpy as np
import pytest

import paper_2201_12523_amd as blco


@pytest.fixture
def torch_cuda(monkeypatch):
    freed = []
    monkeypatch.setattr(blco.torch.cuda, "is_available", lambda: True)
    monkeypatch.setattr(blco.torch.cuda, "is_current_stream_capturing", lambda: False)
    monkeypatch.setattr(blco.torch.cuda, "empty_cache", lambda: freed.append(1))
    return freed


class Library:
    """A library whose last error is the given text."""

    def __init__(self, text):
        self.text = text

    def blco_last_error(self):
        return self.text


@pytest.mark.parametrize("codes,text,calls,frees", [
    ([0], b"", 1, 0), ([-2, 0], b"device allocation of 5 bytes failed", 2, 1),
    ([-2, -2], b"device allocation of 5 bytes failed", 2, 1),
    ([-2], b"budget 5 cannot hold factors", 1, 0), ([-3], b"k failed", 1, 0)])
def test_with_memory(torch_cuda, monkeypatch, codes, text, calls, frees):
    monkeypatch.setattr(blco, "lib", lambda: Library(text))
    left = list(codes)
    assert blco._with_memory(lambda: left.pop(0)) == codes[-1]
    assert len(codes) - len(left) == calls and len(torch_cuda) == frees


def test_a_small_budget_says_so():
    # the message by which a budget that is too small is told from memory that has run out
    rng = np.random.default_rng(1)
    t = blco.build([rng.integers(0, 9, 50).astype(np.uint32) for _ in range(3)],
                   np.ones(50, np.float32), (9, 9, 9), placement="host")
    used, chunk = ctypes.c_size_t(), ctypes.c_int64()
    assert blco.lib().blco_stream_plan(t.handle, 7, 0, 4, blco.F32, 10, 0, ctypes.byref(used),
                                       ctypes.byref(chunk)) == -2
    assert blco.lib().blco_last_error().startswith(b"budget")


@pytest.mark.gpu
def test_no_memory_is_enomem():
    # more device memory than there is: ENOMEM, and the next call on the device is not told of it
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(2)
    dims = (1 << 32, 5, 4)
    coords = [rng.integers(0, d, 40).astype(np.uint32) for d in dims]
    t = blco.build(coords, np.ones(40, np.float32), dims)
    one = torch.zeros(64, device="cuda:0")    # never read: the memory is asked for first
    fac = (ctypes.c_void_p * 3)(*[one.data_ptr()] * 3)
    for ws in (None, one.data_ptr()):
        rc = blco.lib().blco_cp_als_in(t.handle, fac, 64, None, None, None, ws, 256 if ws else 0,
                                       blco._stream())
        assert rc == -2, blco.lib().blco_last_error()
    small = blco.build([c % 4 for c in coords], np.ones(40, np.float32), (4, 4, 4))
    F = [torch.ones(4, 8, device="cuda:0") for _ in range(3)]
    assert float(blco.mttkrp(small, 0, F)[:, 0].sum()) == 40.0
