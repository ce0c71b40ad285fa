"""Tensors streamed in turn on one stream do not share the host link: a call's copies follow the
copies of the call before it, but for the last 64 MiB.  On streams of their own, and from threads,
nothing changes."""
import threading

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2201_12523_amd as blco  # noqa: E402

DEV = torch.device("cuda:0")


def tensor(dims, nnz, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    coords = [torch.randint(0, d, (nnz,), generator=g, device=DEV, dtype=torch.int32) for d in dims]
    return blco.build_device(coords, torch.rand(nnz, generator=g, device=DEV), dims,
                             placement="pinned")


def test_copies_in_turn():
    # more to copy than the lead (64 MiB): the values of the last chunk go in two pieces, in one
    # chunk and in several; tensors in turn on one stream, results as in memory
    dims = (1 << 18, 1 << 17, 1 << 16)
    F = [torch.rand(d, 16, device=DEV) for d in dims]
    for nnz in (22_000_001, 6_000_000):
        ts = [tensor(dims, nnz, s) for s in (1, 2, 3)]
        want = [blco.mttkrp_stream_all(t, F) for t in ts]
        torch.cuda.synchronize()
        fixed = ts[0].info()["device_bytes"] + 2 * 4 * 16 * sum(dims)
        for budget in (8_000_000_000, fixed + 2 * 12 * 19_000_000, fixed + 2 * 12 * 2_500_000):
            got = [blco.mttkrp_stream_all(ts[k % 3], F, device_budget=budget) for k in range(6)]
            torch.cuda.synchronize()
            for k in range(6):
                for x, y in zip(got[k], want[k % 3]):
                    assert float(((x - y).abs() - 2.1e-5 * y).max()) <= 0


def test_streams_and_threads():
    dims = (3000, 2000, 900)
    F = [torch.rand(d, 16, device=DEV) for d in dims]
    ts = [tensor(dims, 300_000, s) for s in range(20)]
    want = [blco.mttkrp_stream_all(t, F, device_budget=1 << 30) for t in ts]
    torch.cuda.synchronize()
    # more streams than the library keeps the last copies of, twice each, in turn
    streams = [torch.cuda.Stream() for _ in ts]
    got = []
    for _ in range(2):
        got = [blco.mttkrp_stream_all(t, F, device_budget=1 << 30, stream=s)
               for t, s in zip(ts, streams)]
    torch.cuda.synchronize()
    res = [None] * 4

    def work(k):
        s = streams[k // 2]            # two threads to a stream
        with torch.cuda.stream(s):
            for t in ts[k::4]:
                res[k] = blco.mttkrp_stream_all(t, F, device_budget=1 << 30)
        s.synchronize()

    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for x in threads:
        x.start()
    for x in threads:
        x.join()
    last = [want[k::4][-1] for k in range(4)]
    for a, b in list(zip(got, want)) + list(zip(res, last)):
        for x, y in zip(a, b):
            assert float(((x - y).abs() - 2.1e-5 * y).max()) <= 0
    del ts, streams
