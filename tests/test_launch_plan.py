"""How launches are planned (blco_plan), on tensors that stay on the host: no GPU is needed."""
import numpy as np
import pytest

import paper_2201_12523_amd as blco
from oracle import encode

u64 = np.uint64


def host_tensor(dims, nnz=100, seed=0):
    rng = np.random.default_rng(seed)
    coords = [rng.integers(0, d, nnz).astype(np.uint32) for d in dims]
    return blco.build(coords, np.ones(nnz, np.float32), dims, placement="host")


def flushed(first, R, narrow):
    """Elements that flush_row writes for a row whose first element is `first` (an output on a
    64-byte line): with 32-bit indices, lane rl of segment j adds to (first + rl) mod 2^32 less the
    row's distance s from its line, plus 16 j."""
    s, out = first & 15, []
    for j in range(-(-R // 16) + 1):
        for rl in range(16):
            q = rl + 16 * j - s
            if 0 <= q < R:
                at = first + rl
                out.append((at & 0xFFFFFFFF if narrow else at) + 16 * j - s)
    return sorted(out)


# outputs around 2^32 elements: what 32-bit element indices can address
@pytest.mark.parametrize("rows,R", [((1 << 32) // R - d, R) for R in (1, 2, 3, 4, 7, 8, 15, 16, 17, 32)
                                    for d in (0, 1, 2, 16, 40)])
def test_output_index_width(rows, R):
    t = host_tensor((rows, 3, 5))
    p = t.plan(0, R)
    assert p["out_stride"] == R
    if rows * R > (1 << 32) - 16:
        assert p["wide"]
    else:
        assert not p["wide"]
        for row in (rows - 1, rows - 2, rows - 3):
            assert flushed(row * R, R, True) == list(range(row * R, row * R + R))


# padded output rows: their elements fit 32-bit indices, and they take a bounded workspace, however
# many rows and non-zeros there are
@pytest.mark.parametrize("R", [1, 7, 10, 17, 31, 33, 50, 63, 97])
def test_padded_output_is_bounded(R):
    padded = 0
    for rows in (3000, 1 << 20, 8_000_000, 16_777_216, 16_777_217, 140_000_000, 1 << 28):
        t = host_tensor((rows, 3, 5))
        for n in (8 * rows - 1, 8 * rows, 32 * rows):
            p = t.plan(0, R, nnz=n)
            if p["out_stride"] != R:
                padded += 1
                assert p["out_stride"] == -(-R // 16) * 16 and not p["wide"]
                assert rows * p["out_stride"] <= (1 << 32) - 16
                assert p["workspace_bytes"] <= 2 << 30
    assert padded


# a call under a budget: the staging comes first, and the workspace fits what is left (or takes at
# most an eighth), whatever the budget is over what the call cannot do without
@pytest.mark.parametrize("gradient", [0, 1])
@pytest.mark.parametrize("R", [10, 35, 64])
def test_workspace_under_a_budget(R, gradient):
    import ctypes

    dims, nnz = (3000, 2000, 900), 1_500_000
    t = host_tensor(dims, nnz)
    fixed, per = sum(dims) * R * 8, 12 + 4 * gradient

    def plan(extra, lent=1 << 62):
        used, chunk = ctypes.c_size_t(), ctypes.c_int64()
        rc = blco.lib().blco_stream_plan(t.handle, 7, gradient, R, blco.F32, fixed + extra, lent,
                                         ctypes.byref(used), ctypes.byref(chunk))
        return rc, used.value, chunk.value

    whole = -(-nnz // 64) * 64
    rc, most, chunk = plan(1 << 33)
    assert rc == 0 and chunk == whole and most > 0   # padding, or copies of the output
    rc, used, chunk = plan(1 << 33, 1000)
    assert rc == 0 and used <= 1000 and chunk == whole
    assert plan(2 * 64 * per - 1)[0] == -2
    used_some = 0
    for extra in ([2 * n * per for n in (64, 65, 1000, 1 << 17, 1 << 18, 300_000, 700_000, 1_200_000)]
                  + [most + 2 * 64 * per - 1, most + 2 * 64 * per, most + 2 * 64 * per + 1]
                  + [2 * whole * per + d for d in (-1, 0, most - 1, most, most + 1)]):
        if extra < 2 * 64 * per:
            continue
        rc, used, chunk = plan(extra)
        assert rc == 0 and used + 2 * chunk * per <= extra
        alone = max(64, min(extra // 2 // per, whole) // 64 * 64)   # the staging without a workspace
        assert chunk == alone or (used <= extra // 8 and chunk >= alone * 7 // 8 - 64)
        if used:
            # a launch over such a chunk uses it
            assert max(t.plan(m, R, use=u, nnz=chunk)["workspace_bytes"] for m in range(3)
                       for u in ("mttkrp", "residual")[:1 + gradient]) >= used
            used_some += 1
        assert plan(extra, used)[1] == used
    assert used_some


def counted(t, dims, key_bits):
    """Distinct rows per non-zero over the sampled windows, from the exported tensor as the oracle
    decodes it; none below 2^19 non-zeros."""
    keys, _, ids, starts = t.export()
    n = keys.size
    if n < 1 << 19:
        return [(0, 0)] * len(dims)
    coords = encode.decode(keys, ids, starts, encode.layout(dims, key_bits))
    first = [(n // 4096 - 1) * i // 63 * 4096 for i in range(64)]
    return [tuple(sum(np.unique(c[a:a + W]).size for a in first) / (64 * W) for W in (2048, 4096))
            for c in coords]


@pytest.mark.parametrize("dims,nnz,key_bits", [((300, 200, 70), 1, 64), ((300, 200, 70), 524_287, 64),
                                               ((300, 200, 70), 524_288, 64), ((70_000, 20_000), 524_289, 64),
                                               ((3000, 2000, 900, 5), 600_000, 64), ((9000,), 700_001, 64),
                                               ((3000, 2000, 900), 600_000, 31)])
def test_counted_flushes(dims, nnz, key_bits):
    rng = np.random.default_rng(nnz)
    coords = [np.minimum(rng.zipf(1.5, nnz) - 1, d - 1).astype(np.uint32) if m == 0 else
              rng.integers(0, d, nnz).astype(np.uint32) for m, d in enumerate(dims)]
    t = blco.build(coords, np.ones(nnz, np.float32), dims, placement="host", key_bits=key_bits)
    for m, want in enumerate(counted(t, dims, key_bits)):
        assert t.plan(m, 32)["flushes"] == pytest.approx(want, abs=1e-12), m


def test_windows_of_short_launches():
    # no more windows than compute units (256 where there is no device), and three quarters as many
    # of the smallest, whose chains of additions are the longest
    t = host_tensor((20_000, 8000, 600), 1000)
    for R in (8, 16, 32, 64):
        for n, window in ((1, 256), (20_000, 256), (49_152, 256), (49_153, 512), (60_000, 512),
                          (131_072, 512), (131_073, 1024), (262_144, 1024), (262_145, 2048)):
            p = t.plan(0, R, nnz=n)
            assert p["window"] == window and p["workgroups"] == -(-n // window)
