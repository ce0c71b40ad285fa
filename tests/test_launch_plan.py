"""How launches are planned (blco_plan), on tensors that stay on the host: no GPU is needed."""
import numpy as np
import pytest

import paper_2201_12523_amd as blco

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
