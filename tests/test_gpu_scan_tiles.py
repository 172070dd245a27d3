"""The scan's tiles at their edges: the last tile of a chunk is read through bounds that end with the tensor's last whole dword."""
import numpy as np
import pytest

from gpu_harness import bits, gpu_compress, same_err
from oracle import adatopk_oracle as orc
from paper_2410_12707_amd import workloads as wl

pytestmark = pytest.mark.gpu
TILE = 8192


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("over", [-3, -1, 0, 1, 2, 3, 5, 257, TILE // 2 + 1])
@pytest.mark.parametrize("keep", [0.01, 0.3])  # a window from the sample, and the exact passes
def test_last_tile(dtype, over, keep):
    n = 26 * TILE + over
    for kind, offset in (("normal", 0), ("normal", 1), ("sparse", 0), ("descending", 0), ("all_equal", 0)):
        x = wl.small_case(kind, n, seed=n % 99, dtype=dtype)
        x[-1] = x[int(np.argmax(np.abs(x.astype(np.float64))))] if dtype != "bf16" else x[int(np.argmax(x & 0x7FFF))]  # the last element is kept or ties
        k = int(n * keep)
        idx, val, err = gpu_compress(x, k, offset_elems=offset)
        ri, rv, re = orc.compress(x, k)
        assert np.array_equal(idx, ri), (kind, offset)
        assert np.array_equal(bits(val), bits(rv)), (kind, offset)
        assert same_err(err, re), (kind, offset)
