"""Single tensors below 2^20 elements, whose key window comes from a sample of them: which ones have one, and that it holds for values
that are not alike all over the tensor."""
import numpy as np
import pytest

from oracle import adatopk_oracle as orc
from paper_2410_12707_amd import workloads as wl
from test_gpu_missed_window import Call

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,n", [("f32", 3 << 16), ("f32", 983_039), ("f32", 983_040), ("f32", 1_000_003), ("f32", (1 << 20) - 1),
                                     ("f32", 1 << 20), ("bf16", 1 << 14), ("f16", 1_000_003)])
def test_every_length_from_the_limit_on_speculates(dtype, n):
    x = wl.small_case("normal", n, seed=n % 1000, dtype=dtype)
    c = Call(x, n // 100)
    c.run()
    assert c.held() == 1
    c.check(x)


def holds(xs, k):
    """How many of the calls find their window held; every result is checked."""
    held = 0
    for x in xs:
        c = Call(x, k)
        c.run()
        held += c.held()
        c.check(x)
    return held


@pytest.mark.parametrize("n,keep", [(200_000, 0.01), (393_216, 0.01), (900_001, 0.01), (1_300_000, 0.01)])
def test_windows_hold_where_keys_are_thin(n, keep):
    # 97 % zeros, a third of the others kept: the sample's bracket is wider than a window of fp32 keys can span
    xs = [wl.small_case("sparse", n, seed=500 + i) for i in range(8)]
    assert holds(xs, int(n * keep)) >= 5
