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


def uneven(kind, n, seed, dtype):
    """Normal values with a scale per plane or channel, or with rows of zeros."""
    rng = np.random.default_rng(seed)
    x = wl.small_case("normal", n, seed=seed)
    if kind == "planes":  # of 56 x 56 values, one scale each
        x *= np.repeat(np.exp(rng.standard_normal(-(-n // 3136)) * 0.5), 3136)[:n].astype(np.float32)
    elif kind == "channels":  # the innermost dimension
        x *= np.tile(np.exp(rng.standard_normal(768)), -(-n // 768))[:n].astype(np.float32)
    else:
        x *= np.repeat(rng.random(-(-n // 768)) < 0.3, 768)[:n]
    return wl.f32_to_bf16_bits(x) if dtype == "bf16" else x.astype(np.float16) if dtype == "f16" else x


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("kind,keep", [("planes", 0.03), ("channels", 0.01), ("rows", 0.1)])
def test_windows_hold_for_values_that_differ_from_place_to_place(kind, keep, dtype):
    xs = [uneven(kind, n, 600 + i, dtype) for i, n in enumerate((200_000, 245_760, 393_216, 393_217, 602_112, 786_432, 900_001, 1_048_575))]
    assert sum(holds([x], int(x.size * keep)) for x in xs) >= 7


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("n", [200_003, 393_216, 1_000_003, 1_048_575])
@pytest.mark.parametrize("scale", [64.0, 1.0 / 64.0])
def test_misled_samples_of_short_tensors(n, scale, dtype):
    # as for longer ones: what the sample sees is 64 times as large or as small as the rest
    from test_gpu_parity import _sampled_elements

    esize = 4 if dtype == "f32" else 2
    batches = 2 if dtype == "f32" else 1  # what expects enough kept elements at 1 %
    x = wl.small_case("normal", n, seed=n % 1000)
    x[_sampled_elements(n, esize, batches)] *= np.float32(scale)
    x = wl.f32_to_bf16_bits(x) if dtype == "bf16" else x.astype(np.float16) if dtype == "f16" else x
    c = Call(x, n // 100)
    c.run()
    assert c.held() == (1 if dtype == "bf16" and scale < 1.0 else 0)  # (a bf16 window spans 16 binades upwards)
    c.check(x)


@pytest.mark.parametrize("dtype,n", [("f32", 3 << 16), ("f32", (3 << 16) + 255), ("bf16", 1 << 14), ("f16", (1 << 14) + 513), ("bf16", 32_767),
                                     ("f16", 65_537)])
@pytest.mark.parametrize("keep", [0.004, 0.01, 0.05, 0.2])
def test_shortest_speculating_tensors(dtype, n, keep):
    # the sample is as long as the tensor or a good part of it, in all its sizes
    for kind in ("normal", "few_levels", "nonfinite", "descending"):
        x = wl.small_case(kind, n, seed=n % 77, dtype=dtype)
        c = Call(x, int(n * keep))
        c.run()
        c.check(x, (kind, keep))
