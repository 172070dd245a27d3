"""Messages by the one-launch kernel for up to 64 K elements and by the placing kernel of dense batches, byte for byte against the oracle's packing: both index
widths, odd keep counts (the padding), several tensors in one buffer with gaps that stay as they are."""
import struct

import numpy as np
import pytest
import torch

import gpu_harness as H
from oracle import adatopk_oracle as orc
from oracle import wire_format as wf
from paper_2410_12707_amd import binding as B
from paper_2410_12707_amd import workloads as wl

pytestmark = pytest.mark.gpu
GAP = 48


def check(got, x, k, ratio, ib, what):
    ri, rv, re = orc.compress(x, k)
    ref = wf.pack(ri, rv, x.size, float(re), ratio, ib)
    assert got[:12] == ref[:12] and got[16:] == ref[16:], what
    assert H.same_err(struct.unpack("<f", got[12:16])[0], re), what


def messages(xs, ks, ib, kernel, offset_elems=0):
    """One call for all tensors; `kernel` has to be one of those it launched."""
    ds = [H.to_device(x, offset_elems) for x in xs]
    ratios = [10.0 + s for s in range(len(xs))]
    sizes = [wf.message_bytes(k, x.dtype, ib) for x, k in zip(xs, ks)]
    at = np.concatenate([[0], np.cumsum([(b + 15) // 16 * 16 + GAP for b in sizes])]).tolist()
    buf = torch.full((at[-1],), 0xAB, dtype=torch.uint8, device="cuda")
    ws = B.new_workspace(sum(x.size for x in xs), len(xs), ds[0].dtype)
    with B.measuring():
        B.measure_read()
        if len(xs) == 1:
            B.adatopk_compress_wire(ds[0], ks[0], ib, ratios[0], buf[:sizes[0]], ws)
        else:
            B.adatopk_compress_wire_segmented(ds, ks, ib, ratios, buf, at[:-1], ws)
        torch.cuda.synchronize()
        assert dict(zip(B.measure_stage_names(), B.measure_read()))[kernel] > 0, kernel
    raw = buf.cpu().numpy().tobytes()
    for s, (x, k) in enumerate(zip(xs, ks)):
        check(raw[at[s]:at[s] + sizes[s]], x, k, ratios[s], ib, (s, x.size, k))
        assert set(raw[at[s] + sizes[s]:at[s + 1]]) <= {0xAB}, "wrote past message %d" % s


@pytest.mark.parametrize("ib", [4, 8])
@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("offset", [0, 2])  # 16-bit types: a base off the 8-byte grid
def test_one_launch(dtype, ib, offset):
    sizes = {"f32": (8193, 40_001, 56_999), "bf16": (8193, 16_383), "f16": (8195, 16_383)}[dtype]
    for n in sizes:
        for kind, k in (("normal", 0), ("normal", 81), ("descending", n // 100 | 1), ("few_levels", 200), ("all_equal", 33), ("nonfinite", 7), ("sparse", n // 110)):
            messages([wl.small_case(kind, n, seed=n + k, dtype=dtype)], [k], ib, "k_mid", offset)
    several = [16_385, 1, 33_001, 0, 8192, 40_000, 257]
    kinds = ["normal", "normal", "descending", "normal", "all_equal", "random_bits", "sparse"]
    xs = [wl.small_case(kind, max(n, 1), seed=n, dtype=dtype)[:n] for n, kind in zip(several, kinds)]
    for share in (0.003, 0.02):
        messages(xs, [int(n * share) for n in several], ib, "k_mid", offset)
    messages([xs[0]] * 70, [165] * 70, ib, "k_mid", offset)  # more than a megaelement


@pytest.mark.parametrize("ib", [4, 8])
@pytest.mark.parametrize("longest", [4200, 6001, 8192])
def test_small_fp32_tensors_in_one_launch(longest, ib):
    lens = [longest, 1, 255, 0, 4095, longest - 1]
    for kind in ("normal", "descending", "all_equal", "nonfinite"):
        messages([wl.small_case(kind, max(n, 1), seed=longest + i)[:n] for i, n in enumerate(lens)], [n // 500 for n in lens], ib, "k_mid")


@pytest.mark.parametrize("dtype,ib", [("f32", 8), ("f32", 4), ("bf16", 8), ("f16", 8)])
def test_dense_batches(dtype, ib):
    n = {"f32": (15 << 20) // 2 + 3, "bf16": (7 << 20) // 2 + 3, "f16": (7 << 20) // 2 + 3}[dtype]
    kinds = ["normal", "few_levels", "normal", "all_zero"]  # windows that hold, lists that overflow, no window
    xs = [wl.small_case(kind, n, seed=i, dtype=dtype) for i, kind in enumerate(kinds)]
    xs.insert(2, wl.small_case("normal", 9001, seed=9, dtype=dtype))
    messages(xs, [n // 2 + 1, n // 3, 91, int(n * 0.9) | 1, n // 4 + 5], ib, "k_place_dense")
