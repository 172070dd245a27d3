"""What a batch of tensors that keep more than a fifth costs where its windows do not hold, and when they do.  Times are the least of several, of one
kernel or call against another."""
import numpy as np
import pytest
import torch

from paper_2410_12707_amd import binding as B

pytestmark = pytest.mark.gpu
TYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}


def normal(n, seed):
    return torch.randn(n, device="cuda", generator=torch.Generator(device="cuda").manual_seed(seed))


class Batch:
    def __init__(self, xs, share):
        self.xs, self.ks = xs, [int(x.numel() * share) for x in xs]
        self.off = np.concatenate([[0], np.cumsum(self.ks)]).tolist()
        self.idx = torch.empty(self.off[-1], dtype=torch.int32, device="cuda")
        self.val = torch.empty(self.off[-1], dtype=xs[0].dtype, device="cuda")
        self.err = torch.empty(len(xs), device="cuda")
        self.ws = B.new_workspace(sum(x.numel() for x in xs), len(xs), xs[0].dtype)

    def compress(self):
        B.adatopk_compress_segmented(self.xs, self.ks, self.idx, self.val, self.off, self.err, self.ws)

    def stages(self):
        times = {}
        with B.measuring():
            for _ in range(6):
                self.compress()
                torch.cuda.synchronize()
                for name, t in zip(B.measure_stage_names(), B.measure_read()):
                    if t > 0:
                        times[name] = min(t, times.get(name, t))
        return times

    def time(self):
        times = []
        for _ in range(8):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            self.compress()
            end.record()
            end.synchronize()
            times.append(start.elapsed_time(end))
        return min(times[2:])


@pytest.mark.parametrize("dtype,share,dense", [("f32", 0.2, False), ("f32", 0.22, True), ("bf16", 0.22, False), ("f16", 0.25, False), ("bf16", 0.26, True)])
def test_lists_are_for_shares_that_fit_them(dtype, share, dense):
    batch = Batch([normal(8 << 20, i).to(TYPES[dtype]) for i in range(4)], share)
    assert ("k_place_dense" in batch.stages()) == dense


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
def test_a_window_that_misses_costs_little(dtype):
    # behind a ReLU, as many kept as are not zero or a few more or less; tensors off the 16-byte grid take the exact passes at once
    xs = [torch.relu(normal((8 << 20) + 8, i)).to(TYPES[dtype]) for i in range(4)]
    once = Batch([x[2:2 - 8] for x in xs], 0.5).time()
    assert Batch([x[:-8] for x in xs], 0.5).time() < 1.25 * once


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("share", [0.3, 0.5])
def test_windows_hold_where_the_scale_varies(dtype, share):
    n = 8 << 20
    xs = []
    for i in range(4):
        scale = torch.exp(0.5 * normal(n // 1600 + 1, 100 + i)).repeat_interleave(1600)[:n]
        xs.append((normal(n, i) * scale).to(TYPES[dtype]))
    batch = Batch(xs, share)
    batch.compress()
    torch.cuda.synchronize()
    assert batch.ws[:64 * len(xs)].view(torch.int32).cpu()[6::16].tolist() == [1] * len(xs)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_no_scan_for_a_window_that_is_not_worth_it(dtype):
    xs = [normal(8 << 20, i).to(TYPES[dtype]) for i in range(4)]
    scan = Batch(xs, 0.5).stages()["k_scan_spec"]
    for alike in ([torch.relu(x) for x in xs], [torch.ones_like(x) for x in xs], [torch.zeros_like(x) for x in xs]):
        assert Batch(alike, 0.5).stages()["k_scan_spec"] < 0.5 * scan


@pytest.mark.parametrize("value", [0.0, 1.0])
def test_a_batch_of_one_key_has_few_parts_per_chunk(value):
    # without lists the last digit's kernel reads what each of the exact passes has read
    stages = Batch([torch.full((8 << 20,), value, device="cuda") for _ in range(4)], 0.65).stages()
    assert stages["k_refine"] < 0.8 * (stages["k_hist1"] + stages["k_scan"])
