"""Host-side checks that need neither a GPU nor the oracle's arithmetic: the benchmark's command
line contract, the seeded input generators, and the product path's refusal to run without its library."""
import json
import os
import subprocess
import sys

import numpy as np

from paper_2410_12707_amd import workloads as wl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_bench_refuses_more_than_one_gpu():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], stdout=subprocess.PIPE,
                       stderr=subprocess.PIPE, text=True, timeout=120)
    assert r.returncode != 0 and "ONE GPU" in r.stderr and r.stdout.strip() == ""


def test_workloads_match_the_benchmark_configurations():
    with open(os.path.join(ROOT, "BASELINE.json")) as f:
        base = json.load(f)
    assert "configs" in base and len(base["configs"]) >= 5
    w1 = wl.config1()
    assert w1.tensors[0].size == 4 * 128 * 768 and w1.ks == [3932] and w1.tensors[0].dtype == np.float32
    assert wl.keep_count(25_165_824, 1, 100) == 251_658 and wl.keep_count(26_214_400, 5, 1000) == 131_072
    s = wl.config_small()
    assert len(s.tensors) == 128 and max(t.size for t in s.tensors) == 8192 and all(k == t.size // 100 for k, t in zip(s.ks, s.tensors))
    r = wl.config_resnet18_samples()
    assert sorted({t.size for t in r.tensors}) == [8192, 16384, 32768, 65536]


def test_generators_are_seeded_and_typed():
    a, b = wl.normal_f32(1000, 5), wl.normal_f32(1000, 5)
    assert np.array_equal(a, b) and not np.array_equal(a, wl.normal_f32(1000, 6))
    h = wl.normal_bf16(1000, 5)
    assert h.dtype == np.uint16
    back = wl.bf16_bits_to_f32(h)
    assert np.all(np.abs(back - a) <= np.abs(a) * 2.0 ** -8)  # round to nearest: half an ulp of 8 significand bits
    assert wl.normal_f16(1000, 5).dtype == np.float16
    for kind in ("normal", "all_equal", "all_zero", "signed_zero_mix", "few_levels", "sparse", "nonfinite", "random_bits",
                 "descending", "ascending"):
        for dtype, npdt in (("f32", np.float32), ("bf16", np.uint16), ("f16", np.float16)):
            x = wl.small_case(kind, 257, seed=3, dtype=dtype)
            assert x.dtype == npdt and x.size == 257
            assert np.array_equal(x.view(np.uint8), wl.small_case(kind, 257, seed=3, dtype=dtype).view(np.uint8))
    g = wl.gelu_of_normal_f32(100_000, 1)
    assert g.min() > -0.2 and (g < 0).mean() > 0.4  # GELU: negative half squashed into (-0.17, 0)


def test_binding_fails_loudly_without_the_library(tmp_path):
    code = ("import os, sys; sys.path.insert(0, %r); os.environ['ADATOPK_LIBRARY'] = %r\n"
            "from paper_2410_12707_amd import binding as B\n"
            "try:\n    B.load_library()\nexcept Exception as e:\n    print('RAISED', type(e).__name__); sys.exit(0)\n"
            "sys.exit(3)\n") % (ROOT, str(tmp_path / "missing.so"))
    r = subprocess.run([sys.executable, "-c", code], stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True, timeout=120)
    assert r.returncode == 0 and "RAISED" in r.stdout, (r.stdout, r.stderr)


def test_marshalling_of_segmented_arguments():
    # what the extension packs is what ctypes would have packed; anything but the plain case is left to Python
    import ctypes

    import torch

    from paper_2410_12707_amd import binding as B

    m = B._load_marshal()
    for values in ([], [0], [1, 2, 3], [2**62, -5], list(range(129))):
        for seq in (values, tuple(values)):
            packed, total = m.int64s(seq, len(values))
            assert packed == bytes((ctypes.c_int64 * len(values))(*values)) and total == sum(values)
    for odd in ([1, 2.0], [True], ["1"], [2**63], [2**62, 2**62], range(2), "12", None):
        assert m.int64s(odd, 2 if odd is None else len(odd)) is None
    assert m.int64s([1, 2], 3) is None and m.int64s([1, 2], 1) is None
    kk, total = B._counts([1, 2.9], 2)  # as int() takes them
    assert list(kk) == [1, 2] and total == 3
    for odd in ([], [torch.zeros(3)], [torch.zeros(3), 1], [torch.nn.Parameter(torch.zeros(2))], torch.zeros(2), None, (x for x in ())):
        assert m.tensors(odd) is None  # host memory, nothing at all, not a tensor, not a list


def test_segmented_arguments_without_the_extension():
    # a package of which only the library was built, or one built for another Python: the same arrays, read in Python
    code = ("import sys, warnings; sys.path.insert(0, %r); sys.modules['paper_2410_12707_amd._marshal'] = None\n"
            "import ctypes, torch\n"
            "from paper_2410_12707_amd import binding as B\n"
            "with warnings.catch_warnings(record=True) as seen:\n"
            "    warnings.simplefilter('always')\n"
            "    assert B._segments([torch.zeros(3)]) is None and B._segments([]) is None\n"
            "    kk, total = B._counts([1, 2, 3], 3)\n"
            "assert bytes(kk) == bytes((ctypes.c_int64 * 3)(1, 2, 3)) and total == 6\n"
            "assert len(seen) == 1 and issubclass(seen[0].category, RuntimeWarning)\n"
            "try:\n    B.adatopk_compress_segmented([torch.zeros(3)], [1], torch.zeros(1, dtype=torch.int32), torch.zeros(1), [0, 1], None, torch.zeros(1))\n"
            "except ValueError as e:\n    assert 'device' in str(e); print('REFUSED')\n") % ROOT
    r = subprocess.run([sys.executable, "-c", code], stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True, timeout=120)
    assert r.returncode == 0 and "REFUSED" in r.stdout, (r.stdout, r.stderr)


def test_extension_is_built_for_this_python_and_rebuilt_after_a_change(tmp_path, monkeypatch):
    import sysconfig

    from paper_2410_12707_amd import build as b

    assert b.MARSHAL_LIB.endswith(sysconfig.get_config_var("EXT_SUFFIX"))
    source, lib = tmp_path / "marshal.cpp", tmp_path / "_marshal.so"
    source.write_text("")
    monkeypatch.setattr(b, "MARSHAL_SOURCE", str(source))
    monkeypatch.setattr(b, "MARSHAL_LIB", str(lib))
    assert b.marshal_is_stale()
    lib.write_text("")
    os.utime(source, (1, 1))
    assert not b.marshal_is_stale()
    os.utime(lib, (0, 0))
    assert b.marshal_is_stale()


def test_bench_counts_the_judging_kernels_reads_of_the_input():
    import bench

    lo = 0x3F800000
    assert bench.judge_reads([lo, 3, 0, 0, 0, 0, 1, 0], lo - 1) == 0   # the window held
    assert bench.judge_reads([lo, 3, 0, 0, 0, 0, 0, 0], lo - 1) == 2   # the k-th key below it: two passes over the input
    assert bench.judge_reads([lo, 3, 0, 0, 0, 0, 0, 0], lo + (2048 << 3)) == 0  # above it: passes over the candidates
    hit = {"k_scan_spec": 24.0, "k_judge": 6.2, "k_emit": 5.7, "k_merge": 18.0}
    assert bench.input_passes(hit, 100_663_296, 0) == 1
    assert bench.input_passes(dict(hit, k_judge=57.0), 100_663_296, 2) == 3
    assert bench.input_passes({"k_hist1": 17.0, "k_scan": 24.0, "k_refine": 6.0}, 100_663_296, 0) == 2
    assert bench.input_passes({"k_scan_spec": 24.0, "k_hist1": 3.9, "k_scan": 4.0}, 100_663_296, 0) == 1  # returned at once


def test_extension_is_rebuilt_after_a_change_of_the_header(tmp_path, monkeypatch):
    from paper_2410_12707_amd import build as b

    paths = [tmp_path / name for name in ("marshal.cpp", "adatopk.h", "_marshal.so")]
    for path, attribute, time in zip(paths, ("MARSHAL_SOURCE", "HEADER", "MARSHAL_LIB"), (1, 1, 2)):
        path.write_text("")
        os.utime(path, (time, time))
        monkeypatch.setattr(b, attribute, str(path), raising=False)
    assert not b.marshal_is_stale()
    os.utime(paths[1], (3, 3))
    assert b.marshal_is_stale()


def test_bench_counts_what_is_placed_from_the_input():
    import bench

    m = 1 << 20
    ns, ks = [8 * m, 8 * m, 8 * m, 8 * m, m - 1, 2 * m], [m // 8, 2 * m, 4 * m, 8 * m, m // 2, 2 * m - 1]
    assert bench.placed_from_input(ns, ks, 4) == (16 * m, 6 * m)  # not: listed, kept whole, short, all but one kept
    assert bench.placed_from_input(ns, ks, 2) == (8 * m, 4 * m)   # 16-bit types list a quarter
    batch = {"k_scan_spec": 161.0, "k_hist1": 8.0, "k_scan": 8.0, "k_refine": 23.0, "k_emit": 9.0, "k_place_dense": 76.0}
    assert bench.input_passes(batch, 805_306_368, 0, 0.25) == 1.25
    assert bench.input_passes({k: v for k, v in batch.items() if k != "k_place_dense"}, 805_306_368, 0, 0.25) == 1
