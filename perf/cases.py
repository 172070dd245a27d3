"""What this framework is timed on: tensors on their way over a slow link and back.

A case is a sender and a receiver on one GPU: the sender compresses one tensor, or all tensors of a
pipeline stage in one call, into (index, value) pairs or into wire messages; the receiver turns what
was sent back into dense tensors, or adds it into a gradient.  Sizes, values and keep counts are
those of ``paper_2410_12707_amd/workloads.py`` and of the paper's message (3 x 1024 x 1600 values at
ratio 100), plus ragged ones.

Fields of a case:
  dtype            "f32", "bf16", "f16"
  tensors, n       how many tensors, and the elements of the largest
  sizes            "equal": all have n; "halving": n, n/2, n/4, n/8 and again; "ragged": no two alike
  values           "normal", "gelu" (of a normal), "student3" (1e-3 times Student's t of 3 degrees of
                   freedom), "relu" (of a normal: half of it zeros)
  keep_lo, keep_hi the kept share: spread over the tensors between the two, evenly in its logarithm
  links            the keep counts come from the bandwidth-adaptive rule instead, for links of 8 Mbps to 10 Gbps
  send             "pairs", "wire4", "wire8" (wire messages with 4- or 8-byte indices)
  receive          "sorted" (the pairs as the sender wrote them), "any" (pairs in any order),
                   "dense" (wire messages), "add" (added into a running gradient)
"""
import math

import torch

from paper_2410_12707_amd import binding as B

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
GOLDEN = 0.6180339887498949


def _case(name, dtype, tensors, n, sizes, values, keep_lo, keep_hi, links, send, receive):
    c = dict(dtype=dtype, tensors=tensors, n=n, sizes=sizes, values=values, keep_lo=keep_lo, keep_hi=keep_hi, links=links,
             send=send, receive=receive)
    return dict(c, name=name) if name else c


def listed():
    return [
        # Small models on small inputs: many messages of a few thousand values in one call, where launches and host work count.
        _case("small_messages_128", "f32", 128, 8192, "halving", "normal", 0.01, 0.01, False, "pairs", "sorted"),
        # The per-sample stage outputs of a ResNet-18 on 32 x 32 inputs, 64 samples in one call.
        _case("resnet18_samples_64", "f32", 64, 65536, "halving", "normal", 0.01, 0.01, False, "pairs", "sorted"),
        # A single GPT-2-small hidden activation (4 x 128 x 768): one call's latency.
        _case("gpt2s_hidden_393k", "f32", 1, 393216, "equal", "normal", 0.01, 0.01, False, "pairs", "sorted"),
        # What a GPT-2-XL stage sends per micro-batch of 3 (3 x 1024 x 1600): the paper's message, fp32 values with int64 indices at ratio 100.
        _case("gpt2xl_message_4.9m", "f32", 1, 4915200, "equal", "normal", 0.01, 0.01, False, "wire8", "dense"),
        # A GPT-2-small post-GELU activation (32 x 1024 x 768) at ratio 100 ...
        _case("gpt2s_gelu_25m_1pct", "f32", 1, 25165824, "equal", "gelu", 0.01, 0.01, False, "pairs", "sorted"),
        # ... and at ratio 10, where the pairs themselves weigh.
        _case("gpt2s_gelu_25m_10pct", "f32", 1, 25165824, "equal", "gelu", 0.1, 0.1, False, "pairs", "sorted"),
        # Backward: a heavy-tailed ResNet-101 activation gradient (32 x 256 x 56 x 56), summed into the argument node's gradient.
        _case("resnet101_grad_25m_add", "f32", 1, 25690112, "equal", "student3", 0.01, 0.01, False, "wire4", "add"),
        # All activations of a GPT-2-medium cut, one link and one ratio each, in one call.
        _case("gpt2m_batch_24x8m", "f32", 24, 8388608, "equal", "normal", 0.001, 0.2, False, "pairs", "sorted"),
        # The same with the ratios planned from the links: the fast links' tensors are kept whole or nearly so.
        _case("gpt2m_planned_24x8m", "f32", 24, 8388608, "equal", "normal", 0.0, 0.0, True, "pairs", "sorted"),
        # A GPT-2-XL hidden activation in bf16 (16 x 1024 x 1600): thousands of ties at the threshold.
        _case("gpt2xl_hidden_26m_bf16", "bf16", 1, 26214400, "equal", "normal", 0.005, 0.005, False, "pairs", "sorted"),
        # A ragged fp16 tensor whose receiver does not rely on the order of the pairs.
        _case("ragged_6.5m_f16", "f16", 1, 6543209, "equal", "normal", 0.02, 0.02, False, "pairs", "any"),
        # A stage that feeds several links: unequal ragged bf16 tensors, one wire message for each link.
        _case("ragged_links_12_bf16", "bf16", 12, 1500001, "ragged", "relu", 0.002, 0.05, False, "wire4", "dense"),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    form = rng.choice(["small", "one", "one", "one", "batch", "batch"])
    dtype = rng.choice(["f32", "f32", "bf16", "f16"])
    values = rng.choice(["normal", "gelu", "student3", "relu"])
    keep = _log_uniform(rng, 0.001, 0.2)
    if form == "small":  # many messages of a few thousand values
        n = int(_log_uniform(rng, 512, 8192))
        return _case(None, dtype, rng.randint(8, 128), n, rng.choice(["equal", "halving", "ragged"]), values, keep, keep, False,
                     "pairs", "sorted")
    if form == "one":
        n = int(_log_uniform(rng, 9000, 40e6))
        send, receive = rng.choice([("pairs", "sorted"), ("pairs", "sorted"), ("pairs", "any"), ("pairs", "add"),
                                    ("wire4", "dense"), ("wire8", "dense"), ("wire4", "add")])
        return _case(None, dtype, 1, n, "equal", values, keep, keep, False, send, receive)
    tensors = rng.randint(2, 24)
    n = int(_log_uniform(rng, 20e3, 8e6))
    sizes = rng.choice(["equal", "halving", "ragged"])
    send, receive = rng.choice([("pairs", "sorted"), ("pairs", "sorted"), ("wire4", "dense"), ("wire8", "dense")])
    if rng.random() < 0.3:
        return _case(None, dtype, tensors, n, sizes, values, 0.0, 0.0, True, send, receive)
    return _case(None, dtype, tensors, n, sizes, values, 0.001, max(keep, 0.002), False, send, receive)


def _sizes(case):
    S, n = case["tensors"], case["n"]
    if case["sizes"] == "halving":
        return [max(1, n >> (i % 4)) for i in range(S)]
    if case["sizes"] == "ragged":  # between n and a thirtieth of it, in no order
        return [n if i == 0 else max(1, int(n * 30.0 ** -((i * GOLDEN) % 1.0))) for i in range(S)]
    return [n] * S


def _keep_counts(case, ns):
    S = len(ns)
    if case["links"]:
        # bandwidths and latencies spread between the ends of the paper's testbeds, the longest latency on the slowest link
        u = [(i * GOLDEN) % 1.0 for i in range(S)]
        bandwidth = [1e6 * 1250.0 ** v for v in u]  # bytes per second
        latency = [5e-2 * 2e-3 ** v for v in u]
        return B.adatopk_plan_keep_counts(latency, [1.0 / b for b in bandwidth], ns, list(DTYPES).index(case["dtype"]), 100.0, 3.0)[1]
    lo, hi = case["keep_lo"], case["keep_hi"]
    return [max(1, int(n * lo * (hi / lo) ** ((i * GOLDEN) % 1.0))) for i, n in enumerate(ns)]


def _values(case, n, gen):
    x = torch.randn(n, device="cuda", generator=gen)
    if case["values"] == "gelu":
        x = torch.nn.functional.gelu(x)
    elif case["values"] == "relu":
        x = torch.relu(x)
    elif case["values"] == "student3":
        chi = torch.zeros_like(x)
        for _ in range(3):
            chi.addcmul_(*[torch.randn(n, device="cuda", generator=gen)] * 2)
        x = x.mul_(1e-3).div_(chi.div_(3.0).sqrt_())
    return x.to(DTYPES[case["dtype"]])


def _aligned(n, to):
    return (n + to - 1) // to * to


def prepare(case, seed):
    """The dense tensors, and what a sender and a receiver keep from step to step: buffers and a workspace."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    dtype, ns = DTYPES[case["dtype"]], _sizes(case)
    ks = _keep_counts(case, ns)
    S, esize = len(ns), torch.empty(0, dtype=dtype).element_size()
    state = {"send": case["send"], "receive": case["receive"], "xs": [_values(case, n, gen) for n in ns], "ks": ks,
             "ws": B.new_workspace(sum(ns), S, dtype)}
    if case["receive"] == "add":  # the argument node's gradient so far
        state["ys"] = [_values(case, n, gen) for n in ns]
    else:  # the receiver's tensors, views of one buffer (16-byte aligned starts)
        starts = [0]
        for n in ns:
            starts.append(starts[-1] + _aligned(n, 64))
        flat = torch.zeros(starts[-1], dtype=dtype, device="cuda")
        state["flat"], state["ys"] = flat, [flat[a:a + n] for a, n in zip(starts, ns)]
    if case["send"] == "pairs":
        total = sum(ks)
        state["idx"] = torch.empty(total, dtype=torch.int32, device="cuda")
        state["val"] = torch.empty(total, dtype=dtype, device="cuda")
        state["err"] = torch.empty(S, dtype=torch.float32, device="cuda")
        state["offset"] = [sum(ks[:i]) for i in range(S + 1)]
    else:
        code, ib = list(DTYPES).index(case["dtype"]), int(case["send"][4:])
        state["index_bytes"] = ib
        state["ratios"] = [n / k for n, k in zip(ns, ks)]
        state["lengths"] = [B.adatopk_wire_bytes(k, code, ib) for k in ks]
        at = [0]
        for length in state["lengths"]:
            at.append(_aligned(at[-1] + length, 16))
        state["at"] = at[:-1]
        state["wire"] = torch.zeros(at[-1], dtype=torch.uint8, device="cuda")
        state["messages"] = [state["wire"][a:a + length] for a, length in zip(state["at"], state["lengths"])]
    return state


def run(state):
    """Compress, then what the receiver does with it."""
    xs, ks, ys, ws = state["xs"], state["ks"], state["ys"], state["ws"]
    if state["send"] == "pairs":
        idx, val, err = state["idx"], state["val"], state["err"]
        if len(xs) > 1:
            B.adatopk_compress_segmented(xs, ks, idx, val, state["offset"], err, ws)
            B.adatopk_decompress_segmented(idx, val, state["offset"], ys)
        else:
            B.adatopk_compress(xs[0], ks[0], idx, val, err, ws)
            receiver = {"sorted": B.adatopk_decompress_sorted, "any": B.adatopk_decompress, "add": B.adatopk_decompress_accumulate}
            receiver[state["receive"]](idx, val, ks[0], ys[0])
        sent = {"idx": idx, "val": val, "err": err}
    else:
        wire, messages, ib = state["wire"], state["messages"], state["index_bytes"]
        if len(xs) > 1:
            B.adatopk_compress_wire_segmented(xs, ks, ib, state["ratios"], wire, state["at"], ws)
        else:
            B.adatopk_compress_wire(xs[0], ks[0], ib, state["ratios"][0], wire, ws)
        for message, length, y in zip(messages, state["lengths"], ys):
            B.adatopk_decompress_wire(message, length, ib, y, accumulate=state["receive"] == "add")
        sent = {"wire": wire}
    return dict(sent, dense=state["flat"] if "flat" in state else ys)


def work(case):
    """Each input read once, each output written once; adding touches the kept places of the gradient only."""
    ns = _sizes(case)
    n, k = sum(ns), sum(_keep_counts(case, ns))
    esize = 4 if case["dtype"] == "f32" else 2
    pairs = k * (esize + (8 if case["send"] == "wire8" else 4))
    received = 2 * k * esize if case["receive"] == "add" else n * esize
    return {"bytes": n * esize + 2 * pairs + received, "flops": 2 * n}


def tolerance(case):
    """Pairs and dense tensors are exact.  The error norm is summed in 64 bits and rounded to 32: another order of
    summation gives it or its neighbour, 1.2e-7 away.  In a wire message it is four bytes of the header."""
    if case["send"] == "pairs":
        return {"rel": 5e-7}
    ns = _sizes(case)
    code, ib = list(DTYPES).index(case["dtype"]), int(case["send"][4:])
    return {"rel": 5e-7, "differ": 4 * len(ns) / sum(B.adatopk_wire_bytes(k, code, ib) for k in _keep_counts(case, ns))}
