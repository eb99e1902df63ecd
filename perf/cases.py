"""The work whose speed counts: W4A16 multiplies as a decode server and a prompt pass make them, and the offline
preparation of the weights, each through the package's binding.

Four phases:
  call     one multiply, called from Python;
  step     the same projection of several layers of a network, one after the other, each on its own activations: what
           one decode step (M rows = one token of each of M sequences) asks of these weights.  A serving program
           records its step once as a HIP graph and replays it; the weights of all layers together exceed the last-level
           cache, so every layer finds its own cold, as it does in a network;
  prompt   one multiply with as many rows as a prompt or a chunk of prompts has tokens, called from Python;
  prepare  FP16 weights to packed codes, scales and zero points, and back to the FP16 weights these stand for (what an
           offline tool does to look at its own error).
Activations are normal with, on request, one channel in a hundred 20 times larger (the outliers LLM layers show); codes
and zero points are uniform on 0..15 and scales uniform on [0.001, 0.02], as in the package's workloads.
"""
import math

import torch

from paper_2601_16536_amd import binding

DTYPES = {"fp16": torch.float16, "bf16": torch.bfloat16}
CACHE_BYTES = 192 << 20  # the weights of a step's layers take about this much or more


def _multiply(name, phase, M, K, N, group=128, dtype="fp16", symmetric=False, outliers=False):
    case = {"phase": phase, "M": M, "K": K, "N": N, "group": group, "dtype": dtype, "symmetric": symmetric,
            "outliers": outliers, "layers": _layers(K, N) if phase == "step" else 1}
    return dict(case, name=name) if name else case


def _prepare(name, K, N, group=128):
    case = {"phase": "prepare", "K": K, "N": N, "group": group}
    return dict(case, name=name) if name else case


def _layers(K, N):
    """Layers of a step: enough to exceed the last-level cache, at most 24."""
    return max(2, min(24, -(-CACHE_BYTES // (K * N // 2))))


def listed():
    return [
        # the smallest call: one token through one small projection, where latency is all
        _multiply("one_call", "call", 1, 4096, 1024),
        # one sequence, down-projections of a mid-sized layer, activations with outliers
        _multiply("decode_1", "step", 1, 14336, 4096, outliers=True),
        # one sequence, the largest down-projection: the benchmark's headline shape
        _multiply("decode_1_large", "step", 1, 28672, 8192),
        # four sequences, up-projections (K < N), BF16 activations on symmetrically quantized weights
        _multiply("decode_4_bf16", "step", 4, 4096, 11008, dtype="bf16", symmetric=True),
        # a few sequences on the largest weights
        _multiply("decode_8_large", "step", 8, 28672, 8192),
        # the top of the decode range
        _multiply("decode_16", "step", 16, 14336, 4096, outliers=True),
        # a batch size nobody rounded, finer quantization groups
        _multiply("batch_37_group64", "step", 37, 10240, 4608, group=64, symmetric=True),
        # ordinary server batches
        _multiply("batch_64", "step", 64, 8192, 8192),
        _multiply("batch_128_bf16", "step", 128, 8192, 8192, dtype="bf16"),
        # a prompt of odd length through an up-projection
        _multiply("prompt_777_bf16", "prompt", 777, 4096, 11008, dtype="bf16"),
        # a long prompt through a large square projection: the largest call
        _multiply("prompt_2048", "prompt", 2048, 8192, 8192),
        # the offline tool on one layer's weights
        _prepare("prepare_weights", 4096, 11008),
    ]


LARGEST = 2048 * 8192 * 8192  # multiply-adds of the largest listed case
LARGEST_WEIGHTS = 28672 * 8192


def draw(rng):
    def log_uniform(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    phase = rng.choices(("call", "step", "prompt", "prepare"), (1, 6, 3, 1))[0]
    group = rng.choices((128, 64, 32, 256), (7, 2, 1, 1))[0]
    while True:
        K = max(1, round(log_uniform(2048, 28672) / group)) * group
        N = max(1, round(log_uniform(1024, 28672) / 8)) * 8
        if K * N <= LARGEST_WEIGHTS:
            break
    if phase == "prepare":
        return _prepare(None, K, N, group)
    # rows: single tokens are the most common step; the rest spread over the batch sizes
    M = {"call": (1, 128), "step": (1, 128), "prompt": (129, 2048)}[phase]
    M = 1 if phase != "prompt" and rng.random() < 0.2 else log_uniform(*M)
    M = max(1, min(M, LARGEST // (K * N)))
    return _multiply(None, phase, M, K, N, group, rng.choice(("fp16", "fp16", "bf16")), rng.random() < 0.3, rng.random() < 0.3)


def _weights(case, gen):
    """Packed codes, scales and zero points (or None) of one layer, on the GPU."""
    K, N, G = case["K"], case["N"], case["K"] // case["group"]

    def words(*shape):
        return torch.randint(-(1 << 31), 1 << 31, shape, dtype=torch.int32, device="cuda", generator=gen)

    Wp = words(K // 8, N)
    scales = (torch.rand((G, N), device="cuda", generator=gen) * 0.019 + 0.001).to(torch.float16)
    return Wp, scales, None if case["symmetric"] else words(G, N // 8)


def _inputs(case, seed):
    """A list of (X, Wpacked, scales, zeros), one for each layer; or the FP16 weights to be prepared."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    if case["phase"] == "prepare":
        # columns of different spread, as the output channels of a layer have
        W = torch.randn((case["K"], case["N"]), device="cuda", generator=gen)
        return (W * (torch.rand(case["N"], device="cuda", generator=gen) * 0.03 + 0.01)).to(torch.float16)
    layers = []
    for _ in range(case["layers"]):
        X = torch.randn((case["M"], case["K"]), device="cuda", generator=gen)
        if case["outliers"]:
            X[:, torch.randperm(case["K"], device="cuda", generator=gen)[: case["K"] // 100]] *= 20.0
        layers.append((X.to(DTYPES[case["dtype"]]),) + _weights(case, gen))
    return layers


def _gemm(case):
    return binding.gemm_bf16 if case["dtype"] == "bf16" else binding.gemm


def prepare(case, seed):
    state = {"case": case, "inputs": _inputs(case, seed)}
    if case["phase"] == "step":
        gemm, group = _gemm(case), case["group"]
        state["Y"] = [torch.empty((case["M"], case["N"]), dtype=X.dtype, device="cuda") for X, _, _, _ in state["inputs"]]

        def step():
            for (X, Wp, scales, zeros), Y in zip(state["inputs"], state["Y"]):
                gemm(X, Wp, scales, zeros, group, out=Y)

        step()  # outside the capture first: the library may have to allocate
        torch.cuda.synchronize()
        state["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(state["graph"]):
            step()
    return state


def run(state):
    case = state["case"]
    if case["phase"] == "prepare":
        Wp, scales, zeros = binding.quantize(state["inputs"], case["group"])
        return Wp, scales, zeros, binding.dequant(Wp, scales, zeros, case["group"])
    if case["phase"] == "step":
        state["graph"].replay()
        return state["Y"]
    X, Wp, scales, zeros = state["inputs"][0]
    return _gemm(case)(X, Wp, scales, zeros, case["group"])


def work(case):
    K, N, G = case["K"], case["N"], case["K"] // case["group"]
    packed = K * N // 2 + G * N * 2
    if case["phase"] == "prepare":  # read W16, write the packed tensors, and W16 again
        return {"bytes": 2 * (2 * K * N) + packed + G * N // 2, "flops": 0}
    M, layers = case["M"], case["layers"]
    zeros = 0 if case["symmetric"] else G * N // 2
    return {"bytes": layers * (packed + zeros + 2 * M * K + 2 * M * N), "flops": layers * 2 * M * K * N}


def tolerance(case):
    # prepare: codes, scales and the FP16 weights they stand for are all rounded once, from FP32 values fixed by the entry
    # points' documentation.  Multiplies: FP32 sums and one rounding to 16 bits at the end.  Measured against exact():
    # rel 2.1e-4 (FP16) and 1.7e-3 (BF16); the largest difference of two correct results is a unit in the last place
    # (2^-10 and 2^-7 of the value), where a sum lies near a tie.  Four times these.
    if case["phase"] == "prepare":
        return "exact"
    return {"rel": 8e-4, "max": 0.004} if case["dtype"] == "fp16" else {"rel": 6.4e-3, "max": 0.032}


def _dequantized(case, Wp, scales, zeros):
    """The weights of one layer in 64 bits."""
    K, N, group = case["K"], case["N"], case["group"]
    shifts = torch.arange(0, 32, 4, device="cuda", dtype=torch.int32)
    q = ((Wp.unsqueeze(1) >> shifts.view(1, 8, 1)) & 15).reshape(K, N)
    z = 8 if zeros is None else ((zeros.unsqueeze(2) >> shifts.view(1, 1, 8)) & 15).reshape(K // group, 1, N)
    w = (q.view(K // group, group, N) - z).to(torch.float64)
    return (w * scales.to(torch.float64).unsqueeze(1)).view(K, N)


def exact(case, seed):
    inputs = _inputs(case, seed)
    if case["phase"] == "prepare":
        W = inputs.to(torch.float64).view(case["K"] // case["group"], case["group"], case["N"])
        return None, (W.amax(1).clamp(min=0.0) - W.amin(1).clamp(max=0.0)) / 15.0, None, None
    Y = [X.to(torch.float64) @ _dequantized(case, Wp, scales, zeros) for X, Wp, scales, zeros in inputs]
    return Y if case["phase"] == "step" else Y[0]
