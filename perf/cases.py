"""The calls whose speed this repository works on, as a program that uses it makes them.

A case is one linear layer's product Y = W X on a pruned weight (through the C binding, with
buffers that the program keeps, or through ``SparseLinear``, the drop-in module), one decode step
of a whole decoder block (a captured HIP graph of six fused products, as a serving loop replays
it), or the loading of one layer (host encoding, then the dense weight back from the device).
Layer shapes are those of ``workloads`` (13B, 66B and 70B class projections and one GPU's share of
the 70B FFN under 8-way row sharding), the smallest test layer, and a ragged one; tokens go from
one sequence's decode step to a prefill of 1024.

Weights are N(0, 0.02) pruned by magnitude per row, X is N(0, 1), all fp16, drawn on the GPU from
the seed alone.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2607_08786_amd import usp
from paper_2607_08786_amd.linear import SparseLinear

# One product Y = act(W X + bias) + residual: ``api`` "spmm" is the binding of the C entry points
# with Y and the workspace allocated once, "module" is SparseLinear. epilogue: any of "bias",
# "relu" / "gelu_tanh" / "silu", "residual", joined by "+", or "".
_PRODUCT = dict(kind="product", api="spmm", sparsity=50, epilogue="")


def listed():
    return [
        # The smallest layer of the test workloads: launch and host latency.
        dict(_PRODUCT, name="tiny_n16", M=1024, K=1024, N=16),
        # One sequence's decode step on one GPU's share of the 70B FFN (8-way row sharding).
        dict(_PRODUCT, name="ffn70b_shard8_n1", M=3584, K=8192, N=1),
        # An attention projection (q, k, v or o with its bias) in a decode step of 16 sequences.
        dict(_PRODUCT, name="attn13b_n16", M=5120, K=5120, N=16, epilogue="bias"),
        # The FFN's first layer, bias and activation fused, 32 sequences.
        dict(_PRODUCT, name="ffn13b_up_n32", M=13824, K=5120, N=32, epilogue="bias+relu"),
        # The FFN's second layer as a module in a model: bias and residual, 64 sequences.
        dict(_PRODUCT, name="ffn13b_down_n64", M=5120, K=13824, N=64, epilogue="bias+residual", api="module"),
        # The benchmark's layer: 70B-class FFN, 16 sequences.
        dict(_PRODUCT, name="ffn70b_n16", M=28672, K=8192, N=16),
        # The same layer at a large decode batch.
        dict(_PRODUCT, name="ffn70b_n128", M=28672, K=8192, N=128),
        # The largest configured layer at its own sparsity and the largest decode batch.
        dict(_PRODUCT, name="ffn66b_n256", M=36864, K=9216, N=256, sparsity=60),
        # Prefill of 1024 tokens through the module.
        dict(_PRODUCT, name="ffn13b_up_n1024", M=13824, K=5120, N=1024, epilogue="bias+relu", api="module"),
        # Nothing a multiple of anything: odd K (no row of X is 16-byte aligned), odd M, odd N.
        dict(_PRODUCT, name="ragged_n21", M=4999, K=4093, N=21, epilogue="bias"),
        # A decode step of a 13B decoder block: q, k, v, o, FFN up, FFN down in one captured graph.
        dict(kind="block", name="block13b_n16", hidden=5120, ffn=13824, N=16, sparsity=50),
        # Loading one layer: the host encoding (paid once per layer and model load) and the dense
        # weight written back by the on-chip decode.
        dict(kind="load", name="load_attn13b", M=5120, K=5120, sparsity=50),
    ]


_MAX_FLOPS = 2.0 * 36864 * 9216 * 256  # dense-equivalent operations of the largest listed product
_MAX_WEIGHTS = 36864 * 9216
_EPILOGUES = ("", "bias", "bias+relu", "bias+gelu_tanh", "bias+silu", "bias+residual", "residual")


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["product"] * 8 + ["block", "load"])
    if kind == "load":
        return dict(kind="load", M=_log_int(rng, 512, 8192), K=_log_int(rng, 512, 8192),
                    sparsity=rng.choice([40, 50, 60, 70]))
    if kind == "block":
        hidden = 64 * _log_int(rng, 16, 80)
        return dict(kind="block", hidden=hidden, ffn=128 * (_log_int(rng, 2 * hidden, 4 * hidden) // 128),
                    N=_log_int(rng, 1, 64), sparsity=rng.choice([40, 50, 60, 70]))
    # Layer sizes as models have them (multiples of 64), and one time in four any number.
    while True:
        M, K = _log_int(rng, 512, 36864), _log_int(rng, 512, 28672)
        if rng.random() < 0.75:
            M, K = (M + 63) // 64 * 64, (K + 63) // 64 * 64
        N = _log_int(rng, 1, 1024)
        if M * K <= _MAX_WEIGHTS and 2.0 * M * K * N <= _MAX_FLOPS:
            break
    return dict(kind="product", M=M, K=K, N=N, sparsity=rng.choice([40, 50, 60, 70]),
                epilogue=rng.choice(_EPILOGUES), api=rng.choice(["spmm", "spmm", "module"]))


class _Draws:
    """Everything one case draws, in a fixed order from the seed."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(int(seed))

    def normal(self, *shape, scale=1.0):
        return torch.randn(*shape, generator=self.g, device="cuda", dtype=torch.float16).mul_(scale)

    def weight(self, M, K, sparsity):
        """An fp16 weight and its keep-mask: the largest magnitudes of every row."""
        W = self.normal(M, K, scale=0.02)
        prune = max(1, K * sparsity // 100)
        mask = torch.empty((M, K), dtype=torch.bool, device="cuda")
        for r in range(0, M, 4096):
            a = W[r:r + 4096].abs()
            mask[r:r + 4096] = a > a.kthvalue(prune, dim=1, keepdim=True).values
        return W, mask


def _host(W, mask):
    return W.cpu().numpy().view(np.uint16), mask.cpu().numpy().view(np.uint8)


def _parts(case):
    return case["epilogue"].split("+") if case["epilogue"] else []


def _activation(parts):
    return next((p for p in parts if p in usp.ACTIVATIONS), "none")


def _product_inputs(case, seed):
    d, parts = _Draws(seed), _parts(case)
    M, K, N = case["M"], case["K"], case["N"]
    W, mask = d.weight(M, K, case["sparsity"])
    X = d.normal(N, K)
    bias = d.normal(M) if "bias" in parts else None
    residual = d.normal(N, M) if "residual" in parts else None
    return W, mask, X, bias, residual, _activation(parts)


# The block's layers: name, output, input (the stand-in for attention's output is q), epilogue.
def _block_layers(case):
    h, f = case["hidden"], case["ffn"]
    return [("q", h, h), ("k", h, h), ("v", h, h), ("o", h, h), ("up", f, h), ("down", h, f)]


def _block_inputs(case, seed):
    d = _Draws(seed)
    layers = []
    for name, M, K in _block_layers(case):
        W, mask = d.weight(M, K, case["sparsity"])
        layers.append((name, W, mask, d.normal(M, scale=0.02)))
    return layers, d.normal(case["N"], case["hidden"])


def _prepare_product(case, seed):
    W, mask, X, bias, residual, act = _product_inputs(case, seed)
    if case["api"] == "module":
        return dict(module=SparseLinear(W, mask, bias, act), X=X, residual=residual)
    A = usp.SparseMatrix(*_host(W, mask))
    Y = torch.empty((case["N"], case["M"]), dtype=torch.float16, device="cuda")
    return dict(A=A, X=X, Y=Y, ws=A.make_workspace(case["N"]), bias=bias, residual=residual, act=act)


def _run_product(s):
    if "module" in s:
        return s["module"](s["X"], s["residual"])
    if s["bias"] is None and s["residual"] is None and s["act"] == "none":
        usp.usp_spmm(s["A"].handle, s["X"], s["Y"], s["ws"])
    else:
        usp.usp_spmm_ex(s["A"].handle, s["X"], s["Y"], s["ws"], s["bias"], s["residual"], s["act"])
    return s["Y"]


def _prepare_block(case, seed):
    layers, X = _block_inputs(case, seed)
    N = case["N"]
    A = {name: usp.SparseMatrix(*_host(W, mask)) for name, W, mask, _ in layers}
    bias = {name: b for name, _, _, b in layers}
    out = {name: torch.empty((N, m.M), dtype=torch.float16, device="cuda") for name, m in A.items()}
    # One workspace for the six products, which run one after another.
    ws = torch.zeros(max(1, max(m.workspace_size(N) for m in A.values())), dtype=torch.uint8, device="cuda")

    def step():
        for name in ("q", "k", "v"):
            usp.usp_spmm_ex(A[name].handle, X, out[name], ws, bias[name])
        usp.usp_spmm_ex(A["o"].handle, out["q"], out["o"], ws, bias["o"], X)
        usp.usp_spmm_ex(A["up"].handle, out["o"], out["up"], ws, bias["up"], activation="relu")
        usp.usp_spmm_ex(A["down"].handle, out["up"], out["down"], ws, bias["down"], out["o"])

    step()  # before the capture, as PyTorch asks for
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    return dict(graph=graph, A=A, X=X, bias=bias, ws=ws, out=out)


def _run_block(s):
    s["graph"].replay()
    return s["out"]


def _run_load(s):
    s["A"] = A = usp.SparseMatrix(s["W"], s["mask"])  # the layer loaded before it is freed
    return A.densify()


def prepare(case, seed):
    if case["kind"] == "product":
        return _prepare_product(case, seed)
    if case["kind"] == "block":
        return _prepare_block(case, seed)
    W, mask = _host(*_Draws(seed).weight(case["M"], case["K"], case["sparsity"]))
    return dict(W=W, mask=mask, A=None)


def run(state):
    if "graph" in state:
        return _run_block(state)
    if "W" in state:
        return _run_load(state)
    return _run_product(state)


def _weight_bytes(M, K, sparsity):
    """One bit per position and the kept fp16 values."""
    return M * K / 8 + 2 * _kept(M, K, sparsity)


def _kept(M, K, sparsity):
    return M * (K - K * sparsity // 100)


def work(case):
    s = case["sparsity"]
    if case["kind"] == "load":
        M, K = case["M"], case["K"]
        # Host weight and mask in, the encoding to the device and read back there, the dense weight out.
        return {"bytes": 3 * M * K + 2 * _weight_bytes(M, K, s) + 2 * M * K, "flops": 0}
    if case["kind"] == "block":
        N = case["N"]
        shapes = [(M, K) for _, M, K in _block_layers(case)]
        return {"bytes": sum(_weight_bytes(M, K, s) + 2 * N * (M + K) + 2 * M for M, K in shapes) +
                2 * 2 * N * case["hidden"],
                "flops": sum(2.0 * _kept(M, K, s) * N for M, K in shapes)}
    M, K, N, parts = case["M"], case["K"], case["N"], _parts(case)
    extra = (2 * M if "bias" in parts else 0) + (2 * M * N if "residual" in parts else 0)
    return {"bytes": _weight_bytes(M, K, s) + 2 * N * (M + K) + extra, "flops": 2.0 * _kept(M, K, s) * N}


def tolerance(case):
    if case["kind"] == "load":
        return "exact"
    if case["kind"] == "block":
        # Four products deep, each rounding its output to fp16 (4e-4 against 64 bits).
        return {"rel": 1.6e-3, "max": 1.6e-2}
    # fp32 sums of exact fp16 products, one rounding to fp16 (2.1e-4 against 64 bits; an ulp is up to
    # 2^-10 of the value).
    return {"rel": 8e-4, "max": 4e-3}


def _masked_product(W, mask, X):
    """X (W * mask)^T in float64, in slices of rows that fit the card several times over."""
    x = X.double()
    out = torch.empty((X.shape[0], W.shape[0]), dtype=torch.float64, device="cuda")
    for r in range(0, W.shape[0], 4096):
        w = torch.where(mask[r:r + 4096], W[r:r + 4096], torch.zeros((), dtype=W.dtype, device="cuda")).double()
        out[:, r:r + 4096] = x @ w.t()
    return out


def _act64(v, act):
    if act == "relu":
        return v.clamp_min(0)
    if act == "gelu_tanh":
        return torch.nn.functional.gelu(v, approximate="tanh")
    if act == "silu":
        return torch.nn.functional.silu(v)
    return v


def exact(case, seed):
    if case["kind"] == "load":
        W, mask = _Draws(seed).weight(case["M"], case["K"], case["sparsity"])
        return torch.where(mask, W, torch.zeros((), dtype=W.dtype, device="cuda")).double()
    if case["kind"] == "block":
        layers, X = _block_inputs(case, seed)
        L = {name: (W, mask, b.double()) for name, W, mask, b in layers}

        def linear(name, x):
            W, mask, b = L[name]
            return _masked_product(W, mask, x) + b

        out = {name: linear(name, X) for name in ("q", "k", "v")}
        out["o"] = linear("o", out["q"]) + X.double()
        out["up"] = linear("up", out["o"]).clamp_min(0)
        out["down"] = linear("down", out["up"]) + out["o"]
        return out
    W, mask, X, bias, residual, act = _product_inputs(case, seed)
    v = _masked_product(W, mask, X)
    if bias is not None:
        v += bias.double()
    v = _act64(v, act)
    if residual is not None:
        v += residual.double()
    return v
