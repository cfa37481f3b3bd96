"""Workloads of the RRS W4A4 linear layer: sizes, inputs, one pass, and a 64-bit reference.

The listed cases are what a language model's linear layers ask of the library: single-token
and batched decode, short and chunked prompts, prefill at the LLaMA-7B shapes, a large prefill,
the runtime channel reorder, the static reorder and the per-channel (QuaRot) setting. `draw`
gives more calls from the same ranges: 1 to 8192 tokens, K from 1024 to 16384, N from 256 to
28672 in steps of 16, group sizes 64 to 512, both weight layouts.

A case's fields: op (which entry points a pass calls), M tokens, K input channels, N output
channels, g smoothing group, tiled (weight layout), perm (static channel reorder), layers (how
many layers with weights of their own a pass goes through, as one decode step does; it keeps
the weights from being served by the 256 MB memory-side cache where a model's would not be).

  linear        rrs.linear                                  -> Y per layer
  quant_gemm    rrs.rotate_smooth_quant, rrs.w4a4_gemm      -> codes, scales, Y
  reorder       rrs.linear_reorder                          -> Y per layer
  per_channel   rrs.rotate_smooth_quant (no smoothing), rrs.w4a4_gemm_per_channel -> Y

Inputs: standard normal tokens with 1 % of the channels scaled by 20 to 100 and a few isolated
spikes of 100 to 500; weights 0.02 times standard normal.
"""
import math

import torch

import paper_2409_20361_amd as rrs


def _case(op, M, K, N, g=128, tiled=False, perm=False, layers=1, name=None):
    c = {"op": op, "M": M, "K": K, "N": N, "g": g, "tiled": tiled, "perm": perm,
         "layers": layers}
    return c if name is None else {"name": name, **c}


def listed():
    return [
        # One token through attention output projections: the smallest call.
        _case("linear", 1, 4096, 4096, layers=8, name="decode_1"),
        # Eight sequences decoding through a wide MLP projection: bound by the weights.
        _case("linear", 8, 8192, 28672, layers=4, name="decode_8"),
        # Sixteen sequences with the runtime reorder on the fused QKV projection.
        _case("reorder", 16, 4096, 12288, layers=4, name="decode_16_reorder"),
        # A larger decode batch (odd count) on gate/up with the streaming weight layout.
        _case("linear", 49, 4096, 22016, tiled=True, layers=3, name="decode_49_tiled"),
        # A short prompt of odd length on a square projection.
        _case("linear", 173, 4096, 4096, name="prompt_173"),
        # A prefill chunk on a square projection of a wider model.
        _case("linear", 512, 8192, 8192, name="chunk_512"),
        # A ragged prompt through a long contraction (down projection), static reorder.
        _case("linear", 777, 16384, 4096, g=256, tiled=True, perm=True, name="down_777_perm"),
        # Rotation without smoothing: one scale per token and per output channel.
        _case("per_channel", 1024, 4096, 12288, name="per_channel_1024"),
        # A ragged prompt with the runtime reorder on the fused QKV projection.
        _case("reorder", 1500, 4096, 12288, name="qkv_1500_reorder"),
        # The fused QKV projection at 2048 tokens, codes shared by the caller.
        _case("quant_gemm", 2048, 4096, 12288, name="qkv_2048"),
        # The fused gate/up projection at 4096 tokens.
        _case("linear", 4096, 4096, 22016, name="gateup_4096"),
        # A large prefill with the finer smoothing group.
        _case("linear", 8192, 8192, 28672, g=64, name="large_8192"),
    ]


_MAX_COST = 8192 * 8192 * 28672


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        op = rng.choice(["linear", "linear", "linear", "quant_gemm", "reorder", "per_channel"])
        M = _log_int(rng, 1, 8192)
        K = rng.choice([1024, 2048, 4096, 4096, 8192, 16384])
        N = 16 * _log_int(rng, 16, 1792)
        g = rng.choice([64, 128, 128, 256, 512])
        perm = op == "linear" and rng.random() < 0.125
        layers = rng.choice([2, 3, 4]) if M <= 64 and op in ("linear", "reorder") else 1
        if M * K * N <= _MAX_COST and M * N <= 8192 * 28672:
            return _case(op, M, K, N, g, rng.random() < 0.4, perm, layers)


def _flags(case):
    return (rrs.WEIGHT_TILED if case["tiled"] else 0) | (
        rrs.SKIP_SMOOTHING if case["op"] == "per_channel" else 0)


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _weight(case, seed, layer):
    gen = _generator(1000003 * (layer + 1) + seed)
    W = torch.randn((case["K"], case["N"]), generator=gen, device="cuda", dtype=torch.float32)
    return W.mul_(0.02).half()


def _inputs(case, seed):
    """X (M x K fp16) and the static channel order (or None)."""
    M, K = case["M"], case["K"]
    gen = _generator(seed)
    X = torch.randn((M, K), generator=gen, device="cuda", dtype=torch.float32)
    nchan = max(1, K // 100)
    cols = torch.randperm(K, generator=gen, device="cuda")[:nchan]
    fac = torch.rand(nchan, generator=gen, device="cuda") * math.log(5.0)
    X[:, cols] *= 20.0 * torch.exp(fac)
    nspike = max(1, M * K // 10000)
    pos = torch.randint(0, M * K, (nspike,), generator=gen, device="cuda")
    mag = 100.0 + 400.0 * torch.rand(nspike, generator=gen, device="cuda")
    sgn = 1.0 - 2.0 * torch.randint(0, 2, (nspike,), generator=gen, device="cuda").float()
    flat = X.view(-1)
    flat.index_put_((pos,), mag * sgn)
    # Two spikes on one place would be written in either order: give such a place one value.
    once, count = torch.unique(pos, return_counts=True)
    flat[once[count > 1]] = 300.0
    perm = None
    if case["perm"]:
        perm = torch.randperm(K, generator=gen, device="cuda").to(torch.int32)
    return X.half(), perm


def prepare(case, seed):
    M, K, N, g = case["M"], case["K"], case["N"], case["g"]
    X, perm = _inputs(case, seed)
    wflags = rrs.WEIGHT_TILED if case["tiled"] else 0
    layers = [rrs.prepare_weight(_weight(case, seed, i), perm, flags=wflags)
              for i in range(case["layers"])]
    if case["op"] == "reorder":
        nbytes = rrs.linear_reorder_workspace_bytes(M, K, g)
    elif case["op"] == "linear":
        nbytes = rrs.linear_workspace_bytes(M, K, g)
    else:
        nbytes = rrs.workspace_bytes(M, K, g)
    state = {"op": case["op"], "g": g, "flags": _flags(case), "X": X, "perm": perm,
             "layers": layers,
             "workspace": torch.zeros(nbytes, dtype=torch.uint8, device="cuda"),
             "Y": [torch.empty((M, N), dtype=torch.float16, device="cuda") for _ in layers]}
    if case["op"] in ("quant_gemm", "per_channel"):
        state["codes"] = (torch.empty((M, K // 2), dtype=torch.uint8, device="cuda"),
                          torch.empty((M,), dtype=torch.float32, device="cuda"),
                          torch.empty((K // g,), dtype=torch.float32, device="cuda"))
    return state


def run(state):
    op, g, flags, X, ws = (state[k] for k in ("op", "g", "flags", "X", "workspace"))
    if op == "linear":
        return [rrs.linear(X, Wq, w_scale, g, perm=state["perm"], workspace=ws, out=Y,
                           flags=flags)
                for (Wq, w_scale), Y in zip(state["layers"], state["Y"])]
    if op == "reorder":
        return [rrs.linear_reorder(X, Wq, w_scale, g, workspace=ws, out=Y, flags=flags)
                for (Wq, w_scale), Y in zip(state["layers"], state["Y"])]
    Wq, w_scale = state["layers"][0]
    Xq, a_scale, s_group = rrs.rotate_smooth_quant(X, g, workspace=ws, out=state["codes"],
                                                   flags=flags)
    if op == "quant_gemm":
        Y = rrs.w4a4_gemm(Xq, a_scale, s_group, Wq, w_scale, g, out=state["Y"][0], flags=flags)
        return [Xq, a_scale, s_group, Y]
    return [rrs.w4a4_gemm_per_channel(Xq, a_scale, Wq, w_scale, out=state["Y"][0],
                                      flags=flags & rrs.WEIGHT_TILED)]


def work(case):
    M, K, N, g, L = (case[k] for k in ("M", "K", "N", "g", "layers"))
    nbytes = L * (2 * M * K + N * K // 2 + 4 * N + 2 * M * N)
    if case["op"] == "quant_gemm":
        nbytes += M * K // 2 + 4 * M + 4 * (K // g)
    if case["perm"]:
        nbytes += 4 * K
    flops = L * (2 * M * N * K + M * K * (K.bit_length() - 1))
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # Y is float16: against `exact` it is off by 2.0e-4 to 4.5e-4 in the 2-norm over the listed
    # cases (its own rounding, and a few codes whose pre-rounding value lies within fp32 rounding
    # of a half-integer). Codes and scales are the same bits in every correct implementation (one
    # fp32 arithmetic decides them), so another order of the fp32 sum over the groups changes Y
    # by one float16 step here and there (1e-3 of the value).
    return {"rel": 1e-3, "max": 5e-3, "differ": 0.0}


def _hadamard(y, dim):
    """The unnormalized Sylvester transform along `dim` (0 or 1) of a matrix, in place of `y`."""
    n = y.shape[dim]
    h = 1
    while h < n:
        if dim == 1:
            v = y.view(y.shape[0], n // (2 * h), 2, h)
            a, b = v[:, :, 0], v[:, :, 1]
        else:
            v = y.view(n // (2 * h), 2, h, y.shape[1])
            a, b = v[:, 0], v[:, 1]
        s = a + b
        b.mul_(-1.0).add_(a)
        a.copy_(s)
        h *= 2
    return y


def _codes(v, m):
    """clamp(round(7 v / m)) with rows or columns of zeros giving zeros."""
    inv = torch.where(m > 0, 7.0 / m, torch.zeros_like(m))
    return torch.clamp(torch.round(v * inv), -7, 7)


def exact(case, seed):
    M, K, N, g = case["M"], case["K"], case["N"], case["g"]
    X, perm = _inputs(case, seed)
    y = _hadamard(X.double(), 1)
    if perm is not None:
        y = y[:, perm.long()]
    order = None
    if case["op"] == "reorder":
        key = y.abs().amax(0).view(K // 32, 32).amax(1)
        order = torch.sort(key, descending=True, stable=True).indices
        y = y.view(M, K // 32, 32)[:, order].reshape(M, K)
    G = K // g
    if case["op"] == "per_channel":
        s = torch.ones(G, dtype=torch.float64, device="cuda")
    else:
        s = y.abs().amax(0).view(G, g).amax(1)
    r = torch.where(s > 0, 1.0 / s, torch.zeros_like(s))
    y = (y.view(M, G, g) * r[None, :, None]).view(M, K)
    a = y.abs().amax(1)
    q = _codes(y, a[:, None])
    del y
    left = (q.view(M, G, g) * s[None, :, None]).view(M, K) * (a[:, None] / 7.0)
    outs = []
    for i in range(case["layers"]):
        u = _hadamard(_weight(case, seed, i).double(), 0)
        if perm is not None:
            u = u[perm.long()]
        b = u.abs().amax(0)
        w = _codes(u, b[None, :])
        del u
        if order is not None:
            w = w.view(K // 32, 32, N)[order].reshape(K, N)
        outs.append((left @ w) * (b[None, :] / 7.0 / K))
        del w
    if case["op"] == "quant_gemm":
        return [None, a / 7.0, s, outs[0]]
    return outs
