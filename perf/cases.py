"""The work a user of the quantized linear layer gives it, as measurable cases.

A case is a dict of plain values.  Four kinds:

  linear     one layer call: an activation quantizer (plain, with Eq. 3's balancing factor, or
             fused behind LayerNorm, GELU, the residual add or the Hadamard rotation) and the
             integer GEMM.  Weights are quantized once and the workspace is kept, as a module
             would; the output is allocated by the call, as in a module's forward.
  block      the linear layers of one transformer block in model order, buffers kept.
  calibrate  offline, per layer: channel statistics of an activation batch (running maximum over
             the batches of a calibration set) and of the weight, and the balancing mask.
  weights    offline, per layer: a floating-point weight matrix to codes and channel scales.

Inputs are drawn on the device with the value structure of the synthetic workloads of this
repository: Gaussian bulk, per-channel spread with a few outlier channels, weights N(0, 0.02).
"""
from __future__ import annotations

import math

import torch

import paper_2406_02540_amd as vq

HIDDEN, MLP = 1152, 4608
PRODUCERS = ("plain", "balanced", "layernorm", "gelu", "residual", "hadamard")

# Layers of a block: (name, tokens or None for the block's own, K, N, producer).
# "deployed": the quantizer sits behind the operation in front of the layer (image DiT).
# "plain": every layer takes fp16 activations (video DiT with the prompt's cross-attention k/v).
BLOCKS = {
    "deployed": (("qkv", None, HIDDEN, 3 * HIDDEN, "layernorm"), ("proj", None, HIDDEN, HIDDEN, "balanced"),
                 ("fc1", None, HIDDEN, MLP, "layernorm"), ("fc2", None, MLP, HIDDEN, "gelu")),
    "plain": (("qkv", None, HIDDEN, 3 * HIDDEN, "plain"), ("proj", None, HIDDEN, HIDDEN, "plain"),
              ("fc1", None, HIDDEN, MLP, "plain"), ("fc2", None, MLP, HIDDEN, "plain"),
              ("ca_kv", 240, 4096, 2 * HIDDEN, "plain")),
}


def _linear(name, M, K, N, bits, producer):
    return {"name": name, "kind": "linear", "M": M, "K": K, "N": N, "bits": bits, "producer": producer}


def listed():
    return [
        # a single small linear, latency bound: one image of 256 tokens
        _linear("small_w8", 256, HIDDEN, HIDDEN, 8, "plain"),
        # the same with 4-bit weights
        _linear("small_w4", 256, HIDDEN, HIDDEN, 4, "plain"),
        # cross-attention k/v of the prompt: few tokens, long K
        _linear("text_kv_w8", 240, 4096, 2304, 8, "plain"),
        # an ordinary-sized MLP input layer behind LayerNorm, a token count that divides nothing
        _linear("ragged_fc1_w8", 1001, HIDDEN, MLP, 8, "layernorm"),
        # sizes that no tile and no vector width divides: stores of N % 8 != 0, a tail in K
        _linear("odd_w8", 2891, 1168, 2820, 8, "balanced"),
        # the rotation-balanced layer in 4 bits at image size
        _linear("image_rotated_qkv_w4", 8192, HIDDEN, 3 * HIDDEN, 4, "hadamard"),
        # image DiT, CFG pair of 64 x 64 patches: the block's layers behind their producers
        {"name": "image_block_w8", "kind": "block", "M": 8192, "bits": 8, "layers": "deployed"},
        # video DiT: the layer behind a residual add
        _linear("video_residual_w8", 32768, HIDDEN, HIDDEN, 8, "residual"),
        # video DiT: MLP output layer behind GELU, 4-bit weights
        _linear("video_gelu_fc2_w4", 32768, MLP, HIDDEN, 4, "gelu"),
        # video DiT, 16 frames of 32 x 32 patches and the CFG pair: the largest call sequence
        {"name": "video_block_w8", "kind": "block", "M": 32768, "bits": 8, "layers": "plain"},
        # offline calibration of one layer on one batch of video activations
        {"name": "calibrate", "kind": "calibrate", "M": 32768, "K": HIDDEN, "N": MLP},
        # offline: a weight rotated and packed to 4 bits
        {"name": "weights_rotated_w4", "kind": "weights", "K": HIDDEN, "N": MLP, "bits": 4, "rotate": True},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_k(rng, step):
    if rng.random() < 0.4:
        return rng.choice((HIDDEN, HIDDEN, 4096, MLP))
    return max(step, min(MLP, _log_int(rng, 256, MLP) // step * step))


def draw(rng):
    u = rng.random()
    if u < 0.70:
        producer = rng.choice(PRODUCERS)
        bits = rng.choice((8, 4))
        K = _draw_k(rng, 128 if producer == "hadamard" else 16 if bits == 8 else 32)
        N = rng.choice((HIDDEN, 3 * HIDDEN, MLP)) if rng.random() < 0.4 else _log_int(rng, 32, MLP)
        if N % 8 and rng.random() < 0.7:
            N = N // 8 * 8
        M = min(_log_int(rng, 1, 32768), 32768 * HIDDEN * MLP // (K * N))
        return {"kind": "linear", "M": M, "K": K, "N": N, "bits": bits, "producer": producer}
    if u < 0.80:
        return {"kind": "block", "M": _log_int(rng, 64, 16384), "bits": rng.choice((8, 4)),
                "layers": rng.choice(("deployed", "plain"))}
    if u < 0.90:
        return {"kind": "calibrate", "M": _log_int(rng, 64, 32768), "K": _draw_k(rng, 8), "N": _log_int(rng, 64, MLP)}
    rotate = rng.random() < 0.4
    return {"kind": "weights", "K": _draw_k(rng, 128 if rotate else 8), "N": _log_int(rng, 64, MLP),
            "bits": rng.choice((8, 4)), "rotate": rotate}


def _samples(M):
    """A classifier-free-guidance pair: two samples wherever there are two tokens."""
    T = (M + 1) // 2
    return T, (M + T - 1) // T


class _Layer:
    """What a program holds for one layer: quantized weights, this pass's inputs, kept scratch."""

    def __init__(self, g, M, K, N, bits, producer, keep_output):
        def normal(*shape):
            return torch.randn(shape, generator=g, device="cuda")

        def uniform(lo, hi, n):
            return torch.rand((n,), generator=g, device="cuda") * (hi - lo) + lo

        self.bits, self.producer = bits, producer
        w = normal(N, K) * 0.02
        self.bias = (normal(N) * 0.01).half()
        self.chan_mul = self.gate = self.scale = self.shift = self.y_in = None
        s = None
        if producer in ("balanced", "layernorm", "hadamard"):
            s = torch.exp(uniform(math.log(0.25), math.log(4.0), K))
            self.chan_mul = 1.0 / s
        if producer == "hadamard":
            w, s = vq.vq_rotate_weight(w, s), None
        self.w, self.w_scale = vq.vq_quantize_weight(w, s, bits)
        # activations: GELU takes the N(0,1)-like output of fc1, the others the spread of a
        # residual stream
        x = normal(M, K)
        if producer != "gelu":
            sigma = torch.exp(uniform(math.log(0.1), math.log(10.0), K))
            sigma[torch.randperm(K, generator=g, device="cuda")[: max(1, K // 100)]] *= 50.0
            x *= sigma
        self.x = x.half()
        self.T, B = _samples(M)
        if producer == "layernorm":
            self.scale, self.shift = normal(B, K) * 0.2, normal(B, K) * 0.5
        if producer == "residual":
            self.y_in, self.gate = normal(M, K).half(), normal(B, K) * 0.5
        self.workspace = torch.empty((max(16, vq.vq_linear_workspace_bytes(M, N, K, bits)),), dtype=torch.uint8, device="cuda")
        self.y = torch.empty((M, N), dtype=torch.float16, device="cuda") if keep_output else None

    def __call__(self):
        p = self.producer
        if p == "layernorm":
            return vq.vq_layernorm_linear(self.x, self.w, self.bits, self.w_scale, self.scale, self.shift, self.T, 1e-6,
                                          self.chan_mul, self.bias, self.y, self.workspace)
        if p == "gelu":
            return vq.vq_gelu_linear(self.x, self.w, self.bits, self.w_scale, True, self.chan_mul, self.bias, self.y,
                                     self.workspace)
        if p == "residual":
            return vq.vq_residual_linear(self.x, self.y_in, self.w, self.bits, self.w_scale, self.gate, self.T, None,
                                         self.chan_mul, self.bias, self.y, self.workspace)
        if p == "hadamard":
            return vq.vq_hadamard_linear(self.x, self.chan_mul, self.w, self.bits, self.w_scale, self.bias, self.y,
                                         self.workspace)
        return vq.vq_linear(self.x, self.chan_mul, self.w, self.bits, self.w_scale, self.bias, self.y, self.workspace)


class _Calibrate:
    def __init__(self, g, M, K, N):
        self.x = torch.randn((M, K), generator=g, device="cuda").mul_(
            torch.exp(torch.rand((K,), generator=g, device="cuda") * math.log(100.0)) * 0.1).half()
        self.w = torch.randn((N, K), generator=g, device="cuda") * 0.02
        # the running maximum over the batches seen before: of their size
        self.amax_x = self.x[: max(1, M // 2)].abs().amax(0).float()

    def __call__(self):
        amax_x = vq.vq_channel_absmax(self.x, self.amax_x, accumulate=True)
        amax_w = vq.vq_channel_absmax(self.w)
        s, chan_mul = vq.vq_balance_mask(amax_x, amax_w, 0.5)
        return amax_x, amax_w, s, chan_mul


class _Weights:
    def __init__(self, g, K, N, bits, rotate):
        self.w = torch.randn((N, K), generator=g, device="cuda") * 0.02
        self.s = torch.exp((torch.rand((K,), generator=g, device="cuda") * 2.0 - 1.0) * math.log(4.0))
        self.bits, self.rotate = bits, rotate

    def __call__(self):
        if self.rotate:
            return vq.vq_quantize_weight(vq.vq_rotate_weight(self.w, self.s), None, self.bits)
        return vq.vq_quantize_weight(self.w, self.s, self.bits)


def _layers_of(case):
    if case["kind"] == "linear":
        return [(case["M"], case["K"], case["N"], case["producer"])]
    return [(m or case["M"], k, n, p) for _, m, k, n, p in BLOCKS[case["layers"]]]


def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    if case["kind"] == "calibrate":
        return _Calibrate(g, case["M"], case["K"], case["N"])
    if case["kind"] == "weights":
        return _Weights(g, case["K"], case["N"], case["bits"], case["rotate"])
    layers = [_Layer(g, M, K, N, case["bits"], p, case["kind"] == "block") for M, K, N, p in _layers_of(case)]
    return layers[0] if case["kind"] == "linear" else layers


def run(state):
    if isinstance(state, list):
        return [layer() for layer in state]
    return state()


def work(case):
    if case["kind"] == "calibrate":
        M, K, N = case["M"], case["K"], case["N"]
        return {"bytes": 2 * M * K + 4 * N * K + 5 * 4 * K, "flops": M * K + N * K}
    if case["kind"] == "weights":
        K, N, bits = case["K"], case["N"], case["bits"]
        return {"bytes": 4 * N * K + N * K * bits // 8 + 4 * N + 4 * K, "flops": N * K * (10 if case["rotate"] else 3)}
    nbytes = flops = 0
    for M, K, N, p in _layers_of(case):
        nbytes += 2 * M * K + N * K * case["bits"] // 8 + 6 * N + 2 * M * N
        if p == "residual":
            nbytes += 4 * M * K + 4 * K * _samples(M)[1]   # the branch output and the new residual stream
        if p == "layernorm":
            nbytes += 8 * K * _samples(M)[1]
        if p in ("balanced", "layernorm", "hadamard"):
            nbytes += 4 * K
        flops += 2 * M * N * K
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # Codes, token scales and integer sums are fully determined, and the dequantization is
    # pinned to one rounding: these paths give the same bits whatever the kernel.
    # The others were compared with their producer in 64 bits; four times the difference seen.
    if case["kind"] == "calibrate":
        return {"rel": 3e-7, "max": 1e-6}   # maxima exact; the mask's powf: 6e-8, 2.2e-7
    if case["kind"] == "weights":           # rotated: scales 3e-7 apart, codes on a tie may differ by one
        return {"rel": 6e-7, "max": 1.2e-6, "differ": 1e-4} if case["rotate"] else "exact"
    if all(p in ("plain", "balanced", "residual") for _, _, _, p in _layers_of(case)):
        return "exact"
    return {"rel": 5e-4}                    # 7e-6 to 1.3e-4: a code next to a tie differs by one
