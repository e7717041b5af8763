"""The work that programs have this library do, as measured cases: inputs, one pass through the
public entry points, the least work of a pass, and the same pass in 64 bits.

Kinds of case (the sizes are the library's own workloads or generic ragged ones):

  linear      one fused projection, called eagerly (`fq.linear`), or its two halves on their own
              (`fq.fwht_quant`, then `fq.gemm`) with the folds, the clip ratio and the bias in use
  expert      the action expert's denoising loop: four projection sites a step, several steps,
              captured in one HIP graph and replayed
  stack       one projection of every layer of a stack, each with its own weights, in one HIP graph
              (decode: the weights come from memory, not from a cache)
  backbone    one selective-INT8 language layer at prefill, its four projection sites called eagerly
  modulation  the weight-only INT4 modulation of every layer of a stack, in one HIP graph
  rotated     the prologue with the stored composite rotation, then the integer GEMM, called eagerly
  gptq        GPTQ rounding of one site's weights from calibration tokens, then packing
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2609_24433_amd import fq


def listed():
    return [
        # the smallest call: one small projection with nothing preallocated; launch and call latency
        {"name": "single_linear", "kind": "linear", "M": 64, "K": 1024, "N": 1024, "b": 64, "bits": 4, "split": False,
         "fold": "none", "bias": False, "clip": 1.0, "heavy": False, "keep": False},
        # the headline workload: ten denoising steps of the action-expert layer
        {"name": "expert_loop", "kind": "expert", "steps": 10, "M": 50, "width": 1024, "kv": 256, "ffn": 4096, "b": 128},
        # the action tokens through the wide down projection of every layer
        {"name": "down_stack_w4_m50", "kind": "stack", "layers": 18, "M": 50, "K": 16384, "N": 2048, "b": 128, "bits": 4},
        # the same in INT8 at a small batch (selective INT8 keeps the down projection at 8 bits)
        {"name": "down_stack_w8_m16", "kind": "stack", "layers": 18, "M": 16, "K": 16384, "N": 2048, "b": 128, "bits": 8},
        # prefill of one language layer with o and down at 8 bits
        {"name": "backbone_mixed", "kind": "backbone", "M": 816, "width": 2048, "kv": 256, "ffn": 16384, "b": 128},
        # prefill down projection at 4 bits
        {"name": "down_w4_m816", "kind": "linear", "M": 816, "K": 16384, "N": 2048, "b": 128, "bits": 4, "split": False,
         "fold": "none", "bias": False, "clip": 1.0, "heavy": True, "keep": True},
        # the longest batches, both widths
        {"name": "down_w4_m4096", "kind": "linear", "M": 4096, "K": 16384, "N": 2048, "b": 128, "bits": 4, "split": False,
         "fold": "none", "bias": False, "clip": 1.0, "heavy": True, "keep": True},
        {"name": "down_w8_m4096", "kind": "linear", "M": 4096, "K": 16384, "N": 2048, "b": 64, "bits": 8, "split": False,
         "fold": "none", "bias": False, "clip": 1.0, "heavy": True, "keep": True},
        # ragged sizes, both folds, a clip ratio and a bias, through the two separate entry points
        {"name": "ragged_split", "kind": "linear", "M": 333, "K": 2944, "N": 3056, "b": 64, "bits": 4, "split": True,
         "fold": "both", "bias": True, "clip": 0.9, "heavy": False, "keep": True},
        # the conditioning token through every layer's modulation
        {"name": "modulation", "kind": "modulation", "layers": 18, "M": 1, "K": 1024, "N": 6144},
        # the composite rotation at prefill
        {"name": "rotated_m816", "kind": "rotated", "M": 816, "K": 2048, "N": 2048, "b": 128, "bits": 4},
        # offline: rounding the action expert's q|k|v weights
        {"name": "gptq_qkv", "kind": "gptq", "T": 2048, "K": 1024, "N": 1536, "b": 128, "bits": 4},
    ]


# ---------------------------------------------------------------- drawn cases

def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _mult(rng, lo, hi, m):
    return max(lo // m, min(hi // m, int(round(_log(rng, lo, hi) / m)))) * m


def _block(rng, K, choices):
    return rng.choice([b for b in choices if K % b == 0])


def draw(rng):
    kind = rng.choice(["linear"] * 5 + ["stack"] * 2 + ["backbone"] * 2 + ["expert", "modulation", "rotated", "gptq"])
    if kind == "linear":
        while True:
            M, K, N = int(_log(rng, 1, 4096.9)), _mult(rng, 512, 16384, 128), _mult(rng, 256, 32768, 16)
            if M * K * N <= 4096 * 16384 * 2048 and K * N <= 1 << 26 and M * N <= 1 << 25:
                break
        return {"kind": kind, "M": M, "K": K, "N": N, "b": _block(rng, K, [32, 64, 128, 256]), "bits": rng.choice([4, 8]),
                "split": rng.random() < 0.4, "fold": rng.choice(["none", "none", "before", "after", "both"]),
                "bias": rng.random() < 0.4, "clip": rng.choice([1.0, 1.0, 0.9]), "heavy": rng.random() < 0.5,
                "keep": rng.random() < 0.7}
    if kind == "expert":
        return {"kind": kind, "steps": 10, "M": rng.randint(16, 64), "width": rng.choice([768, 1024]),
                "kv": rng.choice([128, 256]), "ffn": rng.choice([2048, 3072, 4096]), "b": rng.choice([64, 128])}
    if kind == "stack":
        K = _mult(rng, 1024, 16384, 128)
        return {"kind": kind, "layers": 18, "M": int(_log(rng, 1, 64.9)), "K": K, "N": _mult(rng, 512, 2048, 16),
                "b": _block(rng, K, [32, 64, 128, 256]), "bits": rng.choice([4, 8])}
    if kind == "backbone":
        return {"kind": kind, "M": int(_log(rng, 96, 1024.9)), "width": _mult(rng, 1024, 2048, 128), "kv": rng.choice([128, 256]),
                "ffn": _mult(rng, 4096, 16384, 128), "b": rng.choice([32, 64, 128])}
    if kind == "modulation":
        return {"kind": kind, "layers": 18, "M": int(_log(rng, 1, 16.9)), "K": _mult(rng, 512, 2048, 128),
                "N": _mult(rng, 2048, 12288, 16)}
    if kind == "rotated":
        K = _mult(rng, 512, 4096, 128)
        return {"kind": kind, "M": int(_log(rng, 16, 816.9)), "K": K, "N": _mult(rng, 512, 2048, 16),
                "b": _block(rng, K, [16, 32, 64, 128]), "bits": rng.choice([4, 8])}
    K = _mult(rng, 256, 1024, 128)
    return {"kind": kind, "T": rng.randint(256, 2048), "K": K, "N": _mult(rng, 256, 1536, 16), "b": _block(rng, K, [32, 64, 128]),
            "bits": rng.choice([4, 8])}


# ---------------------------------------------------------------- inputs

class _Draws:
    """Seeded device tensors: tokens with a few outlier channels, N(0, 0.02) weights, positive scales."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(1000003 * (int(seed) + 1))

    def normal(self, *shape):
        return torch.randn(shape, generator=self.g, device="cuda", dtype=torch.float32)

    def uniform(self, n, lo, hi):
        return torch.rand((n,), generator=self.g, device="cuda", dtype=torch.float32) * (hi - lo) + lo

    def tokens(self, M, K, heavy=False):
        x = self.normal(M, K)
        if heavy:  # Student-t with three degrees of freedom
            c = self.normal(M, K).square_()
            for _ in range(2):
                c += self.normal(M, K).square_()
            x /= (c / 3).sqrt_()
        idx = torch.randperm(K, generator=self.g, device="cuda")[:max(1, K // 200)]
        x[:, idx] *= 100.0 if heavy else 50.0
        return x.to(torch.bfloat16)

    def weights(self, N, K):
        return self.normal(N, K).mul_(0.02)


def _linear_inputs(case, seed):
    d = _Draws(seed)
    M, K, N = case["M"], case["K"], case["N"]
    p = {"x": d.tokens(M, K, case["heavy"]), "w": d.weights(N, K), "s": None, "p": None, "bias": None}
    if case["fold"] in ("before", "both"):
        p["s"] = d.uniform(K, 0.5, 2.0)
    if case["fold"] in ("after", "both"):
        p["p"] = d.uniform(K, 0.5, 2.0)
    if case["bias"]:
        p["bias"] = d.uniform(N, -1.0, 1.0)
    return p


def _expert_sites(case):
    W, kv, F = case["width"], case["kv"], case["ffn"]
    return [(W, W + 2 * kv, 4), (W, W, 4), (W, 2 * F, 4), (F, W, 4)]


def _backbone_sites(case):
    W, kv, F = case["width"], case["kv"], case["ffn"]
    return [(W, W + 2 * kv, 4), (W, W, 8), (W, 2 * F, 4), (F, W, 8)]


def _site_inputs(case, seed, sites, steps):
    """Per site: the tokens of every step and the weights of its consumers, packed together."""
    d = _Draws(seed)
    return [([d.tokens(case["M"], K) for _ in range(steps)], d.weights(N, K)) for K, N, _ in sites]


def _stack_inputs(case, seed):
    d = _Draws(seed)
    heavy = case["kind"] == "stack"
    return [(d.tokens(case["M"], case["K"], heavy), d.weights(case["N"], case["K"])) for _ in range(case["layers"])]


def _rotated_inputs(case, seed):
    d = _Draws(seed)
    K, b = case["K"], case["b"]
    r = np.random.default_rng(int(seed))
    blocks = np.stack([np.linalg.qr(r.standard_normal((b, b)))[0] for _ in range(K // b)]).astype(np.float32)
    perm = r.permutation(K).astype(np.int32)
    return {"x": d.tokens(case["M"], K), "w": d.weights(case["N"], K), "perm": torch.from_numpy(perm).cuda(),
            "blocks": torch.from_numpy(blocks).cuda()}


def _gptq_inputs(case, seed):
    d = _Draws(seed)
    return {"calib": d.tokens(case["T"], case["K"], True), "w": d.weights(case["N"], case["K"])}


def _packed(w, b, bits, col=None, post=None):
    codes, scale = fq.quantize_weights(w, b, bits, col, post)
    return fq.pack_weights(codes, bits), scale


def _captured(body):
    """The calls of body() as one HIP graph, after one eager pass."""
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        body()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        body()
    return graph


def _scratch(case, sites):
    return fq.workspace(max(fq.linear_workspace_bytes(case["M"], N, K, bits) for K, N, bits in sites), "cuda")


def prepare(case, seed):
    kind, M = case["kind"], case["M"] if "M" in case else case["T"]
    if kind == "linear":
        p = _linear_inputs(case, seed)
        K, N, bits = case["K"], case["N"], case["bits"]
        st = {"kind": kind, "case": case, "x": p["x"], "bias": p["bias"],
              "pre": None if p["s"] is None else 1.0 / p["s"], "post": None if p["p"] is None else 1.0 / p["p"]}
        st["w"], st["scale"] = _packed(p["w"], case["b"], bits, p["s"], p["p"])
        st["out"] = st["ws"] = None
        if case["keep"]:  # a serving loop keeps its output and its scratch
            st["out"] = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
            need = fq.gemm_workspace_bytes if case["split"] else fq.linear_workspace_bytes
            st["ws"] = fq.workspace(need(M, N, K, bits), "cuda")
        return st
    if kind == "expert":
        sites, b = _expert_sites(case), case["b"]
        inputs = _site_inputs(case, seed, sites, case["steps"])
        packed = [_packed(w, b, bits) for (_, w), (_, _, bits) in zip(inputs, sites)]
        outs = [torch.empty((case["steps"], M, N), dtype=torch.bfloat16, device="cuda") for _, N, _ in sites]
        ws = _scratch(case, sites)

        def loop():
            for t in range(case["steps"]):
                for i, (K, N, bits) in enumerate(sites):
                    fq.linear(inputs[i][0][t], packed[i][0], packed[i][1], N, b, bits, ws=ws, out=outs[i][t])
        return {"kind": "graph", "graph": _captured(loop), "out": outs, "keep": (inputs, packed, ws)}
    if kind == "stack":
        K, N, b, bits = case["K"], case["N"], case["b"], case["bits"]
        layers = [(x,) + _packed(w, b, bits) for x, w in _stack_inputs(case, seed)]
        out = torch.empty((case["layers"], M, N), dtype=torch.bfloat16, device="cuda")
        ws = _scratch(case, [(K, N, bits)])

        def stack():
            for i, (x, w, scale) in enumerate(layers):
                fq.linear(x, w, scale, N, b, bits, ws=ws, out=out[i])
        return {"kind": "graph", "graph": _captured(stack), "out": out, "keep": (layers, ws)}
    if kind == "backbone":
        sites, b = _backbone_sites(case), case["b"]
        inputs = _site_inputs(case, seed, sites, 1)
        packed = [_packed(w, b, bits) for (_, w), (_, _, bits) in zip(inputs, sites)]
        return {"kind": kind, "x": [x[0] for x, _ in inputs], "packed": packed, "sites": sites, "b": b,
                "out": [torch.empty((M, N), dtype=torch.bfloat16, device="cuda") for _, N, _ in sites],
                "ws": _scratch(case, sites)}
    if kind == "modulation":
        K, N = case["K"], case["N"]
        layers = [(x,) + _packed(w, 1, 4) for x, w in _stack_inputs(case, seed)]
        out = torch.empty((case["layers"], M, N), dtype=torch.bfloat16, device="cuda")
        ws = fq.workspace(fq.w4a16_workspace_bytes(M, N, K), "cuda")

        def stack():
            for i, (x, w, scale) in enumerate(layers):
                fq.gemm_w4a16(x, w, scale, N, ws=ws, out=out[i])
        return {"kind": "graph", "graph": _captured(stack), "out": out, "keep": (layers, ws)}
    if kind == "rotated":
        p = _rotated_inputs(case, seed)
        codes, scale = fq.quantize_weights_rotated(p["w"], p["perm"], p["blocks"], case["b"], case["bits"])
        return {"kind": kind, "case": case, "x": p["x"], "perm": p["perm"], "blocks": p["blocks"],
                "w": fq.pack_weights(codes, case["bits"]), "scale": scale}
    p = _gptq_inputs(case, seed)
    return {"kind": kind, "case": case, "calib": p["calib"], "w": p["w"]}


# ---------------------------------------------------------------- one pass

def run(state):
    kind = state["kind"]
    if kind == "graph":
        state["graph"].replay()
        return state["out"]
    if kind == "backbone":
        for x, (w, scale), (K, N, bits), y in zip(state["x"], state["packed"], state["sites"], state["out"]):
            fq.linear(x, w, scale, N, state["b"], bits, ws=state["ws"], out=y)
        return state["out"]
    c = state["case"]
    if kind == "linear":
        if not c["split"]:
            return fq.linear(state["x"], state["w"], state["scale"], c["N"], c["b"], c["bits"], c["clip"], state["pre"],
                             state["bias"], state["ws"], state["out"], state["post"])
        codes, delta = fq.fwht_quant(state["x"], c["b"], c["bits"], c["clip"], state["pre"], post_inv=state["post"])
        y = fq.gemm(codes, delta, state["w"], state["scale"], c["N"], c["K"], c["bits"], state["bias"], ws=state["ws"],
                    out=state["out"])
        return {"codes": codes, "delta": delta, "y": y}
    if kind == "rotated":
        codes, delta = fq.rotate_quant(state["x"], state["perm"], state["blocks"], c["b"], c["bits"])
        y = fq.gemm(codes, delta, state["w"], state["scale"], c["N"], c["K"], c["bits"])
        return {"codes": codes, "delta": delta, "y": y}
    codes, scale = fq.gptq_quantize_weights(state["w"], state["calib"], c["b"], c["bits"])
    return {"codes": codes, "scale": scale, "packed": fq.pack_weights(codes, c["bits"])}


# ---------------------------------------------------------------- the least work of a pass

def _projection_work(M, K, N, bits):
    """A fused projection: bf16 tokens, packed weights and scales in, bf16 out; the contraction."""
    return 2 * M * K + N * K * bits // 8 + 4 * N + 2 * M * N, 2 * M * N * K


def work(case):
    kind = case["kind"]
    if kind == "gptq":
        T, K, N = case["T"], case["K"], case["N"]
        # tokens and weights read, codes, scales and the packed weights written; the second moment (one triangle), the factor
        # and the sweep
        return {"bytes": 2 * T * K + 4 * N * K + N * K + 4 * N + N * K * case["bits"] // 8,
                "flops": T * K * (K + 1) + 2 * K ** 3 // 3 + N * K * K}
    M = case["M"]
    if kind in ("expert", "backbone"):
        sites = _expert_sites(case) if kind == "expert" else _backbone_sites(case)
        steps = case["steps"] if kind == "expert" else 1
        by = fl = 0
        for K, N, bits in sites:
            b, f = _projection_work(M, K, N, bits)
            w = N * K * bits // 8 + 4 * N  # the weights serve every step
            by += steps * (b - w) + w
            fl += steps * f
        return {"bytes": by, "flops": fl}
    K, N = case["K"], case["N"]
    by, fl = _projection_work(M, K, N, case.get("bits", 4))
    if kind in ("stack", "modulation"):
        return {"bytes": case["layers"] * by, "flops": case["layers"] * fl}
    if kind == "rotated":
        return {"bytes": by + 4 * K * case["b"] + 4 * K + M * K * case["bits"] // 8 + 4 * M, "flops": fl + 2 * M * K * case["b"]}
    if case["split"]:
        by += M * K * case["bits"] // 8 + 4 * M
    by += 4 * K * ((case["fold"] in ("before", "both")) + (case["fold"] in ("after", "both"))) + (4 * N if case["bias"] else 0)
    return {"bytes": by, "flops": fl}


def tolerance(case):
    if case["kind"] == "gptq":
        # another correct factor differs in its last bits, and torch's gave the same codes; one code that falls the other way on a
        # near-tie carries into later columns of its row (a few hundred of a million codes)
        return {"rel": 1e-6, "differ": 1e-3}
    if case["kind"] == "modulation":
        # fp32 sums in another order: 3e-5 against sums in 64 bits; a bf16 step is up to 2^-7 of a value
        return {"rel": 1.2e-4, "max": 2.4e-2}
    # codes, scales and integer sums are fixed bit for bit; the rescale's factors in another order took a few bf16 results to their
    # neighbours: 1.4e-5 at most
    return {"rel": 6e-5, "max": 2.4e-2, "differ": 0.0}


# ---------------------------------------------------------------- the same in 64 bits

def _butterfly(x, b):
    """Unnormalized Sylvester transform of consecutive blocks of b, in float64."""
    z = x.double()
    M, K = z.shape
    h = 1
    while h < b:
        z = z.reshape(M, K // (2 * h), 2, h)
        z = torch.stack((z[:, :, 0] + z[:, :, 1], z[:, :, 0] - z[:, :, 1]), dim=2).reshape(M, K)
        h *= 2
    return z


def _round(z, bits, clip, cb):
    """Symmetric per-row rounding: codes (float64 integers) and the row's scale."""
    q = 2 ** (bits - 1) - 1
    a = z.abs().amax(dim=1, keepdim=True) * clip
    codes = torch.clamp(torch.round(z * torch.where(a > 0, q / a, torch.zeros_like(a))), -q, q)
    return codes, (a * cb / q)[:, 0]


def _projection64(x, w, b, bits, clip=1.0, s=None, p=None, bias=None):
    cb = 1.0 / math.sqrt(b)
    pre = None if s is None else (1.0 / s).double()
    post = None if p is None else (1.0 / p).double()
    zx = _butterfly(x.double() if pre is None else x.double() * pre, b)
    zw = _butterfly(w.double() if s is None else w.double() * s.double(), b)
    a, delta = _round(zx if post is None else zx * post, bits, clip, cb)
    c, scale = _round(zw if p is None else zw * p.double(), bits, 1.0, cb)
    y = (a @ c.t()) * (delta[:, None] * scale[None, :])
    return delta, y if bias is None else y + bias.double()


def exact(case, seed):
    kind = case["kind"]
    if kind == "linear":
        p = _linear_inputs(case, seed)
        delta, y = _projection64(p["x"], p["w"], case["b"], case["bits"], case["clip"], p["s"], p["p"], p["bias"])
        return {"codes": None, "delta": delta, "y": y} if case["split"] else y
    if kind in ("expert", "backbone"):
        sites = _expert_sites(case) if kind == "expert" else _backbone_sites(case)
        steps = case["steps"] if kind == "expert" else 1
        got = []
        for (xs, w), (_, _, bits) in zip(_site_inputs(case, seed, sites, steps), sites):
            ys = [_projection64(x, w, case["b"], bits)[1] for x in xs]
            got.append(torch.stack(ys) if kind == "expert" else ys[0])
        return got
    if kind == "stack":
        return torch.stack([_projection64(x, w, case["b"], case["bits"])[1] for x, w in _stack_inputs(case, seed)])
    if kind == "modulation":
        got = []
        for x, w in _stack_inputs(case, seed):
            c, scale = _round(w.double(), 4, 1.0, 1.0)
            got.append((x.double() @ c.t()) * scale[None, :])
        return torch.stack(got)
    if kind == "rotated":
        p = _rotated_inputs(case, seed)
        b, bits = case["b"], case["bits"]

        def rotate(v):
            v = v.double()[:, p["perm"].long()]
            z = torch.empty_like(v)
            for k in range(v.shape[1] // b):
                z[:, k * b:(k + 1) * b] = v[:, k * b:(k + 1) * b] @ p["blocks"][k].double().t().contiguous()
            return z
        a, delta = _round(rotate(p["x"]), bits, 1.0, 1.0)
        c, scale = _round(rotate(p["w"]), bits, 1.0, 1.0)
        return {"codes": None, "delta": delta, "y": (a @ c.t()) * (delta[:, None] * scale[None, :])}
    p = _gptq_inputs(case, seed)
    _, scale = _round(_butterfly(p["w"], case["b"]), case["bits"], 1.0, 1.0 / math.sqrt(case["b"]))
    return {"codes": None, "scale": scale, "packed": None}
