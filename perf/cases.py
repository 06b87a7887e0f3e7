"""The work that a user of this library has it do, as cases that can be timed and compared.

Four kinds of pass, all through the public entry points (MoeLayer, and the moe_* calls of the binding):

  layer   one MoE layer, forward or forward + backward, bf16 or fp32 storage, with the library's options (permutations
          folded into the GEMMs, activation recomputation, either GeLU, capacity overflow)
  dtd     the local halves of duplicate token dropping on one rank of a tensor-parallel group: its dispatch share, the
          expert FFN from the all-gathered shares, combine, and the drop of the gradient shares
  adamw   the mixed-precision AdamW step over a group of expert parameters, up-cast in registers or staged in tiles

The large shapes are the layers of the paper's base models (1.3B, 2.7B, 6.7B, 13B, 16 experts) as `synth.WORKLOADS` lists
them; tokens are whole 2048-token sequences in training and whatever a batch holds in serving.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2303_06318_amd import moe, synth
from paper_2303_06318_amd.layer import MoeLayer

# How far a token leans to "its" expert, in standard deviations of the logits: a trained router separates tokens, so
# that few of them are near ties, and spreads them about evenly over the experts.
LEAN = 4.0
TILE = 1_800_000          # the paper's optimizer tile (parameters)


def _layer(name, T, h, E, f, cf, *, dtype="bf16", act="erf", backward=False, fused=False, recompute=False, skew=False):
    c = {"kind": "layer", "T": T, "h": h, "E": E, "f": f, "cf": cf, "dtype": dtype, "act": act, "backward": backward,
         "fused": fused, "recompute": recompute, "skew": skew}
    return {"name": name, **c} if name else c


def _workload(name, key, **options):
    w = synth.WORKLOADS[key]
    return _layer(name, w.T, w.h, w.E, w.f, w.capacity_factor, dtype=w.dtype, backward=options.pop("backward", w.backward),
                  skew=w.zipf_bias, **options)


def _dtd(name, T, h, E, f, cf, G):
    c = {"kind": "dtd", "T": T, "h": h, "E": E, "f": f, "cf": cf, "tp": G}
    return {"name": name, **c} if name else c


def _adamw(name, n, dtype, staged, ts):
    c = {"kind": "adamw", "n": n, "dtype": dtype, "staged": staged, "ts": ts}
    return {"name": name, **c} if name else c


def listed():
    return [
        # a unit-test sized layer in fp32: nothing but launches and host work
        _workload("tiny_f32_train", "cfg1_tiny_f32", backward=True),
        # a validation run in full precision: a small model trained in fp32 to compare against
        _layer("f32_train", 2048, 1024, 8, 1024, 1.25, dtype="f32", backward=True),
        # serving: a small batch of tokens through the 1.3B base's experts, every expert's weights read for a few rows
        _layer("serve_100_tokens", 100, 2048, 16, 8192, 2.0, fused=True),
        # inference over four sequences with the 1.3B base's layer, the three calls
        _workload("fwd_1p3b", "cfg2_1p3b_fwd"),
        # inference over eight sequences with a 6.7B shard, permutations folded into the GEMMs
        _workload("fwd_6p7b_fused", "cfg3_6p7b_tp4_fwd", fused=True),
        # an untrained or collapsed router: nearly all tokens want a few of 64 experts and overflow them
        _workload("fwd_skewed", "cfg4_skewed_fwd"),
        # training, one sequence per micro-batch (what a memory-limited run uses): 128 rows per expert on average
        _layer("train_1p3b_1seq", 2048, 2048, 16, 8192, 1.25, backward=True),
        # training, eight sequences, the 6.7B shard: the benchmark's own workload
        _workload("train_6p7b", "cfg5_6p7b_tp4_fwdbwd"),
        # training with activation recomputation, the 13B shard (sizes that no tile divides), tanh GeLU, fused combine
        _workload("train_13b_recompute", "cfg7_13b_tp8_fwdbwd", act="tanh", fused=True, recompute=True),
        # one rank of a tensor-parallel group of 4 under duplicate token dropping, two sequences of the 6.7B shard
        _dtd("dtd_6p7b_tp4", 4096, 4096, 16, 4096, 1.25, 4),
        # the optimizer step over a layer's expert parameters, up-cast in registers ...
        _adamw("adamw_register", 1 << 26, "bf16", False, 1 << 26),
        # ... and with the paper's tile of 1.8 M parameters staged in fp32
        _adamw("adamw_staged", 1 << 25, "bf16", True, TILE),
    ]


def _log_int(rng, lo, hi, multiple=1):
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / multiple)) * multiple
    return min(max(v, lo), hi)


def draw(rng):
    kind = rng.choice(["fwd", "fwd", "train", "train", "train", "f32", "dtd", "adamw"])
    act = rng.choice(["erf", "erf", "tanh"])
    if kind == "adamw":
        staged = rng.random() < 0.4
        n = _log_int(rng, 1 << 20, 1 << 25 if staged else 1 << 26)
        return _adamw(None, n, rng.choice(["bf16", "bf16", "bf16", "f32"]), staged, rng.choice([TILE, 8 * TILE]))
    if kind == "f32":
        h, f = _log_int(rng, 64, 1024, 4), _log_int(rng, 64, 1024, 4)
        return _layer(None, _log_int(rng, 64, 2048), h, rng.choice([2, 4, 8]), f, rng.choice([1.0, 1.25, 2.0]), dtype="f32",
                      act=act, backward=rng.random() < 0.7)
    E = rng.choice([4, 8, 16, 16, 16, 32, 64])
    while True:                      # no more weights than 16 experts of 2048 x 8192, no more work than the 6.7B shard's
        h, f = _log_int(rng, 1024, 5144, 8), _log_int(rng, 1024, 8192, 8)
        if E * h * f <= 1 << 28:
            break
    most = min(16384, (1 << 38) // (h * f))
    cf = rng.choice([1.0, 1.25, 1.25, 2.0])
    if kind == "dtd":
        return _dtd(None, _log_int(rng, 1024, min(most, 8192)), h, E, f, 1.25, rng.choice([2, 4, 8]))
    if kind == "train":
        return _layer(None, _log_int(rng, 1024, most), h, E, f, cf, act=act, backward=True, fused=rng.random() < 0.4,
                      recompute=rng.random() < 0.25)
    return _layer(None, _log_int(rng, 64, most), h, E, f, cf, act=act, fused=rng.random() < 0.5, skew=rng.random() < 0.25)


def _cap(c):
    return int(math.ceil(c["cf"] * c["T"] / c["E"]))


class _State:
    pass


def _randn(gen, shape, std, dtype):
    out = torch.empty(shape, dtype=dtype, device="cuda")
    flat = out.view(-1)
    step = 1 << 26                   # drawn in fp32 and rounded, a piece at a time
    for i in range(0, flat.numel(), step):
        n = min(step, flat.numel() - i)
        flat[i:i + n] = torch.randn(n, generator=gen, device="cuda", dtype=torch.float32).mul_(std)
    return out


def _tokens(gen, c, w_gate, dtype):
    """Standard normal tokens; with an even router every token leans to an expert of its own."""
    x = _randn(gen, (c["T"], c["h"]), 1.0, torch.float32)
    if not c.get("skew"):
        towards = torch.nn.functional.normalize(w_gate, dim=0).t().contiguous()
        x += LEAN * towards[torch.randint(c["E"], (c["T"],), generator=gen, device="cuda")]
    return x.to(dtype)


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    s = _State()
    s.case = c = case
    if c["kind"] == "adamw":
        s.dtype = moe.MOE_BF16 if c["dtype"] == "bf16" else moe.MOE_F32
        td = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
        s.grad = _randn(gen, (c["n"],), 1e-3, td)
        s.grad[seed % 97::97] = 0
        s.master = _randn(gen, (c["n"],), 0.02, torch.float32)
        s.m = _randn(gen, (c["n"],), 3e-4, torch.float32)
        s.v = _randn(gen, (c["n"],), 1e-3, torch.float32).square_()
        s.param = s.master.to(td)
        s.staging = torch.empty(min(c["ts"], c["n"]), dtype=torch.float32, device="cuda") if c["staged"] else None
        s.hp = moe.make_adamw(lr=1e-4, beta1=0.9, beta2=0.95, eps=1e-8, weight_decay=0.1, step=100)
        return s
    f32 = c.get("dtype") == "f32"
    td = torch.float32 if f32 else torch.bfloat16
    T, h, E, f, C = c["T"], c["h"], c["E"], c["f"], _cap(c)
    s.w_gate = _randn(gen, (h, E), 0.02, torch.float32)
    s.x = _tokens(gen, c, s.w_gate, td)
    s.w1 = _randn(gen, (E, h, f), 0.02, td)
    s.w2 = _randn(gen, (E, f, h), 0.02, td)
    s.bias = torch.from_numpy(synth.zipf_logit_bias(E)).cuda() if c.get("skew") else None
    if c["kind"] == "dtd":
        # the all-gathered shares that the collective hands this rank, and the upstream gradient of its chunks
        s.layer = L = MoeLayer(T, h, E, f, C, moe.MOE_BF16)
        G, Cg = c["tp"], (C + c["tp"] - 1) // c["tp"]
        s.shares = torch.empty((G, E, Cg, h), dtype=td, device="cuda")
        s.share = torch.empty((E, Cg, h), dtype=td, device="cuda")
        s.d_share = torch.zeros((E, Cg, h), dtype=td, device="cuda")
        s.d_buf = _randn(gen, (E, C, h), 1.0, td)
        L.gate(s.x, s.w_gate)
        for r in range(G):
            moe.moe_dispatch_dtd(L.shape, s.x, L.token_of_slot, r, G, s.shares[r])
        s.share.zero_()              # rows of empty slots stay as they are: zeros here
        return s
    s.layer = MoeLayer(T, h, E, f, C, moe.MOE_F32 if f32 else moe.MOE_BF16,
                       moe.MOE_GELU_TANH if c["act"] == "tanh" else moe.MOE_GELU_ERF, backward=c["backward"],
                       recompute=c["recompute"])
    s.d_out = _randn(gen, (T, h), 1.0, td) if c["backward"] else None
    return s


def run(s):
    c = s.case
    if c["kind"] == "adamw":
        moe.moe_adamw_tiled(c["n"], c["ts"], s.hp, s.grad, s.master, s.m, s.v, s.param, s.staging, s.dtype)
        return [s.master, s.m, s.v, s.param]
    L = s.layer
    if c["kind"] == "dtd":
        L.gate(s.x, s.w_gate)
        moe.moe_dispatch_dtd(L.shape, s.x, L.token_of_slot, 0, c["tp"], s.share)
        moe.moe_expert_ffn_fwd_dtd(L.shape, s.shares, c["tp"], s.w1, s.w2, L.kept, None, L.hact, L.y, L.ws)
        moe.moe_combine(L.shape, L.y, L.expert, L.slot, L.gate_p, L.out)
        moe.moe_dtd_drop(L.shape, s.d_buf, L.kept, 0, c["tp"], s.d_share)
        return {"logits": L.logits, "expert": L.expert, "share": s.share, "out": L.out, "d_share": s.d_share}
    L.forward(s.x, s.w_gate, s.w1, s.w2, logit_bias=s.bias, fused=c["fused"])
    got = {"logits": L.logits, "expert": L.expert, "gate_p": L.gate_p, "out": L.out}
    if c["backward"]:
        L.backward(s.d_out, s.x, s.w_gate, s.w1, s.w2)
        got.update(d_x=L.d_x, d_w1=L.d_w1, d_w2=L.d_w2, d_w_gate=L.d_w_gate)
    return got


def _kept(c):
    """Expected kept tokens and experts that hold any, from a small sample of the router's logits."""
    rng = np.random.default_rng(0)
    E, T, sigma = c["E"], c["T"], 0.02 * math.sqrt(c["h"])
    if not c.get("skew"):
        share = np.full(E, 1.0 / E)
    else:
        top = np.argmax(sigma * rng.standard_normal((20000, E)) + synth.zipf_logit_bias(E), axis=1)
        share = np.bincount(top, minlength=E) / 20000.0
    mean, sd = T * share, np.sqrt(T * share * (1 - share))
    counts = np.clip(np.rint(mean[:, None] + sd[:, None] * rng.standard_normal((E, 64))), 0, T)
    return float(np.minimum(counts, _cap(c)).sum(0).mean()), float((counts > 0).sum(0).mean())


def work(case):
    c = case
    if c["kind"] == "adamw":
        z = 2 if c["dtype"] == "bf16" else 4
        return {"bytes": c["n"] * (z + 12 + 12 + z), "flops": c["n"] * 16}
    z = 4 if c.get("dtype") == "f32" else 2
    T, h, E, f = c["T"], c["h"], c["E"], c["f"]
    kept, active = _kept(c)
    tokens, weights, gate = T * h * z, 2 * h * f * z, h * E * 4 + T * (4 * E + 8)
    if c["kind"] == "dtd":
        rows = kept * h * z
        # shares in, one share of the dispatch and of the gradient out
        return {"bytes": 2 * tokens + rows + 3 * rows / c["tp"] + active * weights + gate, "flops": 4 * h * f * kept + 2 * T * h * E}
    b, n = 2 * tokens + active * weights + gate, 4 * h * f * kept + 2 * T * h * E
    if c["backward"]:
        b += 2 * tokens + E * weights + h * E * 4
        n += 8 * h * f * kept + 4 * T * h * E
    return {"bytes": b, "flops": n}


def tolerance(case):
    """Measured against the same pass in 64 bits on the path's own inputs, times about four: fp32 storage rel 9e-7 and
    6e-6 of the rms at most, bf16 storage rel 3.7e-3 and 0.048.  "differ" leaves room for near ties of the router."""
    if case["kind"] == "adamw":
        # fp32 state updated in place; the bf16 copy of a weight may round the other way (2^-8 of the value)
        return {"rel": 1e-5, "max": 1e-2}
    if case.get("dtype") == "f32":
        return {"rel": 1e-5, "max": 1e-4, "differ": 1e-3}
    return {"rel": 1.2e-2, "max": 0.15, "differ": 1e-3}
