"""The work users of this framework have it do, as timed cases.

Every case goes through the package's public entry points (`runtime.Session`, `runtime.LadderSession`,
`runtime.TieredSession`, `binding.pac_dequant_linear*`) the way a training program calls them: the activation cache is
filled and the parameters are set beforehand, one pass is one call on the next batch of a seeded epoch order.
Sizes are the workloads of `paper_2408_10746_amd.inputs` and of the tests, or generic.
"""
import math

import numpy as np
import torch

from paper_2408_10746_amd import binding as pb
from paper_2408_10746_amd.inputs import Workload, outlier_channels
from paper_2408_10746_amd.runtime import LadderSession, Session, TieredSession

DEV = "cuda:0"


def listed():
    return [
        # the smallest run people start with: fp32 cache, short epochs; a few dozen launches of little work
        dict(name="train_tiny_f32", kind="train", dtype="f32", L=4, d=256, n_max=64, len_lo=0, B=8, r=32, C=2, N=64),
        # a small model on ragged sentences, four at a time: every tile has a remainder
        dict(name="train_small_ragged", kind="train", dtype="bf16", L=5, d=128, n_max=70, len_lo=20, B=4, r=64, C=3, N=64),
        # T5-Base-shaped adapters on 128-token sentences: the ordinary training step
        dict(name="train_t5base", kind="train", dtype="bf16", L=12, d=768, n_max=128, len_lo=0, B=32, r=96, C=3, N=256),
        # validation between epochs: forward only, ragged sentences, the odd batch that an epoch ends with
        dict(name="eval_t5base_ragged", kind="eval", dtype="bf16", L=12, d=768, n_max=128, len_lo=17, B=29, r=96, C=3, N=232),
        # the same adapters trained from an fp32 cache, the precision the paper trains in
        dict(name="train_t5base_f32", kind="train", dtype="f32", L=12, d=768, n_max=128, len_lo=0, B=32, r=96, C=3, N=128),
        # BART/T5-Large-shaped adapters
        dict(name="train_large", kind="train", dtype="bf16", L=24, d=1024, n_max=128, len_lo=0, B=32, r=128, C=2, N=128),
        # LLaMA-7B-shaped adapters, with the outlier channels such hidden states have
        dict(name="train_llama7b", kind="train", dtype="bf16", L=32, d=4096, n_max=256, len_lo=0, B=16, r=256, C=4, N=64,
             outliers=True),
        # the largest: long ragged documents, wide adapters
        dict(name="train_longseq", kind="train", dtype="bf16", L=32, d=4096, n_max=1024, len_lo=256, B=8, r=512, C=2, N=24),
        # the ladder of reduced transformer layers, T5-Base-shaped
        dict(name="ladder_t5base", kind="ladder", dtype="bf16", L=12, d=768, n_max=128, len_lo=0, B=32, r=96, C=3, N=128,
             heads=12),
        # the first epoch's cache fill: one batch of fp32 hidden states of ragged sentences, rounded and packed
        dict(name="fill_t5base_ragged", kind="fill", dtype="bf16", L=12, d=768, n_max=128, len_lo=17, B=32),
        # the first epoch's linear layer on 8-bit weights: one 4096 x 4096 projection of 4096 tokens
        dict(name="linear_int8", kind="linear", M=4096, K=4096, N=4096, block=64, bits=8),
        # a cache in host memory: the next batch is reloaded while this one trains
        dict(name="tier_t5base", kind="tier", dtype="bf16", L=12, d=768, n_max=128, len_lo=0, B=32, r=96, C=3, N=64),
    ]


def _log_int(rng, lo, hi, step=1):
    x = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return int(min(hi, max(lo, round(x / step) * step)))


def _tokens(c):
    """Expected valid tokens of one batch."""
    return c["B"] * (c["n_max"] if c["len_lo"] <= 0 else (c["len_lo"] + c["n_max"]) / 2)


def draw(rng):
    kind = rng.choice(["train"] * 5 + ["eval", "f32", "ladder", "ladder", "fill", "linear", "linear", "tier"])
    while True:
        c = _draw_one(rng, kind)
        w = work(c)
        # no dearer than the listed cases of the same kind
        most = {"train": 1.5e12, "eval": 0.5e12, "f32": 6e10, "ladder": 6e10, "fill": 1e12, "linear": 1.4e11, "tier": 1e11}[kind]
        if w["flops"] <= most and w["bytes"] <= 6e8:
            return c


def _draw_one(rng, kind):
    if kind == "linear":
        block = rng.choice([32, 64, 64, 128, 256])
        c = dict(kind="linear", M=_log_int(rng, 16, 4096), K=max(1, _log_int(rng, 256, 4096) // block) * block,
                 N=_log_int(rng, 64, 4096), block=block, bits=rng.choice([8, 4]))
        if rng.random() < 0.4:  # straight into the cache, as one layer of a backbone would
            c.update(kind="linear_to_cache", N=max(32, c["N"] // 32 * 32), n_max=_log_int(rng, 16, 256), dtype="bf16")
            c["B"] = max(1, min(64, c.pop("M") // c["n_max"]))
            c["len_lo"] = rng.choice([0, max(1, c["n_max"] // 4)])
        return c
    n_max = _log_int(rng, 16, 1024)
    B = _log_int(rng, 1, 32)
    while B * n_max > 8192:
        n_max //= 2
    c = dict(kind="train" if kind == "f32" else kind, dtype="bf16", L=_log_int(rng, 2, 32), d=_log_int(rng, 128, 4096, 32),
             n_max=n_max, len_lo=rng.choice([0, max(1, n_max // 4), max(1, n_max // 2)]), B=B)
    if kind == "fill":
        c["dtype"] = rng.choice(["bf16", "bf16", "f32"])
        return c
    c["r"] = min(512, max(32, round(c["d"] / rng.choice([4, 8, 8, 16]) / 32) * 32))
    c["C"] = rng.choice([2, 3, 4, 5])
    c["N"] = B * rng.choice([2, 3, 4])
    if kind == "f32":
        c["dtype"] = "f32"
    if kind == "ladder":
        c["dtype"] = rng.choice(["bf16", "bf16", "f32"])
        c["d"] = _log_int(rng, 128, 1024, 32)
        c["r"] = min(256, max(32, round(c["d"] / rng.choice([4, 8, 8]) / 32) * 32))
        c["n_max"] = min(c["n_max"], 256)
        c["len_lo"] = min(c["len_lo"], c["n_max"] // 2)
        c["heads"] = c["r"] // rng.choice([h for h in (4, 8, 16, 32, 64) if c["r"] % h == 0 and c["n_max"] * h <= 4096])
    return c


# ---- inputs -----------------------------------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _workload(c):
    return Workload("case", L=c["L"], d=c["d"], n_max=c["n_max"], B=c["B"], r=c.get("r", 32), C=c.get("C", 2),
                    N=c.get("N", c["B"]), cache_dtype=c["dtype"], len_lo=c["len_lo"],
                    outlier_frac=0.01 if c.get("outliers") else 0.0)


def _lengths(c, n, rng):
    """Lengths spread evenly over [len_lo, n_max], in the seed's order: every seed packs the same number of tokens."""
    return None if c["len_lo"] <= 0 else rng.permutation(np.linspace(c["len_lo"], c["n_max"], n).round().astype(np.int32))


def _hidden(c, w, count, gen):
    """Hidden states as a layer norm leaves them: zero mean, unit variance per token, a few large channels where asked."""
    a = torch.randn((count, c["L"], c["n_max"], c["d"]), generator=gen, device=DEV)
    a = torch.nn.functional.layer_norm(a, (c["d"],), eps=1e-5)
    if w.outlier_frac:
        a[..., torch.from_numpy(outlier_channels(1234, c["d"], w.outlier_frac)).to(DEV)] *= w.outlier_scale
    return a.contiguous()


def _fill(sess, c, w, lens, gen):
    chunk = max(1, min(32, c["B"], (1 << 28) // (c["L"] * c["n_max"] * c["d"])))
    for s0 in range(0, c["N"], chunk):
        ids = np.arange(s0, min(c["N"], s0 + chunk))
        sess.cache_fill(ids, _hidden(c, w, len(ids), gen), None if lens is None else lens[ids])


def _adapter_params(w, p, gen):
    """A partly trained side network: N(0, 1/fan_in) projections, the up-projections smaller, gates spread around 0.5."""
    p.normal_(generator=gen)
    d, r, n = w.d, w.r, w.layer_block
    layers = p[:w.L * n].view(w.L, n)
    layers[:, :d * r] *= d ** -0.5
    layers[:, d * r:d * r + r] *= 0.1
    layers[:, d * r + r:2 * d * r + r] *= 0.3 * r ** -0.5
    layers[:, 2 * d * r + r:-1] *= 0.1
    layers[:, -1] = 0.5 + 0.1 * layers[:, -1]
    p[w.L * n:] *= d ** -0.5


def _ladder_params(w, p, gen):
    p.normal_(generator=gen)
    d, r = w.d, w.r
    sizes = [(d * r, d ** -0.5, 0), (r, 0.1, 0), (r, 0.1, 1), (r, 0.1, 0), (3 * r * r, r ** -0.5, 0), (3 * r, 0.1, 0),
             (r * r, r ** -0.5, 0), (r, 0.1, 0), (r, 0.1, 1), (r, 0.1, 0), (4 * r * r, r ** -0.5, 0), (4 * r, 0.1, 0),
             (4 * r * r, (4 * r) ** -0.5, 0), (r, 0.1, 0), (1, 0.1, 0.5), (3, 0, 0)]
    n = sum(s for s, _, _ in sizes)
    layers, at = p[:w.L * n].view(w.L, n), 0
    for size, scale, offset in sizes:
        layers[:, at:at + size] = layers[:, at:at + size] * scale + offset
        at += size
    p[w.L * n:w.L * n + r * d] *= 0.3 * r ** -0.5
    p[w.L * n + r * d:] *= d ** -0.5


class _Batches:
    """A seeded epoch order, its batches' labels already on the GPU."""

    def __init__(self, c, rng):
        order = rng.permutation(c["N"]).astype(np.int64)
        self.ids = [order[k:k + c["B"]] for k in range(0, c["N"] - c["B"] + 1, c["B"])]
        self.labels = [torch.from_numpy(rng.integers(0, c["C"], size=c["B"], dtype=np.int32)).to(DEV) for _ in self.ids]
        self.k = 0

    def at(self, k):
        return self.ids[k % len(self.ids)], self.labels[k % len(self.ids)]


def prepare(case, seed):
    c, rng, gen = case, np.random.default_rng(seed), _gen(seed)
    kind = c["kind"]
    if kind in ("linear", "linear_to_cache"):
        W = torch.randn((c["N"], c["K"]), generator=gen, device=DEV) * c["K"] ** -0.5
        codes = torch.empty(c["N"] * c["K"] * c["bits"] // 8, dtype=torch.int8, device=DEV)
        consts = torch.empty(c["N"] * c["K"] // c["block"], device=DEV)
        stream = torch.cuda.current_stream().cuda_stream
        pb.pac_quant_blockwise(W.data_ptr(), W.numel(), c["block"], c["bits"], codes.data_ptr(), consts.data_ptr(), stream)
        rows = c["M"] if kind == "linear" else c["B"] * c["n_max"]
        s = dict(case=c, codes=codes, consts=consts,
                 x=torch.randn((rows, c["K"]), generator=gen, device=DEV).to(torch.bfloat16))
        if kind == "linear":
            s["y"] = torch.empty((rows, c["N"]), device=DEV)
        else:
            w = Workload("case", L=2, d=c["N"], n_max=c["n_max"], B=c["B"], r=32, C=2, N=c["B"], cache_dtype=c["dtype"])
            s["lens"], s["ids"] = _lengths(c, c["B"], rng), np.arange(c["B"])
            s["sess"] = Session(w, lens=s["lens"])
            s["sess"].cache.zero_()
        return s
    w = _workload(c)
    if kind == "fill":
        lens = _lengths(c, c["B"], rng)
        return dict(case=c, sess=Session(w, lens=lens), lens=lens, ids=np.arange(c["B"]), acts=_hidden(c, w, c["B"], gen))
    lens = _lengths(c, c["N"], rng)
    if kind == "ladder":
        sess = LadderSession(w, c["heads"], lens=lens)
        _ladder_params(w, sess.params, gen)
    else:
        sess = (TieredSession if kind == "tier" else Session)(w, lens=lens)
        _adapter_params(w, sess.params, gen)
    sess.hp = pb.pac_adamw(1e-4, 0.9, 0.999, 1e-8, 0.01)
    _fill(sess, c, w, lens, gen)
    s = dict(case=c, sess=sess, batches=_Batches(c, rng))
    if kind == "tier":
        sess.prefetch(0, s["batches"].at(0)[0])
    return s


def run(state):
    c = state["case"]
    kind, sess = c["kind"], state.get("sess")
    if kind == "linear":
        pb.pac_dequant_linear(state["x"].data_ptr(), c["M"], c["K"], state["codes"].data_ptr(), state["consts"].data_ptr(),
                              c["N"], c["block"], c["bits"], state["y"].data_ptr(), torch.cuda.current_stream().cuda_stream)
        return state["y"]
    if kind == "linear_to_cache":
        pb.pac_dequant_linear_to_cache(sess.ctx, sess.cache.data_ptr(), sess.cache_bytes, state["ids"], state["lens"], 1,
                                       state["x"].data_ptr(), c["K"], state["codes"].data_ptr(), state["consts"].data_ptr(),
                                       c["block"], c["bits"], torch.cuda.current_stream().cuda_stream)
        return sess.cache.view(torch.bfloat16)
    if kind == "fill":
        sess.cache_fill(state["ids"], state["acts"], state["lens"])
        return sess.cache
    b = state["batches"]
    ids, labels = b.at(b.k)
    if kind == "eval":
        sess.loss_grad(ids, labels, want_grads=False)
        out = [sess.loss, sess.logits[:c["B"] * c["C"]]]
    else:
        if kind == "tier":
            sess.prefetch(b.k + 1, b.at(b.k + 1)[0])
            sess.step_staged(b.k, ids, labels, keep_grads=False)
        else:
            sess.step(ids, labels, keep_grads=False)
        out = [sess.loss, sess.params, sess.m, sess.v]
    b.k += 1
    return out


# ---- what a pass cannot do without ----------------------------------------------------------------------------------

def work(case):
    c = case
    if c["kind"] in ("linear", "linear_to_cache"):
        rows = c["M"] if c["kind"] == "linear" else _tokens(c)
        weights = c["N"] * c["K"] * (c["bits"] / 8 + 4 / c["block"])
        out = 4 if c["kind"] == "linear" else 2
        return dict(bytes=rows * c["K"] * 2 + weights + rows * c["N"] * out, flops=2.0 * rows * c["N"] * c["K"])
    tokens = _tokens(c)
    size = 2 if c["dtype"] == "bf16" else 4
    values = tokens * c["L"] * c["d"]
    if c["kind"] == "fill":  # fp32 hidden states in, cache values out
        return dict(bytes=values * (4 + size), flops=0)
    d, r, L = c["d"], c["r"], c["L"]
    if c["kind"] == "ladder":
        params = L * (d * r + 12 * r * r + 13 * r) + r * d + d + (d + 1) * c["C"]
        per_token = L * (2.0 * d * r + 24.0 * r * r + 4.0 * r * tokens / c["B"])
        return dict(bytes=values * size + 24 * params, flops=3 * tokens * per_token)
    params = _workload(c).P
    if c["kind"] == "eval":  # cache slice and parameters in, logits out
        return dict(bytes=values * size + 4 * params, flops=4.0 * tokens * d * r * L)
    # cache slice in; parameters and both moments in and out
    return dict(bytes=values * size + 24 * params, flops=12.0 * tokens * d * r * L)


def tolerance(case):
    """About four times what was seen on an MI355X: fp32 paths with the batch in another order (so every token sum in
    another order), bf16 paths in their other formulations, the linear layer against float64.  A parameter whose
    gradient is next to nothing may step either way, hence the larger "max"."""
    c = case
    if c["kind"] == "fill":
        return "exact"
    if c["kind"] == "linear":  # fp32 sums
        return {"rel": 2e-6, "max": 2e-5}
    if c["kind"] == "linear_to_cache":  # those sums, now and then rounded to the other bf16 neighbour
        return {"rel": 2e-4, "max": 1e-2}
    if c["kind"] == "ladder" or c["dtype"] == "f32":  # fp32 throughout
        return {"rel": 1e-5, "max": 2e-3}
    return {"rel": 1.5e-2, "max": 0.8}  # bf16 operands, fp32 sums
