"""The calls a program makes of this library, at the sizes it makes them.

Three kinds of call ("op"):
  forward  MoELayer.forward: route, mixed-precision expert FFN, combine, over
           a packed layer (decode at a few tokens, prefill at thousands)
  switch   MoELayer.switch_dataset: requantize every cached channel at new
           per-expert precisions and install the copy mask
  pack     api.moe_quant_pack: quantize and pack one fp32 expert matrix
"""
from __future__ import annotations

import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2503_21135_amd import MoELayer, api

# Layer shapes and bit-width recipes: (bits, share of the routed experts).
# "pool": cached channels per routed expert and kind; switched on: "on".
FAMILIES = {
    "tiny": dict(d=256, E=8, S=0, k=2, f=512, fs=0, group=64, mixed=((8, .25), (4, .5), (2, .25)),
                 pool=1.0, on=0.10, t_max=2048),
    "tiny128": dict(d=256, E=8, S=1, k=2, f=512, fs=256, group=128,
                    mixed=((8, .125), (6, .5), (4, .125), (3, .125), (2, .125)), pool=1.0, on=0.10, t_max=2048),
    "mixtral": dict(d=4096, E=8, S=0, k=2, f=14336, fs=0, group=128, mixed=((8, .25), (4, .5), (2, .25)),
                    pool=0.05, on=0.05, t_max=4096),
    "deepseek": dict(d=2048, E=64, S=2, k=6, f=1408, fs=1408, group=128,
                     mixed=((8, .20), (4, .50), (3, .15), (2, .15)), pool=0.05, on=0.05, t_max=8192),
    "qwen": dict(d=2048, E=60, S=1, k=4, f=1408, fs=5632, group=128,
                 mixed=((8, .20), (4, .50), (3, .15), (2, .15)), pool=0.10, on=0.06, t_max=4096),
}


def listed():
    def fwd(name, family, T, bits="mixed", zipf=0.0):
        return {"name": name, "op": "forward", "family": family, "T": T, "bits": bits, "zipf": zipf}
    return [
        # the smallest call: one token through a test-sized layer (launch latency)
        fwd("tiny 1", "tiny", 1),
        # single-stream generation: one token, two wide experts' weights read
        fwd("mixtral 1", "mixtral", 1),
        # batched generation, the headline decode step
        fwd("mixtral 64", "mixtral", 64),
        # a chunk of a prompt, ragged
        fwd("mixtral 333", "mixtral", 333),
        # prompt processing with skewed expert loads
        fwd("mixtral 4096", "mixtral", 4096, zipf=1.1),
        # a small ragged decode batch over many narrow experts
        fwd("deepseek 17", "deepseek", 17),
        # batched generation over many narrow experts and shared ones
        fwd("deepseek 128", "deepseek", 128),
        # prompt processing over many narrow experts
        fwd("deepseek 8192", "deepseek", 8192),
        # a large generation batch on a layer with a partly switched channel pool
        fwd("qwen 512", "qwen", 512),
        # the unquantized 16-bit layer the packed one is compared with
        fwd("deepseek bf16 128", "deepseek", 128, bits="16"),
        # a new dataset arrives: cached channels requantized, mask installed
        {"name": "mixtral switch", "op": "switch", "family": "mixtral"},
        # loading a layer: one expert's gate matrix quantized at 4 bits
        {"name": "pack 14336x4096 b4", "op": "pack", "R": 14336, "K": 4096, "b": 4, "group": 128},
    ]


def draw(rng):
    op = rng.choices(("forward", "switch", "pack"), (8, 1, 1))[0]
    if op == "pack":
        group = rng.choice((64, 128))
        return {"op": op, "R": round(math.exp(rng.uniform(math.log(512), math.log(14336)))),
                "K": 128 * rng.randint(2, 64), "b": rng.choice((2, 4, 8) if group == 64 else (2, 3, 4, 6, 8)),
                "group": group}
    family = rng.choice(sorted(FAMILIES))
    if op == "switch":
        return {"op": op, "family": family, "epoch": rng.randint(0, 1000)}
    F = FAMILIES[family]
    T = round(math.exp(rng.uniform(0.0, math.log(F["t_max"]))))
    bits = rng.choice(("mixed",) * 7 + (("8", "4", "2", "16") if F["group"] == 64 else ("8", "6", "4", "3", "2", "16")))
    return {"op": op, "family": family, "T": T, "bits": bits, "zipf": rng.choice((0.0, 0.0, round(rng.uniform(0.3, 1.2), 2)))}


# ------------------------------------------------------------------ inputs
def _rand(seed, stream):
    return torch.Generator(device="cuda").manual_seed(1_000_003 * (int(seed) + 1) + stream)


def _expert_bits(F, bits, r):
    E = F["E"]
    if bits != "mixed":
        return np.full(E, int(bits), np.int32)
    n = [int(round(p * E)) for _, p in F["mixed"]]
    n[1] += E - sum(n)
    seq = [b for (b, _), c in zip(F["mixed"], n) for _ in range(c)]
    return np.asarray(seq, np.int32)[r.permutation(E)]


class LayerInputs:
    """What MoELayer takes: the shapes, fp32 weights N(0, 0.02^2), router,
    per-expert bit-widths and cached channels of one layer.  The matrices are
    windows of one random block, at an offset of their own each."""

    def __init__(self, family, bits, seed, epoch=0):
        F = self.F = FAMILIES[family]
        unq = bits == "16"
        E, S, d, f, fs = F["E"], F["S"], F["d"], F["f"], F["fs"]
        r = self.r = np.random.default_rng([int(seed), 17])
        self.epoch = epoch
        self.cfg = SimpleNamespace(n_experts=E, n_shared=S, top_k=F["k"], d_model=d, d_ff=f, d_ff_shared=fs,
                                   group=64 if unq else F["group"],
                                   rows=lambda kind, e: d if kind == 2 else (f if e < E else fs),
                                   cols=lambda kind, e: d if kind != 2 else (f if e < E else fs))
        self.bits = np.concatenate([_expert_bits(F, bits, r), np.full(S, 16 if unq else 8, np.int32)]).astype(np.int32)
        self.router = r.standard_normal((E, d), dtype=np.float32) * np.float32(0.02)
        size = d * max(f, fs)
        self.slack = size // 4
        block = torch.empty(size + self.slack, device="cuda").normal_(0.0, 0.02, generator=_rand(seed, 1))
        self.block = torch.empty(block.shape, pin_memory=True).copy_(block)
        self._hdr = []
        for kind in range(3):
            R = self.cfg.rows(kind, 0)
            n = 0 if unq else int(round(F["pool"] * R))
            rows = [np.sort(r.choice(R, n, replace=False)) for _ in range(E)]
            self._hdr.append(np.stack([np.repeat(np.arange(E), n), np.concatenate(rows)], 1).astype(np.int32))

    def window(self, block, expert, kind):
        R, K = self.cfg.rows(kind, expert), self.cfg.cols(kind, expert)
        o = (expert * 3 + kind) * 100_003 * 4 % self.slack
        return block[o:o + R * K].view(R, K)

    def weight(self, expert, kind):
        return self.window(self.block, expert, kind).numpy()

    def copy_headers(self, kind):
        return self._hdr[kind]

    def slots_on(self, kind, epoch=0):
        F, E, R = self.F, self.cfg.n_experts, self.cfg.rows(kind, 0)
        n = len(self._hdr[kind]) // E
        m = min(n, int(round(F["on"] * R)))
        r = np.random.default_rng([epoch, kind, 23])
        return np.concatenate([e * n + np.sort(r.choice(n, m, replace=False)) for e in range(E)]).astype(np.int32)

    def channel_cache(self, kind):
        h = self._hdr[kind]
        n = len(h) // self.cfg.n_experts
        return np.concatenate([self.weight(e, kind)[h[e * n:(e + 1) * n, 1]].astype(np.float16)
                               for e in range(self.cfg.n_experts)]).view(np.uint16)


def _tokens(F, T, seed):
    """bf16 activations N(0, 1), one input column in a hundred scaled by 20."""
    x = torch.randn(T, F["d"], device="cuda", generator=_rand(seed, 2))
    cols = torch.randperm(F["d"], device="cuda", generator=_rand(seed, 3))[:max(1, F["d"] // 100)]
    x[:, cols] *= 20.0
    return x.to(torch.bfloat16)


def _zipf_bias(x, router, k, s):
    """Router bias that moves the expert loads toward Zipf(s)."""
    E = router.shape[0]
    base = x.double() @ router.double().t()
    tgt = (torch.arange(E, device=x.device) + 1.0).double() ** -s
    tgt /= tgt.sum()
    b = torch.zeros(E, dtype=torch.float64, device=x.device)
    for _ in range(20):
        load = torch.bincount((base + b).topk(k, 1).indices.flatten(), minlength=E).double() / (x.shape[0] * k)
        b += (tgt / load.clamp_min(1e-6)).log()
    return b.float()


def _state(case, seed):
    if case["op"] == "pack":
        w = torch.empty(case["R"], case["K"], device="cuda").normal_(0.0, 0.02, generator=_rand(seed, 1))
        return SimpleNamespace(op="pack", w=w)
    inputs = LayerInputs(case["family"], case.get("bits", "mixed"), seed, case.get("epoch", 0))
    if case["op"] == "switch":
        new = _expert_bits(inputs.F, "mixed", np.random.default_rng([int(seed), 29]))
        return SimpleNamespace(op="switch", inputs=inputs, new_bits=new)
    x = _tokens(inputs.F, case["T"], seed)
    router = torch.from_numpy(inputs.router).cuda()
    bias = _zipf_bias(x, router, inputs.F["k"], case["zipf"]) if case["zipf"] else None
    return SimpleNamespace(op="forward", inputs=inputs, x=x, bias=bias, router=router)


def prepare(case, seed):
    st = _state(case, seed)
    if st.op == "pack":
        R, K, b, g = case["R"], case["K"], case["b"], case["group"]
        st.b, st.group = b, g
        st.ld = api.moe_code_row_words(K, b)
        st.codes = torch.zeros(R, st.ld, dtype=torch.int32, device="cuda")
        st.sz = torch.zeros(K // g, R, dtype=torch.int32, device="cuda")
        return st
    st.layer = MoELayer(st.inputs)
    if st.op == "switch":
        for kind in range(3):
            st.layer.channel_cache(kind)
    else:
        st.layer.set_epoch(0)
        st.layer.buffers(case["T"])
    st.inputs.block = None   # packed: the fp32 weights are not kept
    return st


def run(state):
    if state.op == "forward":
        return state.layer.forward(state.x, state.bias)
    if state.op == "pack":
        R, K = state.w.shape
        api.moe_quant_pack(state.w, state.b, state.group, state.codes, state.sz, ld_codes=state.ld,
                           sz_row_stride=1, sz_group_stride=R)
        return {"codes": state.codes[:, :K * state.b // 32], "sz": state.sz}
    L = state.layer
    L.switch_dataset(state.new_bits, state.inputs.epoch)
    out = {"order_gu": L.order_gu, "order_dn": L.order_dn, "class_cnt": L.class_cnt}
    for kind, kd in enumerate(L.kinds):
        n, K = kd["n_slots"], L.cfg.cols(kind, 0)
        rw = api.moe_code_row_words(K, 8)
        out["codes%d" % kind] = kd["copy_codes"][:n * rw].view(n, rw)[:, :K // 4]
        out["sz%d" % kind] = kd["copy_sz"][:n * (K // L.cfg.group)]
        out["row_slot%d" % kind] = kd["row_slot"]
    return out


# ------------------------------------------------------------------ work
def work(case):
    if case["op"] == "pack":
        n = case["R"] * case["K"]
        return {"bytes": 4 * n + n * case["b"] // 8 + 4 * n // case["group"], "flops": 2 * n}
    F = FAMILIES[case["family"]]
    d, E, S, k, f, fs, g = (F[n] for n in ("d", "E", "S", "k", "f", "fs", "group"))
    if case["op"] == "switch":
        n = sum(E * round(F["pool"] * R) * K for R, K in ((f, d), (f, d), (d, f)))
        return {"bytes": 3 * n + 4 * n // g + 4 * E * (2 * (2 * f + d) + f + d), "flops": 2 * n}
    T, bits = case["T"], case["bits"]
    on = 0.0 if bits == "16" else F["on"]
    mean = sum(b * p for b, p in F["mixed"]) if bits == "mixed" else float(bits)
    reached = E * (1.0 - (1.0 - k / E) ** T)
    sz = 0.0 if bits == "16" else 4.0 / g
    per = ((1.0 - on) * mean + on * 8) / 8 + sz
    weights = 3 * d * (reached * f * per + S * fs * ((2.0 if bits == "16" else 1.0) + sz))
    return {"bytes": weights + 4 * E * d + T * d * 6, "flops": 6.0 * d * T * (k * f + S * fs) + 2.0 * T * E * d}


def tolerance(case):
    """Packing and requantization are defined bit for bit.  A layer's output
    carries one rounding of the hidden values to bf16, whose flips under
    another summation order move it by up to 2e-4, and at prefill sizes one
    fp16 rounding per weight (1.0e-3 to 1.2e-3 against exact weights); two
    such results differ by at most 1.7e-3."""
    return {"rel": 2e-3} if case["op"] == "forward" else "exact"


# ------------------------------------------------------------------ 64 bits
def _quantize(w, b, g):
    """(codes, scale, zero) of rows of w in binary64: scale the smallest
    binary16 that is at least (max - min) / (2^b - 1), integer zero point."""
    G = w.double().view(w.shape[0], -1, g)
    mn, mx = G.amin(2).clamp_max(0.0), G.amax(2).clamp_min(0.0)
    s = (mx - mn) / (2 ** b - 1)
    h = s.half()
    h = torch.where(h.double() < s, (h.view(torch.int16) + 1).view(torch.half), h)
    h = torch.where(s == 0, torch.ones_like(h), h)
    sd = h.double()
    z = torch.round(-mn / sd)
    q = (torch.round(G / sd[..., None]) + z[..., None]).clamp_(0, 2 ** b - 1)
    return q, sd, z, h


def _dequantized(w, b, g):
    if b == 16:
        return w.to(torch.bfloat16).double()
    q, s, z, _ = _quantize(w, b, g)
    return (q.sub_(z[..., None]).mul_(s[..., None])).view(w.shape)


def _half_split(q, b):
    """Codes [..., 32/b] of each word -> the word (even codes in the low half)."""
    word = torch.zeros(q.shape[:-1], dtype=torch.int64, device=q.device)
    for i in range(q.shape[-1]):
        word |= q[..., i] << ((i >> 1) * b + 16 * (i & 1))
    return word


def _words(q, b):
    """Packed words [R][K*b/32] of integer codes [R][K]."""
    R = q.shape[0]
    q = q.to(torch.int64)
    if b in (3, 6):
        q = q.view(R, -1, 32)
        low = b - b // 3                      # 2 or 4 low bits, then the rest
        n = 32 // low
        parts = [_half_split((q[..., i:i + n] & (2 ** low - 1)), low) for i in range(0, 32, n)]
        n = 32 // (b - low)
        parts += [_half_split(q[..., i:i + n] >> low, b - low) for i in range(0, 32, n)]
        w = torch.stack(parts, -1)
    else:
        w = _half_split(q.view(R, -1, 32 // b), b)
    w = w.view(R, -1)
    return torch.where(w >= 2 ** 31, w - 2 ** 32, w).to(torch.int32)


def _sz_words(h, z):
    w = (h.view(torch.int16).to(torch.int64) & 0xFFFF) | ((z.half().view(torch.int16).to(torch.int64) & 0xFFFF) << 16)
    return torch.where(w >= 2 ** 31, w - 2 ** 32, w).to(torch.int32)


def exact(case, seed):
    st = _state(case, seed)
    if st.op == "pack":
        q, _, z, h = _quantize(st.w, case["b"], case["group"])
        return {"codes": _words(q.view(st.w.shape), case["b"]), "sz": _sz_words(h, z).t().contiguous()}
    inp, cfg = st.inputs, st.inputs.cfg
    block = inp.block.cuda()
    E, S, g = cfg.n_experts, cfg.n_shared, cfg.group
    if st.op == "switch":
        out, on = {}, []
        for kind in range(3):
            hdr, R = inp.copy_headers(kind), cfg.rows(kind, 0)
            codes, sz = [], []
            for e in range(E):
                rows = torch.from_numpy(hdr[hdr[:, 0] == e, 1]).long().cuda()
                q, _, z, h = _quantize(inp.window(block, e, kind)[rows].half(), int(st.new_bits[e]), g)
                codes.append(_words(q.view(len(rows), -1), 8))
                sz.append(_sz_words(h, z).flatten())
            out["codes%d" % kind], out["sz%d" % kind] = torch.cat(codes), torch.cat(sz)
            slots = inp.slots_on(kind, inp.epoch)
            rs = np.full(E * R, -1, np.int32)
            rs[hdr[slots, 0] * R + hdr[slots, 1]] = slots
            out["row_slot%d" % kind] = torch.from_numpy(rs)
            on.append((rs >= 0).reshape(E, R))
        cls = [on[0] + 2 * on[1], on[2].astype(int)]
        out["order_gu"], out["order_dn"] = (torch.from_numpy(np.argsort(c, 1, kind="stable").astype(np.int32).ravel())
                                            for c in cls)
        out["class_cnt"] = torch.from_numpy(np.concatenate(
            [np.stack([(c == j).sum(1) for j in range(4)], 1).ravel() for c in cls]).astype(np.int32))
        return out
    x = st.x.double()
    logits = x @ st.router.double().t()
    if st.bias is not None:
        logits += st.bias.double()
    val, ids = logits.topk(inp.F["k"], 1)
    wts = torch.softmax(val, 1)
    y = torch.zeros_like(x)
    for e in range(E + S):
        if e < E:
            t, j = (ids == e).nonzero(as_tuple=True)
            wt = wts[t, j]
        else:
            t, wt = torch.arange(x.shape[0], device="cuda"), torch.ones(x.shape[0], dtype=torch.float64, device="cuda")
        if len(t) == 0:
            continue
        W = []
        for kind in range(3):
            w = inp.window(block, e, kind)
            dq = _dequantized(w, int(inp.bits[e]), g)
            hdr = inp.copy_headers(kind)
            rows = hdr[inp.slots_on(kind, 0)] if len(hdr) else hdr
            rows = torch.from_numpy(rows[rows[:, 0] == e, 1]).long().cuda()
            if len(rows):
                dq[rows] = _dequantized(w[rows], 8, g)
            W.append(dq)
        xe = x[t]
        gate = xe @ W[0].t()
        hid = (torch.nn.functional.silu(gate) * (xe @ W[1].t())).to(torch.bfloat16).double()
        y.index_add_(0, t, wt[:, None] * (hid @ W[2].t()))
    return y
