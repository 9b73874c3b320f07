"""Performance cases of the MiKV mixed-precision KV cache on one MI355X.

Four kinds of work, one attention layer each, through the package's public
entry points:

  importance  mikv_prefill_importance: the H2O scores of a prompt;
  fill        MikvDecoder.prefill with given scores: balancer (where used),
              first selection, quantization of the prompt into both pools;
  attend      mikv_decode_attention on a filled cache, both pools'
              probabilities emitted;
  decode      a generation: the prompt placed with given scores, then `steps`
              whole decode steps (mikv_decode_step, importance fused).  A step
              changes the cache, so a pass starts from an emptied one, as a
              serving loop reuses a cache's buffers for the next prompt.

Shapes and precisions are those of paper_2402_18096_amd.workloads and of the
test and precision-variant tables, plus ragged lengths.
"""
from __future__ import annotations

import math

import torch

from paper_2402_18096_amd import mikv, workloads

D = 128
SCALE = 1.0 / math.sqrt(128.0)
DEV = "cuda"


def _case(name, kind, batch, q_heads, kv_heads, context, hi=16, lo=2, group=32, num=1, den=10, window=64,
          in_ratio=True, balanced=False, k_dist="normal", kv_outliers=4, kv_scale=10.0, q_outliers=0, q_scale=1.0,
          steps=0, key_block=0):
    c = dict(kind=kind, batch=batch, q_heads=q_heads, kv_heads=kv_heads, context=context, hi=hi, lo=lo, group=group,
             num=num, den=den, window=window, in_ratio=in_ratio, balanced=balanced, k_dist=k_dist,
             kv_outliers=kv_outliers, kv_scale=kv_scale, q_outliers=q_outliers, q_scale=q_scale, steps=steps,
             key_block=key_block)
    if name:
        c["name"] = name
    return c


_LLAMA13 = dict(hi=8, lo=2, group=32, num=1, den=5, window=64, balanced=True, k_dist="student_t4", kv_outliers=0,
                kv_scale=1.0, q_outliers=4, q_scale=10.0)
_LLAMA7 = dict(hi=8, lo=4, group=64, num=1, den=4, window=64)
_MISTRAL = dict(hi=16, lo=2, group=32, num=1, den=10, window=128, kv_outliers=8, kv_scale=20.0)
_LONG = dict(hi=16, lo=2, group=32, num=1, den=10, window=128)


def listed():
    return [
        # Scores of a served batch's prompts: a 7B layer, 4096 tokens each.
        _case("importance_7b", "importance", 8, 32, 32, 4096),
        # The same for long prompts under GQA (the mistral_7b workload's prompt): the largest call.
        _case("importance_gqa_16k", "importance", 16, 32, 8, 16384, kv_outliers=8, kv_scale=20.0),
        # One interactive request with a short prompt of no round length.
        _case("importance_ragged", "importance", 1, 40, 40, 1531),
        # A large batch's prompts into the cache, balanced keys, INT8 + INT2 (the llama2_13b workload).
        _case("fill_13b", "fill", 32, 40, 40, 8192, **_LLAMA13),
        # Few long prompts into an fp16 + INT2 cache (the long_context workload).
        _case("fill_long", "fill", 4, 32, 32, 32768, **_LONG),
        # Attention for a single sequence of no round length, INT3 retained pool: one request being decoded.
        _case("attend_int3_b1", "attend", 1, 40, 40, 5003, hi=16, lo=3, group=64, num=1, den=5, window=33),
        # Attention with eight query heads per KV head (the 70B head layout), INT8 + INT2, ragged length.
        _case("attend_gqa8", "attend", 4, 64, 8, 7001, hi=8, lo=2, group=64, num=1, den=5, window=64),
        # The smallest generation: 4 heads, 512 tokens; launches and latency (the tiny workload).
        _case("decode_tiny", "decode", 1, 4, 4, 512, hi=16, lo=2, group=32, num=1, den=5, window=32, in_ratio=False,
              steps=16),
        # The ordinary generation: a 7B layer, batch 8, 4096 tokens (the llama2_7b workload and its 64 steps).
        _case("decode_7b", "decode", 8, 32, 32, 4096, steps=64, **_LLAMA7),
        # The largest cache by bytes, balanced INT8 + INT2 (the llama2_13b workload and its 32 steps).
        _case("decode_13b", "decode", 32, 40, 40, 8192, steps=32, **_LLAMA13),
        # GQA with long contexts (the mistral_7b workload).
        _case("decode_mistral", "decode", 16, 32, 8, 16384, steps=64, **_MISTRAL),
        # The longest context (the long_context workload, the benchmark's default).
        _case("decode_long", "decode", 4, 32, 32, 32768, steps=64, **_LONG),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case: every kind, head layout, precision and option the cache has, sizes over the listed range."""
    kind = rng.choice(("importance", "fill", "attend", "decode", "decode"))
    G = rng.choice((1, 1, 1, 2, 4, 8))
    kv_heads = rng.choice((4, 8, 32, 40) if G == 1 else (4, 8))
    if kind == "importance":
        T = _log_int(rng, 64, 16384)
        most = max(1, (1 << 34) // (kv_heads * G * T * T))
        return _case(None, kind, _log_int(rng, 1, min(32, most)), kv_heads * G, kv_heads, T)
    T = _log_int(rng, 300, 32768)
    B = _log_int(rng, 1, min(32, max(1, (1 << 21) // (kv_heads * T))))
    hi, lo = rng.choice(((16, 2), (16, 2), (8, 2), (8, 4), (16, 4), (16, 3), (4, 2), (16, 0)))
    num, den = rng.choice(((1, 4), (1, 5), (1, 10)))
    window = rng.choice((32, 33, 64, 128))
    key_block = 64 if G == 1 and hi == 16 and lo in (2, 3, 4) and window >= 64 and rng.random() < 0.4 else 0
    balanced = not key_block and rng.random() < 0.3
    steps = _log_int(rng, 4, 32) if kind == "decode" else 0
    out = dict(k_dist="student_t4", kv_outliers=0, kv_scale=1.0, q_outliers=4, q_scale=10.0) if balanced else {}
    return _case(None, kind, B, kv_heads * G, kv_heads, T, hi=hi, lo=lo, group=rng.choice((32, 64)), num=num, den=den,
                 window=window, in_ratio=rng.random() < 0.7, balanced=balanced, steps=steps, key_block=key_block, **out)


# -- inputs -----------------------------------------------------------------------

def _workload(c, seed):
    return workloads.Workload("case", c["batch"], c["q_heads"], c["kv_heads"], c["context"], max(1, c["steps"]),
                              c["hi"], c["lo"], c["group"], c["num"], c["den"], c["window"], c["in_ratio"],
                              c["balanced"], c["k_dist"], c["kv_outliers"], c["kv_scale"], c["q_outliers"],
                              c["q_scale"], 1 + int(seed) % (1 << 40), key_block=c["key_block"])


def _scores(wl):
    """Seeded Zipf(1.1) scores per head over a random order of the positions (as workloads.initial_scores, drawn on the GPU)."""
    g = torch.Generator(device=DEV)
    g.manual_seed(wl.seed * 16 + 9)
    n = wl.context
    base = torch.arange(1, n + 1, dtype=torch.float64, device=DEV).pow(-1.1)
    base = (base * (n / base.sum())).float()
    order = torch.rand(wl.batch, wl.kv_heads, n, generator=g, device=DEV).argsort(dim=-1)
    return base[order].contiguous()


def prepare(case, seed):
    wl = _workload(case, seed)
    kind = case["kind"]
    s = {"kind": kind, "wl": wl}
    if kind == "importance":
        s["k"] = workloads.prefill_kv(wl, DEV)[0]
        s["q"] = workloads.prefill_queries(wl, DEV)
        s["scores"] = torch.empty(wl.batch, wl.kv_heads, wl.context, dtype=torch.float32, device=DEV)
        n = mikv.lib().mikv_prefill_importance_workspace_size(wl.batch, wl.q_heads, wl.context)
        s["ws"] = torch.empty(n, dtype=torch.uint8, device=DEV)
        return s
    s["dec"] = mikv.MikvDecoder(wl, max_len=wl.context + case["steps"], device=DEV, fused=True)
    s["k"], s["v"] = workloads.prefill_kv(wl, DEV)
    s["sc"] = _scores(wl)
    s["qp"] = workloads.prefill_queries(wl, DEV) if wl.balanced else None
    s["q"], s["kn"], s["vn"] = workloads.decode_inputs(wl, max(1, case["steps"]), DEV)
    if kind == "attend":
        s["dec"].prefill(s["k"], s["v"], s["sc"], s["qp"])
    if kind == "decode":
        s["outs"] = torch.empty(case["steps"], wl.batch, wl.q_heads, D, dtype=torch.float32, device=DEV)
    return s


def _fill(s):
    """The prompt into the cache, whose buffers are used again: its pools are emptied first."""
    dec = s["dec"]
    dec.cache.n_hi.zero_()
    dec.cache.n_lo.zero_()
    dec.prefill(s["k"], s["v"], s["sc"], s["qp"])


def run(s):
    kind = s["kind"]
    if kind == "importance":
        mikv.mikv_prefill_importance(s["q"], s["k"], s["scores"], SCALE, s["ws"])
        return {"scores": s["scores"]}
    dec = s["dec"]
    c, wl = dec.cache, s["wl"]
    if kind == "attend":
        lo = dec.probs_lo if c.lo_bits else None
        mikv.mikv_decode_attention(c, dec.length, s["q"][0], dec.out, dec.probs_hi, lo, dec.balance, SCALE, 0,
                                   dec.attn_ws)
        return {"out": dec.out, "probs_hi": dec.probs_hi, "probs_lo": lo}
    _fill(s)
    if kind == "fill":
        # rows of the pools are compared as stored words; unused ones are what the buffers were made with
        return {"balance": dec.balance, "hi_acc": c.hi_acc, "hi_k": c.hi_k, "hi_v": c.hi_v, "hi_kp": c.hi_kp,
                "hi_vp": c.hi_vp, "hi_pos": c.hi_pos, "lo_k": c.lo_k, "lo_v": c.lo_v, "lo_kp": c.lo_kp,
                "lo_vp": c.lo_vp, "lo_kb": c.lo_kb, "lo_pos": c.lo_pos, "n_hi": c.n_hi, "n_lo": c.n_lo, "map": c.map}
    lo = dec.probs_lo if c.lo_bits else None
    for t in range(s["outs"].shape[0]):
        dec.length += 1
        L = dec.length
        mikv.mikv_decode_step(c, L, s["q"][t], s["kn"][t], s["vn"][t], s["outs"][t], dec.k_heavy(L), wl.window,
                              dec.probs_hi, lo, dec.balance, SCALE, mikv.ATTN_ACCUMULATE, dec.step_ws)
    words = lambda x: x.view(torch.int16) if x.dtype == torch.float16 else x  # fp16 rows as the words they are
    return {"out": s["outs"], "hi_acc": c.hi_acc, "hi_k": words(c.hi_k), "hi_v": words(c.hi_v), "hi_kp": c.hi_kp,
            "hi_vp": c.hi_vp, "hi_pos": c.hi_pos, "lo_k": c.lo_k, "lo_v": c.lo_v, "lo_kp": c.lo_kp, "lo_vp": c.lo_vp,
            "lo_pos": c.lo_pos, "n_hi": c.n_hi, "n_lo": c.n_lo, "map": c.map}


# -- what a pass cannot do without ----------------------------------------------------

def _budget(c, L):
    k = c["num"] * L // c["den"] - (c["window"] if c["in_ratio"] else 0)
    return max(0, k)


def _token_bytes(c, bits):
    if bits == 0:
        return 0
    if bits == 16:
        return 4 * D
    codes = D * bits // 8
    key = codes + (4 * D // c["key_block"] if c["key_block"] else 4 * (D // c["group"]))
    return key + codes + 4 * (D // c["group"])


def work(case):
    c = case
    NH, BQ, T = c["batch"] * c["kv_heads"], c["batch"] * c["q_heads"], c["context"]
    if c["kind"] == "importance":
        # one causal Q K^T
        return {"bytes": 2 * D * T * (NH + BQ) + 4 * NH * T, "flops": 2 * D * BQ * T * (T + 1) // 2}

    def packed(L):
        n_hi = min(L, _budget(c, L) + min(L, c["window"]))
        return NH * (n_hi * _token_bytes(c, c["hi"]) + (L - n_hi) * _token_bytes(c, c["lo"])), n_hi

    def step(L):  # the packed cache, the probabilities and the output
        kv, n_hi = packed(L)
        n = L if c["lo"] else n_hi
        return kv + 4 * BQ * n + 4 * BQ * D + 2 * BQ * D, 4 * D * BQ * n

    if c["kind"] == "attend":
        b, f = step(T)
        return {"bytes": b, "flops": f}
    n_hi = packed(T)[1]
    n = T if c["lo"] else n_hi
    fill = 4 * D * NH * T + 4 * NH * T + packed(T)[0] + 4 * NH * n + 4 * NH * n_hi + NH * T
    if c["balanced"]:
        fill += 2 * D * BQ * T + 4 * NH * D
    if c["kind"] == "fill":
        return {"bytes": fill, "flops": 4 * D * NH * T}
    flops = 0
    for t in range(c["steps"]):
        b, f = step(T + 1 + t)
        fill += b + 4 * D * NH
        flops += f
    return {"bytes": fill, "flops": flops}


def tolerance(case):
    """About four times the largest distance from `exact` that the cases show, drawn ones among them."""
    if case["kind"] == "fill":
        return "exact"  # codes, scales, fp16 rows and positions are defined bit for bit
    if case["kind"] == "importance":
        return {"rel": 4e-5, "max": 1e-3}
    if case["kind"] == "attend":
        return {"rel": 1.3e-4, "max": 5e-3}
    # A near-tie of two scores at the cut may fall the other way under another order of summation: the two
    # tokens then trade precision and slots, which shows in a few stored words (a larger share of a small
    # cache) and slightly in the outputs that follow.
    return {"rel": 1e-4, "max": 0.1, "differ": min(0.01, 1e-4 + 1.0 / (64 * case["batch"] * case["kv_heads"]))}


# -- the same in 64 bits, in plain torch -------------------------------------------------

def _exact_importance(q, k):
    B, Hq, T, _ = q.shape
    G = Hq // k.shape[1]
    out = torch.zeros(B, k.shape[1], T, dtype=torch.float64, device=q.device)
    rows = max(64, min(T, (1 << 28) // T // max(1, min(Hq, 8))))
    step = max(1, min(Hq, 8) // G)  # KV heads at a time
    for b in range(B):
        for h0 in range(0, k.shape[1], step):
            h1 = min(k.shape[1], h0 + step)
            kk = k[b, h0:h1].double()
            qq = q[b, h0 * G:h1 * G].double().reshape(h1 - h0, G, T, D)
            for i0 in range(0, T, rows):
                i1 = min(T, i0 + rows)
                x = qq[:, :, i0:i1].reshape(h1 - h0, G * (i1 - i0), D) @ kk[:, :i1].transpose(1, 2).contiguous()
                x = (x * SCALE).reshape(h1 - h0, G, i1 - i0, i1)
                x[..., i0:].masked_fill_(
                    torch.ones(i1 - i0, i1 - i0, dtype=torch.bool, device=q.device).triu(1), -math.inf)
                out[b, h0:h1, :i1] += torch.softmax(x, dim=-1).sum(dim=(1, 2))
    return out


def _quantized(x, bits, group):
    """Eq. 1 of fp32 rows [..., 128]: the decoded values in 64 bits (alpha * code + beta, alpha and beta fp16)."""
    g = x.reshape(*x.shape[:-1], D // group, group)
    mn, mx = g.amin(-1, keepdim=True), g.amax(-1, keepdim=True)
    return _decoded(g, mn, mx, bits).reshape(x.shape)


def _decoded(x, mn, mx, bits):
    top = float((1 << bits) - 1)
    # (through 64 bits: torch divides a GPU tensor by a number with a multiplication)
    a, b = ((mx - mn).double() / top).float().half().float(), mn.half().float()
    code = torch.where(a == 0, torch.zeros_like(x), torch.clamp(torch.round((x - b) / a), 0, top))
    return a.double() * code.double() + b.double()


class _ExactCache:
    """Keys and values by position, decoded, in 64 bits; scores in 64 bits."""

    def __init__(self, c, k, v, scores, qp):
        self.c, T = c, c["context"]
        self.NH, self.G = c["batch"] * c["kv_heads"], c["q_heads"] // c["kv_heads"]
        self.max_len = T + c["steps"]
        z = lambda *s, dt: torch.zeros(*s, dtype=dt, device=k.device)
        self.K, self.V = (z(self.NH, self.max_len, D, dt=torch.float64) for _ in range(2))
        self.raw = z(self.NH, self.max_len, D, dt=torch.float16) if c["key_block"] else None
        self.is_hi, self.live = (z(self.NH, self.max_len, dt=torch.bool) for _ in range(2))
        self.acc = z(self.NH, self.max_len, dt=torch.float64)
        self.balance = None
        if c["balanced"]:
            qm = qp.abs().amax(2).reshape(c["batch"], c["kv_heads"], self.G, D).amax(2).double()
            km = k.abs().amax(2).double()
            self.balance = torch.where((qm == 0) | (km == 0), torch.ones_like(qm), (qm / km).sqrt()).float()
        k, v = k.reshape(self.NH, T, D), v.reshape(self.NH, T, D)
        sc = scores.reshape(self.NH, T)
        hi = torch.zeros(self.NH, T, dtype=torch.bool, device=k.device)
        thr = max(0, T - c["window"])
        kh = min(thr, _budget(c, T))
        if kh > 0:
            hi.scatter_(1, sc[:, :thr].topk(kh, dim=1).indices, True)
        hi[:, thr:] = True
        self.is_hi[:, :T], self.live[:, :T], self.acc[:, :T] = hi, hi | (c["lo"] != 0), sc.double()
        if self.raw is not None:
            self.raw[:, :T] = k
        for h0 in range(0, self.NH, 64):  # some heads at a time: the temporaries are 64-bit
            h = slice(h0, min(self.NH, h0 + 64))
            kf = self._balanced(k[h].float(), h)
            m = hi[h].unsqueeze(-1)
            lk, lv = self._low(kf, None, h), self._low(v[h].float(), True, h)
            self.K[h, :T] = torch.where(m, self._high(kf), lk)
            self.V[h, :T] = torch.where(m, self._high(v[h].float()), lv)
        self.length = T

    def _balanced(self, kf, h=slice(None)):
        return kf if self.balance is None else kf * self.balance.reshape(self.NH, 1, D)[h]

    def _high(self, x):
        return x.half().double() if self.c["hi"] == 16 else _quantized(x, self.c["hi"], self.c["group"])

    def _low(self, x, is_v, h):
        c = self.c
        if not c["lo"]:
            return torch.zeros_like(x, dtype=torch.float64)
        if is_v or not c["key_block"]:
            return _quantized(x, c["lo"], c["group"])
        n = x.shape[1] // 64 * 64  # whole blocks; the others are in the window
        b = x[:, :n].reshape(x.shape[0], n // 64, 64, D)
        lo = _decoded(b, b.amin(2, keepdim=True), b.amax(2, keepdim=True), c["lo"]).reshape(x.shape[0], n, D)
        return torch.cat([lo, x[:, n:].double()], 1)

    def attend(self, q):
        c, L = self.c, self.length
        qh = q.double().reshape(self.NH, self.G, D)
        if self.balance is not None:
            qh = qh / self.balance.double().reshape(self.NH, 1, D)
        s = torch.empty(self.NH, self.G, L, dtype=torch.float64, device=q.device)
        o = torch.empty(self.NH, self.G, D, dtype=torch.float64, device=q.device)
        s = torch.matmul(self.K[:, :L], qh.transpose(1, 2).contiguous()).transpose(1, 2) * SCALE
        s = s.masked_fill(~self.live[:, None, :L], -math.inf)
        p = torch.softmax(s, dim=-1)
        o = torch.matmul(p, self.V[:, :L])
        return o.reshape(c["batch"], c["q_heads"], D), p

    def step(self, q, kn, vn):
        c, L = self.c, self.length
        kf = self._balanced(kn.reshape(self.NH, 1, D).float())
        vf = vn.reshape(self.NH, 1, D).float()
        self.K[:, L:L + 1], self.V[:, L:L + 1] = self._high(kf), self._high(vf)
        if self.raw is not None:
            self.raw[:, L] = kn.reshape(self.NH, D)
        self.is_hi[:, L] = self.live[:, L] = True
        self.length = L = L + 1
        o, p = self.attend(q)
        self.acc[:, :L] += p.sum(1)
        thr = max(0, L - c["window"])
        elig = self.is_hi[:, :L].clone()
        elig[:, thr:] = False
        n_dem = int(elig[0].sum()) - _budget(c, L)  # every head holds the same counts
        if n_dem > 0:
            key = torch.where(elig, self.acc[:, :L], torch.full_like(self.acc[:, :L], math.inf))
            idx = key.topk(n_dem, dim=1, largest=False).indices
            rows = torch.arange(self.NH, device=q.device)[:, None]
            self.is_hi[rows, idx] = False
            if not c["lo"]:
                self.live[rows, idx] = False
            else:
                self.V[rows, idx] = _quantized(self.V[rows, idx].float(), c["lo"], c["group"])
                if c["key_block"]:
                    blk = self.raw[rows[..., None], (idx // 64 * 64)[..., None] + torch.arange(64, device=q.device)]
                    blk = blk.float()
                    self.K[rows, idx] = _decoded(self.K[rows, idx].float(), blk.amin(2), blk.amax(2), c["lo"])
                else:
                    self.K[rows, idx] = _quantized(self.K[rows, idx].float(), c["lo"], c["group"])
        return o


def exact(case, seed):
    c = case
    s = prepare(case, seed)
    if c["kind"] == "importance":
        return {"scores": _exact_importance(s["q"], s["k"])}
    dec = s["dec"]
    cache = dec.cache
    if c["kind"] == "fill":
        acc = None
        cap, T = cache.cap_hi, c["context"]
        e = _ExactCache(dict(c, steps=0), s["k"][:, :, :, :], s["v"], s["sc"], s["qp"])
        order = torch.where(e.is_hi, torch.arange(T, device=DEV), T).sort(dim=1).values[:, :cap]
        acc = torch.zeros(e.NH, cap, dtype=torch.float64, device=DEV)
        padded = torch.cat([e.acc, torch.zeros(e.NH, 1, dtype=torch.float64, device=DEV)], 1)
        acc[:, :order.shape[1]] = padded.gather(1, order)
        none = ("hi_k", "hi_v", "hi_kp", "hi_vp", "hi_pos", "lo_k", "lo_v", "lo_kp", "lo_vp", "lo_kb", "lo_pos",
                "n_hi", "n_lo", "map")
        bal = None if e.balance is None else (
            s["qp"].abs().amax(2).reshape(c["batch"], c["kv_heads"], e.G, D).amax(2).double()
            / s["k"].abs().amax(2).double()).sqrt()
        return {"balance": bal, "hi_acc": acc, **{n: None for n in none}}
    e = _ExactCache(c, s["k"], s["v"], s["sc"], s["qp"])
    if c["kind"] == "attend":
        o, p = e.attend(s["q"][0])
        got = {"out": o, "probs_hi": None, "probs_lo": None}
        p = p.reshape(e.NH, e.G, -1)
        for name, hi, cap in (("probs_hi", True, cache.cap_hi), ("probs_lo", False, cache.cap_lo)):
            if not hi and not c["lo"]:
                continue
            T = c["context"]
            # tokens lie in their pool in position order
            order = torch.where(e.is_hi == hi, torch.arange(T, device=DEV), T).sort(dim=1).values[:, :cap]
            padded = torch.cat([p, torch.zeros(e.NH, e.G, 1, dtype=torch.float64, device=DEV)], 2)
            rows = torch.zeros(e.NH, e.G, cap, dtype=torch.float64, device=DEV)
            rows[:, :, :order.shape[1]] = padded.gather(2, order[:, None].expand(-1, e.G, -1))
            got[name] = rows.reshape(c["batch"], c["q_heads"], cap)
        return got
    outs = [e.step(s["q"][t], s["kn"][t], s["vn"][t]) for t in range(c["steps"])]
    none = ("hi_acc", "hi_k", "hi_v", "hi_kp", "hi_vp", "hi_pos", "lo_k", "lo_v", "lo_kp", "lo_vp", "lo_pos", "n_hi",
            "n_lo", "map")
    return {"out": torch.stack(outs), **{n: None for n in none}}
