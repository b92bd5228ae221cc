"""Timed cases of libham: what a program asks of it, through its public entry points.

Four kinds of case, by the entry points that a pass calls:

* ``step``     one fused decode-attention step of a base layer (``ham_op_attention_step``): projection rows
               in, K and V appended, attention over the cache.  One row per sequence, ragged lengths.
* ``attn``     attention of one row per sequence over a cache that is already filled
               (``ham_op_decode_attention``).
* ``prefill``  a prompt batch through ``ham_prefill`` (token ids) or ``ham_prefill_embeds`` (input vectors at
               given positions): the time to the first group.
* ``decode``   a saved prefill continued by some macro-steps (``ham_state_restore`` + ``ham_macro_step``), as a
               server that forks sequences after a shared prompt; with ``prefill`` inside the pass when
               ``fresh`` is set (a whole request).

The models are the tiny, 1B and 8B shapes of ``synth.configs``; the 8B shape runs with fewer base layers, whose
kernels and sizes are those of all 32, so that its prompts take part of a second.  Decodes feed given tokens back
(teacher forcing), so that results stay comparable when two builds round differently; group lengths follow the
law of the benchmark schedules (1, 2, 1, 3, 1, 2, 1, 4, ...), with a last step of four tokens for everybody, so
that every decision's logits are an output.  ``exact`` computes the same in float64 with plain torch, K and V
rounded to the cache type as the model defines.
"""
import math

import torch

from paper_2505_20438_amd import ham

DEV = "cuda:0"
F32, BF16 = ham.HAM_F32, ham.HAM_BF16
CTX_ROWS = 4  # context rows of the micro decoder (fewer only where the base model has fewer layers)

SHAPES = {
    "tiny": dict(d=256, H=4, Hk=2, hd=64, F=704, V=1024, micro=1),
    "1b": dict(d=2048, H=32, Hk=8, hd=64, F=8192, V=128256, micro=2),
    "8b": dict(d=4096, H=32, Hk=8, hd=128, F=14336, V=128256, micro=2),
}
RULER = (1, 2, 1, 3, 1, 2, 1, 4)  # group lengths: the geometric law with p = 1/2, capped at 4


def listed():
    def model(name, kind, shape, layers, batch, prompt, **kw):
        return dict({"name": name, "kind": kind, "shape": shape, "layers": layers, "batch": batch, "prompt": prompt,
                     "dtype": "bf16", "steps": 0, "embeds": False, "fresh": False}, **kw)

    return [
        # the attention step of a single sequence of the 1B shape: the smallest call, launches and latency
        {"name": "step_1b_b1", "kind": "step", "dtype": "bf16", "rows": 1, "hd": 64, "kv": 700},
        # the same of a full ragged batch of the 8B shape
        {"name": "step_8b_b32", "kind": "step", "dtype": "bf16", "rows": 32, "hd": 128, "kv": 2560},
        # ... and of few sequences with long contexts (the dominant kernel of the long-context workload)
        {"name": "step_8b_long", "kind": "step", "dtype": "bf16", "rows": 4, "hd": 128, "kv": 33300},
        # attention over a filled cache of odd length, two sequences
        {"name": "attn_8b_b2", "kind": "attn", "dtype": "bf16", "rows": 2, "hd": 128, "kv": 1999},
        # a whole request to the tiny fp32 model: prompt of 64, 16 macro-steps; launch-bound
        model("request_tiny_f32", "decode", "tiny", 2, 1, 64, dtype="f32", steps=16, fresh=True),
        # time to the first group of a medium prompt, one sequence, all layers of the 1B shape
        model("prefill_1b_512", "prefill", "1b", 16, 1, 512),
        # a batch of short prompts of odd length (chat turns), all layers of the 1B shape
        model("prefill_1b_16x77", "prefill", "1b", 16, 16, 77),
        # a long document: 16 chunks of the prompt kernels at the 8B shape
        model("prefill_8b_32k", "prefill", "8b", 2, 1, 32768),
        # a batch of prompts given as input vectors at their own positions, odd chunk length
        model("prefill_8b_4x2000", "prefill", "8b", 3, 4, 2000, embeds=True),
        # generation of one sequence, all layers of the 1B shape: small launches in a chain
        model("decode_1b_b1", "decode", "1b", 16, 1, 512, steps=16),
        # generation with long contexts: attention reads most of the bytes
        model("decode_8b_long", "decode", "8b", 4, 4, 32768, steps=8),
        # batched generation, 8B shape
        model("decode_8b_b32", "decode", "8b", 4, 32, 2048, steps=8),
    ]


def draw(rng):
    def spread(lo, hi):  # over the logarithm, odd sizes among them
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(("step", "step", "attn", "prefill", "prefill", "prefill", "decode", "decode", "request"))
    dtype = "f32" if rng.random() < 0.2 else "bf16"
    if kind in ("step", "attn"):
        rows = spread(1, 64)
        return {"kind": kind, "dtype": dtype, "rows": rows, "hd": rng.choice((64, 128)),
                "kv": spread(40, min(33000, 130000 // rows))}
    c = {"kind": kind, "dtype": "bf16", "steps": 0, "embeds": False, "fresh": False}
    if kind == "request":
        c.update(kind="decode", shape="tiny", layers=rng.randint(2, 4), batch=spread(1, 16), prompt=spread(16, 900),
                 dtype=dtype, steps=rng.randint(2, 12), fresh=True)
    elif kind == "prefill":
        c.update(shape=rng.choice(("1b", "8b")), layers=rng.randint(2, 4), batch=spread(1, 32))
        c.update(prompt=spread(20, min(9000, 14000 // c["batch"])), embeds=rng.random() < 0.3)
    else:
        c.update(shape=rng.choice(("1b", "8b")), layers=rng.randint(2, 4), batch=spread(1, 64), steps=rng.randint(3, 8))
        c.update(prompt=spread(30, min(12000, 50000 // c["batch"])))
    return c


# ---------------------------------------------------------------- inputs
def _rng(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed) * 2 + 1)


def _dtype(case):
    return F32 if case["dtype"] == "f32" else BF16


def _attn_inputs(case, seed):
    """Rows, caches and lengths of one attention call (32 q-heads on 8 kv-heads, both shapes)."""
    g = _rng(seed)
    R, hd, kv, H, Hk = case["rows"], case["hd"], case["kv"], 32, 8
    t = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    S = (kv + 64) // 64 * 64 + 64
    # ragged: between four fifths of the longest and the longest, one sequence at the bound
    n = torch.randint(max(1, kv - kv // 5), kv + 1, (R,), generator=g, device=DEV, dtype=torch.int32)
    n[0] = kv

    def randn(*shape, to=torch.float32):
        return torch.randn(*shape, generator=g, device=DEV).to(to)

    s = {"R": R, "H": H, "Hk": Hk, "hd": hd, "S": S, "n": n, "on": torch.ones_like(n), "K": randn(R, Hk, S, hd, to=t),
         "V": randn(R, Hk, S // 32, hd, 32, to=t)}
    if case["kind"] == "step":
        a = torch.rand(R, hd // 2, generator=g, device=DEV) * 6.28
        s.update(qkv=randn(R, (H + 2 * Hk) * hd), cos=a.cos().contiguous(), sin=a.sin().contiguous(), slot=n - 1)
    else:
        s["q"] = randn(R, H * hd)
    return s


def _act(x, case):
    """fp32 or fp64 rows in the activation layout: as they are, or bf16 hi and lo planes."""
    if case["dtype"] == "f32":
        return x.contiguous()
    hi = x.float().to(torch.bfloat16).to(x.dtype)
    return torch.stack([hi, (x - hi).float().to(torch.bfloat16).to(x.dtype)], dim=1)


def _shape(case):
    return dict(SHAPES[case["shape"]], L=case["layers"], bf=case["dtype"] == "bf16")


def _lengths(case, step):
    B = case["batch"]
    if step and step == case["steps"]:
        return [4] * B
    return [RULER[(b + step) % 8] for b in range(B)]


def _model_inputs(case, seed):
    g = _rng(seed)
    B, P, s = case["batch"], case["prompt"], _shape(case)
    r = {"prompt": torch.randint(0, s["V"], (B, P), generator=g, device=DEV, dtype=torch.int32), "forced": [], "teacher": []}
    for step in range(case["steps"] + 1):
        r["forced"].append(torch.tensor(_lengths(case, step), dtype=torch.int32, device=DEV))
        r["teacher"].append(torch.randint(0, s["V"], (B, 4), generator=g, device=DEV, dtype=torch.int32))
    if case["embeds"]:
        r["rows"] = torch.randn(B, P, s["d"], generator=g, device=DEV) * 0.02
        r["pos"] = torch.cumsum(torch.randint(1, 5, (B, P), generator=g, device=DEV), 1).to(torch.int32) - 1
    return r


def _config(case):
    s = _shape(case)
    return ham.make_config(n_layers=s["L"], d_model=s["d"], n_heads=s["H"], n_kv_heads=s["Hk"], head_dim=s["hd"],
                           ffn_dim=s["F"], vocab=s["V"], micro_layers=s["micro"], stop_mode=ham.HAM_STOP_FORCED,
                           dtype=_dtype(case), max_batch=case["batch"],
                           max_prompt=case["prompt"] * (4 if case["embeds"] else 1),  # positions of groups of <= 4
                           max_steps=max(1, case["steps"]))


def _prefill(st):
    if "rows" in st:
        st["rt"].prefill_embeds(st["rows"], st["pos"], st["budget"], st["forced"][0], st["teacher"][0])
    else:
        st["rt"].prefill(st["prompt"], st["budget"], st["forced"][0], st["teacher"][0])


def prepare(case, seed):
    if case["kind"] in ("step", "attn"):
        s = _attn_inputs(case, seed)
        s["case"], s["dtype"] = case, _dtype(case)
        s["out"] = torch.zeros(s["R"], 2, s["H"] * s["hd"], dtype=s["K"].dtype, device=DEV)
        if case["dtype"] == "f32":
            s["out"] = s["out"][:, 0].contiguous()
        nb = ham.ham_op_attention_workspace_bytes(s["R"], s["H"], s["Hk"], s["hd"])
        s["ws"], s["err"] = torch.zeros(nb, dtype=torch.uint8, device=DEV), torch.zeros_like(s["n"])
        s["stream"] = torch.cuda.current_stream().cuda_stream
        if "q" in s:
            s["q"] = _act(s["q"], case).to(s["K"].dtype).contiguous()
        return s
    st = dict(_model_inputs(case, seed), case=case, budget=[0] * case["batch"])
    cfg, s, B = _config(case), _shape(case), case["batch"]
    rt = st["rt"] = ham.HamRuntime(cfg, int(seed), DEV)
    dbg = torch.zeros(4 * B * (s["V"] + s["d"] + 1), device=DEV)
    ham.ham_set_debug(rt.handle, dbg)
    a, b = 4 * B * s["V"], 4 * B * (s["V"] + s["d"])
    st["dbg"] = (dbg[:a].view(4, B, s["V"]), dbg[a:b].view(4, B, s["d"]), dbg[b:].view(4, B))
    i0 = ham.ham_state_info(cfg, 0)
    S, n = i0["slots"], s["L"] * B * s["Hk"] * i0["slots"] * s["hd"]
    t, es = (torch.bfloat16, 2) if s["bf"] else (torch.float32, 4)
    st["K"], st["V"] = (rt.state[o:o + n * es].view(t) for o in (i0["k_offset"], i0["v_offset"]))
    st["K"] = st["K"].view(s["L"], B, s["Hk"], S, s["hd"])
    st["V"] = st["V"].view(s["L"], B, s["Hk"], S // 32, s["hd"], 32)
    if case["steps"] and not case["fresh"]:
        _prefill(st)
        st["saved"] = torch.empty_like(rt.state)
        rt.save_state(st["saved"])
    return st


# ---------------------------------------------------------------- one pass
def _results(case, logits, hidden, stop, K, V):
    """What a pass wrote: the last step's decisions and the K and V slots it filled."""
    if not case["steps"]:
        logits, hidden, stop = logits[0], hidden[0], stop[0]
    a, b = case["prompt"] if case["steps"] and not case["fresh"] else 0, case["prompt"] + case["steps"]
    return {"logits": logits, "hidden": hidden, "stop": stop, "K": K[:, :, :, a:b], "V": V[:, :, :, a // 32:(b + 31) // 32]}


def run(s):
    case = s["case"]
    if case["kind"] == "step":
        ham.ham_op_attention_step(s["dtype"], s["qkv"], s["cos"], s["sin"], s["K"], s["V"], s["n"], s["slot"], s["on"],
                                  case["kv"] - 1, s["err"], s["out"], s["ws"], s["stream"], s["H"], s["Hk"], s["hd"], s["S"])
        return {"out": s["out"], "K": s["K"], "V": s["V"], "err": s["err"]}
    if case["kind"] == "attn":
        ham.ham_op_decode_attention(s["dtype"], s["q"], s["K"], s["V"], s["n"], s["on"], case["kv"], s["out"], s["ws"],
                                    s["stream"], s["H"], s["Hk"], s["hd"], s["S"])
        return {"out": s["out"]}
    if "saved" in s:
        s["rt"].restore_state(s["saved"])
    else:
        _prefill(s)
    for step in range(1, case["steps"] + 1):
        s["rt"].macro_step(s["forced"][step], s["teacher"][step])
    return _results(case, *s["dbg"], s["K"], s["V"])


# ---------------------------------------------------------------- work and tolerance
def work(case):
    es = 4 if case["dtype"] == "f32" else 2
    if case["kind"] in ("step", "attn"):
        kv = case["rows"] * 0.9 * case["kv"]
        return {"bytes": kv * 8 * case["hd"] * 2 * es + case["rows"] * 40 * case["hd"] * 4, "flops": 4.0 * kv * 32 * case["hd"]}
    s, B, P, N = _shape(case), case["batch"], case["prompt"], case["steps"]
    qkv, HD = (s["H"] + 2 * s["Hk"]) * s["hd"], s["H"] * s["hd"]
    layer = s["d"] * (qkv + HD + 3 * s["F"])
    kvd, C = 2 * s["Hk"] * s["hd"], min(CTX_ROWS, s["L"])
    b = f = 0.0

    def gemm(params, rows):
        nonlocal b, f
        b, f = b + params * es, f + 2.0 * params * rows

    def decisions(step):
        lens = _lengths(case, step)
        gemm(s["V"] * s["d"], B)
        for k in range(1, 4):
            live = sum(n > k for n in lens)
            if live:
                gemm(s["micro"] * layer, live * (C + 1 if k == 1 else 1))
                gemm(s["V"] * s["d"], live)

    if not N or case["fresh"]:
        gemm((s["L"] - 1) * layer, B * P)          # the last layer: K and V of every row, the rest of one row each
        gemm(s["d"] * kvd, B * P)
        gemm(layer - s["d"] * kvd, B)
        f += 2.0 * B * P * P * HD * (s["L"] - 1) + 4.0 * B * P * HD
        b += B * P * (kvd * es * s["L"] + s["d"] * (4 if case["embeds"] else es))
        decisions(0)
    for step in range(1, N + 1):
        fused = [n for n in _lengths(case, step - 1) if n > 1]
        if fused:
            gemm(3 * HD * s["d"], sum(fused))
            gemm(s["d"] * HD + s["d"] * s["d"], len(fused))
        gemm(s["L"] * layer, B)
        b += s["L"] * B * (P + step) * kvd * es
        f += 4.0 * s["L"] * B * (P + step) * HD
        decisions(step)
    return {"bytes": b, "flops": f}


def tolerance(case):
    """About four times what two correct builds differ by (sums in another order against float64, see exact)."""
    if case["dtype"] == "f32":
        return {"rel": 5e-6, "max": 2e-4}
    if case["kind"] in ("step", "attn"):
        return {"rel": 8e-4, "max": 0.02}    # hi and lo planes: a hi value may round the other way
    return {"rel": 8e-3, "max": 0.1}         # a cached bf16 K or V may round the other way and travels on


# ---------------------------------------------------------------- float64
_MASK = {n: (1 << (64 - n)) - 1 for n in (11, 27, 30, 31)}


def _sm64(key, i):
    """SplitMix64 output i (int64 tensor) of the stream seeded with key; wraps modulo 2^64."""
    def signed(c):
        return c - (1 << 64) if c >> 63 else c
    z = (i + 1) * signed(0x9E3779B97F4A7C15) + signed(key)
    z = (z ^ ((z >> 30) & _MASK[30])) * signed(0xBF58476D1CE4E5B9)
    z = (z ^ ((z >> 27) & _MASK[27])) * signed(0x94D049BB133111EB)
    return z ^ ((z >> 31) & _MASK[31])


def _normal(seed, tid, index, bf):
    """Generated weights at row-major indices: Box-Muller on SplitMix64, times 0.02, rounded to the storage type."""
    key = int(_sm64(int(seed), torch.tensor([tid]))[0]) % (1 << 64)
    r1, r2 = _sm64(key, 2 * index), _sm64(key, 2 * index + 1)
    u1 = (((r1 >> 11) & _MASK[11]).double() + 1.0) * 2.0 ** -53
    u2 = ((r2 >> 11) & _MASK[11]).double() * 2.0 ** -53
    v = (torch.sqrt(-2.0 * torch.log(u1)) * torch.cos((2.0 * math.pi) * u2) * 0.02).float()
    return (v.to(torch.bfloat16) if bf else v).double()


class _Model64:
    """The model of ``synth.configs`` in float64 (norm gains are 1): weights from the seed, kept once made."""

    def __init__(self, s, seed):
        self.s, self.seed, self.kept = s, seed, {}

    def w(self, tid, rows, cols):
        if tid not in self.kept:
            out = torch.empty(rows * cols, dtype=torch.float64, device=DEV)
            for i in range(0, rows * cols, 1 << 25):
                j = min(rows * cols, i + (1 << 25))
                out[i:j] = _normal(self.seed, tid, torch.arange(i, j, device=DEV), self.s["bf"])
            self.kept[tid] = out.view(rows, cols)
        return self.kept[tid]

    def embed(self, ids):
        d = self.s["d"]
        return _normal(self.seed, 0, ids.long()[..., None] * d + torch.arange(d, device=DEV), self.s["bf"])

    def stored(self, x):
        return (x.float().to(torch.bfloat16) if self.s["bf"] else x.float()).double()

    @staticmethod
    def norm(x):
        return x / torch.sqrt((x * x).mean(-1, keepdim=True) + 1e-5)

    def rope(self, v, pos):  # v [B][T][heads][hd], pos [B][T]
        hd = self.s["hd"]
        a = pos.double()[..., None] * 500000.0 ** (-2.0 * torch.arange(hd // 2, dtype=torch.float64, device=DEV) / hd)
        c, sn = a.cos().float().double()[:, :, None], a.sin().float().double()[:, :, None]
        x, y = v[..., :hd // 2], v[..., hd // 2:]
        return torch.cat([x * c - y * sn, y * c + x * sn], -1)

    def layer(self, j, X, pos, caches):
        """Layer j on new rows X [B][T][d]; caches: K and V [B][Hk][slots][hd], grown by T slots."""
        s = self.s
        B, T, d = X.shape
        H, Hk, hd, F = s["H"], s["Hk"], s["hd"], s["F"]
        w = lambda t, r, c: self.w(16 + 8 * j + t, r, c).T  # noqa: E731
        u = self.norm(X).reshape(B * T, d)
        q = self.rope((u @ w(0, H * hd, d)).view(B, T, H, hd), pos)
        k = self.stored(self.rope((u @ w(1, Hk * hd, d)).view(B, T, Hk, hd), pos)).transpose(1, 2)
        v = self.stored((u @ w(2, Hk * hd, d)).view(B, T, Hk, hd)).transpose(1, 2)
        K, V = caches.get(j, (k[:, :, :0], v[:, :, :0]))
        S0 = K.shape[2]
        K, V = caches[j] = (torch.cat([K, k], 2), torch.cat([V, v], 2))
        o = torch.empty(B, T, H, hd, dtype=torch.float64, device=DEV)
        for b in range(B):
            for h in range(H):
                for t0 in range(0, T, 4096):
                    t1 = min(T, t0 + 4096)
                    sc = q[b, t0:t1, h] @ K[b, h * Hk // H, :S0 + t1].T / math.sqrt(hd)
                    if T > 1:
                        sc.masked_fill_(torch.arange(S0 + t1, device=DEV) > S0 + torch.arange(t0, t1, device=DEV)[:, None], -math.inf)
                    o[b, t0:t1, h] = torch.softmax(sc, -1) @ V[b, h * Hk // H, :S0 + t1]
        x = X.reshape(B * T, d) + o.reshape(B * T, H * hd) @ w(3, d, H * hd)
        u = self.norm(x)
        x = x + (torch.nn.functional.silu(u @ w(4, F, d)) * (u @ w(5, F, d))) @ w(6, d, F)
        return x.view(B, T, d)

    def base(self, X, pos, caches):
        """Base layers; the last row's output and the context rows of the micro decoder."""
        L = self.s["L"]
        C = min(CTX_ROWS, L)
        at, ctx = [-(-(i + 1) * L // C) for i in range(C)], []
        for j in range(L):
            X = self.layer(j, X, pos, caches)
            if j + 1 in at:
                ctx.append(X[:, -1])
        return X[:, -1], torch.stack(ctx, 1)

    def decisions(self, x, ctx, tokens, lens):
        """Logits, normed hidden rows and stop logits of the four decisions (rows past a group's length unused)."""
        s, out = self.s, []
        B, C = ctx.shape[:2]
        caches = {}
        for k in range(4):
            if k and max(lens) > k:
                X = self.embed(tokens[:, k - 1:k])
                X = torch.cat([ctx, X], 1) if k == 1 else X
                pos = (torch.arange(C + 1, device=DEV) if k == 1 else torch.tensor([C + k - 1], device=DEV)).expand(B, -1)
                for j in range(s["micro"]):
                    X = self.layer(s["L"] + j, X, pos, caches)
                x = X[:, -1]
            h = self.norm(x)
            out.append((h @ self.w(7, s["V"], s["d"]).T, h, (h @ self.w(8, 1, s["d"]).T)[:, 0]))
        return [torch.stack(v) for v in zip(*out)]

    def fuse(self, tokens, n):
        """The compositional embedder on one group of n tokens."""
        s = self.s
        d, H, hd = s["d"], s["H"], s["hd"]
        if n == 1:
            return self.embed(tokens[:1])[0]
        e = self.embed(tokens[:n]) + self.w(1, 4, d)[:n]
        q, k, v = (x @ self.w(t, H * hd, d).T for x, t in ((e.mean(0, keepdim=True), 2), (e, 3), (e, 4)))
        a = torch.softmax((q.view(1, H, hd) * k.view(n, H, hd)).sum(-1) / math.sqrt(hd), 0)
        o = (a[..., None] * v.view(n, H, hd)).sum(0).reshape(1, H * hd)
        return (o @ self.w(5, d, H * hd).T @ self.w(6, d, d).T)[0]


def _exact_attn(case, seed):
    s = _attn_inputs(case, seed)
    R, H, Hk, hd, S = (s[k] for k in ("R", "H", "Hk", "hd", "S"))
    t = s["K"].dtype
    if case["kind"] == "step":
        x = s["qkv"].double()
        c, sn = s["cos"].double()[:, None], s["sin"].double()[:, None]

        def rope(v):
            a, b = v[..., :hd // 2], v[..., hd // 2:]
            return torch.cat([a * c - b * sn, b * c + a * sn], -1)
        q = rope(x[:, :H * hd].view(R, H, hd))
        k = rope(x[:, H * hd:(H + Hk) * hd].view(R, Hk, hd)).float().to(t)
        v = x[:, (H + Hk) * hd:].view(R, Hk, hd).float().to(t)
        r, at = torch.arange(R, device=DEV), s["slot"].long()
        s["K"][r, :, at] = k
        s["V"][r, :, at // 32, :, at % 32] = v
    else:
        q = s["q"].double().view(R, H, hd)
    out = torch.empty(R, H, hd, dtype=torch.float64, device=DEV)
    for r in range(R):
        n = int(s["n"][r])
        V = s["V"][r].permute(0, 1, 3, 2).reshape(Hk, S, hd)[:, :n].double()
        p = torch.softmax(q[r].view(Hk, H // Hk, hd) @ s["K"][r, :, :n].double().transpose(1, 2) / math.sqrt(hd), -1)
        out[r] = (p @ V).reshape(H, hd)
    out = _act(out.view(R, H * hd), case)
    return {"out": out} if case["kind"] == "attn" else {"out": out, "K": s["K"].double(), "V": s["V"].double(), "err": None}


def exact(case, seed):
    if case["kind"] in ("step", "attn"):
        return _exact_attn(case, seed)
    B, P, N = case["batch"], case["prompt"], case["steps"]
    if work(case)["flops"] + (case["kind"] == "decode") * 2e9 * B * P > 4e14 or B * case["layers"] > 300:
        return None
    x, s = _model_inputs(case, seed), _shape(case)
    m = _Model64(s, int(seed))
    rows = x["rows"].double() if case["embeds"] else m.embed(x["prompt"])
    pos = x["pos"] if case["embeds"] else torch.arange(P, device=DEV).expand(B, P)
    caches, last, lens = {}, pos[:, -1].clone(), _lengths(case, 0)
    h, ctx = m.base(rows, pos, caches)
    if not N:
        got = [v[None] for v in (m.norm(h), (m.norm(h) @ m.w(8, 1, s["d"]).T)[:, 0])]
        got = [(m.norm(h) @ m.w(7, s["V"], s["d"]).T)[None]] + got
    for step in range(1, N + 1):
        rows = torch.stack([m.fuse(x["teacher"][step - 1][b], lens[b]) for b in range(B)])[:, None]
        last = last + torch.tensor(lens, device=DEV)
        h, ctx = m.base(rows, last[:, None], caches)
        lens = _lengths(case, step)
        if step == N:
            got = m.decisions(h, ctx, x["teacher"][step], lens)
    S = (P + max(1, N) + 63) // 64 * 64
    K, V = (torch.stack([torch.nn.functional.pad(caches[j][i], (0, 0, 0, S - P - N)) for j in range(s["L"])]) for i in (0, 1))
    V = V.view(s["L"], B, s["Hk"], S // 32, 32, s["hd"]).transpose(-1, -2)
    return _results(case, *got, K, V)
