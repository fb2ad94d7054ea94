"""The workloads this library's speed is judged by, and what each has to return.

One draft-and-verify iteration is draft steps, one verify pass, accept and
commit; before it come prompt prefills.  The cases call those entry points as
a serving program does: weights packed once, a model handle and a KV cache per
model, resident contexts, one stream.  Shapes are the 7B-like and the 1.1B-like
decoder of synth.py; depths of 4 or 8 layers are the draft models (layer
prefixes of the target) and blocks of the target, 32 and 22 layers are whole
targets.  Weights, contexts, prompts and drafted tokens are seeded random
values with the distributions of synth.py (random N(0, 0.02^2) matrices,
N(0, (0.02 sqrt d)^2) keys and values, uniform token ids); RMSNorm gains are
drawn around 1.

Cases are plain dicts:
  op       accept | draft | verify | prefill
  shape    7b | 1b,  layers, weights (bf16 | int4)
  batch, gamma, temperature
  ctx_lo, ctx_hi   resident context lengths, spread evenly over the batch
  first, last      draft: the slots one pass runs (greedy drafts run them all,
                   a sampled draft runs one: its token decides the next slot)
  prompt, rows     prefill: tokens per prompt, rows per pass of the handle
  vocab, kind      accept: row length, probs | logits
"""
import ctypes
import math

import torch

from paper_2608_10362_amd import binding, synth

SHAPES = {"7b": synth.LLAMA_7B, "1b": synth.LLAMA_1B}
DEV = "cuda"


# ---------------------------------------------------------------- the cases
def _accept(name, batch, gamma, vocab, temperature, kind):
    return {"name": name, "op": "accept", "batch": batch, "gamma": gamma, "vocab": vocab,
            "temperature": temperature, "kind": kind}


def _model(name, op, shape, layers, weights, batch, ctx_lo, ctx_hi, **more):
    return {"name": name, "op": op, "shape": shape, "layers": layers, "weights": weights, "batch": batch,
            "ctx_lo": ctx_lo, "ctx_hi": ctx_hi, **more}


def listed():
    return [
        # the decision of a single stream: the smallest call there is, all latency
        _accept("accept_b1", 1, 4, 32000, 1.0, "logits"),
        # the decision of a full batch over a large vocabulary
        _accept("accept_b16_128k", 16, 6, 128256, 0.8, "logits"),
        # a small draft proposing greedily for one stream (the paper's mode): launches and latency
        _model("draft_1b_greedy", "draft", "1b", 4, "bf16", 1, 511, 511, gamma=4, first=0, last=3, temperature=0.0),
        # a 7B-wide draft proposing for eight streams, sampled; first slot, two pending rows a stream
        _model("draft_7b_b8", "draft", "7b", 4, "bf16", 8, 700, 2100, gamma=4, first=0, last=0, temperature=0.8),
        # the whole 7B target verifying one stream
        _model("verify_7b_b1", "verify", "7b", 32, "bf16", 1, 2048, 2048, gamma=4),
        # the whole 1.1B target (grouped-query attention) verifying four streams
        _model("verify_1b_b4", "verify", "1b", 22, "bf16", 4, 301, 1023, gamma=4),
        # a block of the 7B target verifying eight streams of ordinary length
        _model("verify_7b_b8", "verify", "7b", 4, "bf16", 8, 513, 2048, gamma=4),
        # a block of the 7B target verifying sixteen long streams
        _model("verify_7b_b16_long", "verify", "7b", 4, "bf16", 16, 1024, 8192, gamma=6),
        # INT4 layer weights, one stream
        _model("verify_7b_int4_b1", "verify", "7b", 8, "int4", 1, 2048, 2048, gamma=4),
        # INT4 layer weights, eight streams
        _model("verify_7b_int4_b8", "verify", "7b", 4, "int4", 8, 513, 2048, gamma=4),
        # prompt prefill of a 7B block in 512-row passes: the largest
        _model("prefill_7b", "prefill", "7b", 4, "bf16", 1, 0, 0, prompt=2048, rows=512),
        # three ragged-sized prompts on a small draft in one pass of its rows and a remainder
        _model("prefill_1b_b3", "prefill", "1b", 4, "bf16", 3, 0, 0, prompt=301, rows=600),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["accept", "draft", "verify", "verify", "verify", "prefill"])
    temperature = rng.choice([0.0, 0.8, 1.0])
    gamma = rng.randint(1, 8)
    if op == "accept":
        c = _accept("", _log(rng, 1, 16), gamma, _log(rng, 2000, 128256), temperature, rng.choice(["logits", "probs"]))
    else:
        shape = rng.choice(["7b", "7b", "1b"])
        weights = "int4" if op != "prefill" and rng.random() < 0.25 else "bf16"
        layers = rng.randint(1, 4) if shape == "7b" else rng.randint(1, 22)
        batch = _log(rng, 1, 16)
        hi = _log(rng, 64, 8192)
        lo = rng.randint(32, hi)
        if op == "prefill":
            total = _log(rng, 70, 2048)
            batch = min(batch, 4)
            prompt = max(2, total // batch)
            if shape == "1b":
                layers = min(layers, 8)
            c = _model("", op, shape, layers, weights, batch, 0, 0, prompt=prompt,
                       rows=rng.choice([64, 128, 256, 512, 1024]))
        elif op == "draft":
            first = 0 if rng.random() < 0.5 else rng.randrange(gamma)
            last = gamma - 1 if temperature == 0.0 else first
            c = _model("", op, shape, min(layers, 4), weights, batch, lo, hi, gamma=gamma, first=first, last=last,
                       temperature=temperature)
        else:
            if weights == "int4":
                batch = max(1, min(batch, 64 // (gamma + 1)))
            c = _model("", op, shape, layers, weights, batch, lo, hi, gamma=gamma)
    del c["name"]
    return c


# ---------------------------------------------------------------- inputs
def _lengths(case):
    """Resident context lengths: evenly spread, in a scattered order."""
    B, lo, hi = case["batch"], case["ctx_lo"], case["ctx_hi"]
    if B == 1:
        return [hi]
    return [lo + (hi - lo) * ((7 * b + 3) % B) // (B - 1) for b in range(B)] if B % 7 else \
        [lo + (hi - lo) * b // (B - 1) for b in range(B)]


class _Gen:
    """Numbered draws of one seed, the same on each call."""

    def __init__(self, seed):
        self.seed = seed
        self.g = torch.Generator(device=DEV)

    def normal(self, idx, shp, sigma, mean=0.0, dtype=torch.bfloat16):
        self.g.manual_seed((self.seed * 1000003 + idx) & 0x7FFFFFFFFFFF)
        return torch.empty(shp, dtype=torch.float32, device=DEV).normal_(mean, sigma, generator=self.g).to(dtype)

    def ints(self, idx, shp, hi):
        self.g.manual_seed((self.seed * 1000003 + idx) & 0x7FFFFFFFFFFF)
        return torch.randint(0, hi, shp, dtype=torch.int32, device=DEV, generator=self.g)


def _layer_weights(shape, gen, l):
    d, f = shape.d_model, shape.ffn_dim
    dims = {"attn_norm": (d,), "wq": (shape.q_dim, d), "wk": (shape.kv_dim, d), "wv": (shape.kv_dim, d),
            "wo": (d, shape.q_dim), "ffn_norm": (d,), "w_gate": (f, d), "w_up": (f, d), "w_down": (d, f)}
    return {k: gen.normal(100 + 16 * l + i, s, 0.1 if len(s) == 1 else 0.02, 1.0 if len(s) == 1 else 0.0)
            for i, (k, s) in enumerate(dims.items())}


def _top_weights(shape, gen):
    d, V = shape.d_model, shape.vocab
    return {"embed": gen.normal(1, (V, d), 0.02), "lm_head": gen.normal(2, (V, d), 0.02),
            "final_norm": gen.normal(3, (d,), 0.1, 1.0)}


def _context(shape, gen, l, b, n):
    sigma = 0.02 * shape.d_model ** 0.5
    shp = (n, shape.n_kv_heads, shape.head_dim)
    return gen.normal(5000 + 2 * (64 * l + b), shp, sigma), gen.normal(5001 + 2 * (64 * l + b), shp, sigma)


def _tokens(case, gen, vocab):
    """(pending pairs [B, 2], pending counts, drafted tokens [B, gamma])."""
    B, g = case["batch"], case["gamma"]
    pend = gen.ints(10, (B, 2), vocab)
    n_pend = [1 + (b + 1) % 2 if case["op"] == "draft" else 1 for b in range(B)]
    return pend, n_pend, gen.ints(11, (B, g), vocab)


def _resident(case):
    """Cache positions filled before the call: the contexts, and for a draft
    that starts at a later slot also its earlier slots."""
    lens = _lengths(case)
    if case["op"] != "draft" or case["first"] == 0:
        return lens
    n_pend = [1 + (b + 1) % 2 for b in range(case["batch"])]
    return [n + p + case["first"] - 1 for n, p in zip(lens, n_pend)]


def prepare(case, seed):
    gen = _Gen(seed)
    B = case["batch"]
    if case["op"] == "accept":
        g, V, T = case["gamma"], case["vocab"], case["temperature"]
        lg = gen.normal(20, (B, g + 1, V), 1.3, dtype=torch.float32)
        # a draft that resembles the target: about half of its tokens are accepted
        q = torch.softmax((0.8 * lg[:, :g] + gen.normal(21, (B, g, V), 0.8, dtype=torch.float32)) / (T or 1.0), -1)
        gen.g.manual_seed(gen.seed * 1000003 + 22)
        d = torch.multinomial(q.reshape(B * g, V), 1, generator=gen.g).reshape(B, g).to(torch.int32)
        p = lg if case["kind"] == "logits" else torch.softmax(lg / (T or 1.0), -1)
        z = lambda: torch.zeros(B, dtype=torch.int32, device=DEV)  # noqa: E731
        return {"case": case, "p": p.contiguous(), "q": q.contiguous(), "d": d, "n_acc": z(), "next": z(),
                "status": torch.zeros(1, dtype=torch.int32, device=DEV), "ws": binding.accept_workspace(B, g, V, DEV),
                "seed": int(seed)}
    shape = SHAPES[case["shape"]].with_layers(case["layers"])
    L, V = case["layers"], shape.vocab
    w = _top_weights(shape, gen)
    w["layers"] = [_layer_weights(shape, gen, l) for l in range(L)]
    dw = binding.DeviceWeights(shape, w, device=DEV, weight_format=case["weights"])
    del w
    st = {"case": case, "seed": int(seed), "dw": dw}
    if case["op"] == "prefill":
        cap = (case["prompt"] + 63) // 64 * 64
        st["model"] = binding.Model(dw, L, max_rows=max(case["rows"], B), max_ctx=cap)
        st["kv"] = binding.KVCache(st["model"], B, cap)
        st["kv"].data.zero_()
        st["tokens"] = gen.ints(12, (B, case["prompt"]), V)
        return st
    g = case["gamma"]
    lens, filled = _lengths(case), _resident(case)
    cap = (max(lens) + g + 2 + 63) // 64 * 64
    rows = B * (g + 1) if case["op"] == "verify" else 2 * B
    st["model"] = binding.Model(dw, L, max_rows=rows, max_ctx=cap)
    st["kv"] = kv = binding.KVCache(st["model"], B, cap)
    for l in range(L):
        for b in range(B):
            kv.write_context(l, b, 0, *_context(shape, gen, l, b, filled[b]))
    pend, n_pend, drafts = _tokens(case, gen, V)
    kv.set_state(lens, pend.cpu().numpy(), n_pend)
    st["d"] = drafts
    if case["op"] == "verify":
        st["logits"] = torch.empty((B, g + 1, V), dtype=torch.float32, device=DEV)
    else:
        n = case["last"] - case["first"] + 1
        st["logits"] = [torch.empty((B, V), dtype=torch.float32, device=DEV) for _ in range(n)]
        st["q"] = torch.zeros((B, g, V), dtype=torch.float32, device=DEV) if case["temperature"] > 0 else None
    return st


# ---------------------------------------------------------------- one pass
def run(st):
    case = st["case"]
    B = case["batch"]
    if case["op"] == "accept":
        kind = binding.INPUT_LOGITS if case["kind"] == "logits" else binding.INPUT_PROBS
        T = case["temperature"]
        binding.specdec_accept(B, case["gamma"], case["vocab"], kind, T, st["p"], st["q"] if T > 0 else None, st["d"],
                               case["gamma"], None, st["seed"], 0, st["n_acc"], st["next"], st["status"], st["ws"])
        return {"n_accepted": st["n_acc"], "next": st["next"], "status": st["status"]}
    model, kv = st["model"], st["kv"]
    if case["op"] == "prefill":
        # a new prompt takes over the cache
        binding._check(binding.lib().specdec_kv_init(ctypes.byref(kv.kv), model.handle, B, kv.kv.capacity,
                                                     kv.data.data_ptr(), kv.data.numel(), kv.state.data_ptr(),
                                                     torch.cuda.current_stream().cuda_stream), "specdec_kv_init")
        binding.specdec_prefill(model, kv, st["tokens"])
        return {"kv": kv.data.view(torch.bfloat16), "state": kv.state}
    g = case["gamma"]
    if case["op"] == "verify":
        binding.specdec_verify(model, kv, g, st["d"], g, st["logits"])
        return {"logits": st["logits"]}
    for i, s in enumerate(range(case["first"], case["last"] + 1)):
        binding.specdec_draft_step(model, kv, g, s, case["temperature"], st["seed"], 0, None, st["q"], st["d"], g,
                                   st["logits"][i])
    out = {"logits": list(st["logits"]), "d": st["d"]}
    if st["q"] is not None:
        out["q"] = st["q"]
    return out


# ---------------------------------------------------------------- what a pass cannot do without
def work(case):
    B = case["batch"]
    if case["op"] == "accept":
        g, V = case["gamma"], case["vocab"]
        rows = g + 1 + (g if case["temperature"] > 0 else 0)  # the target's rows, and the draft's when sampling
        return {"bytes": 4.0 * B * V * rows, "flops": 4.0 * B * V * rows}
    s = SHAPES[case["shape"]]
    L, d, f, V, q, kvd = case["layers"], s.d_model, s.ffn_dim, s.vocab, s.q_dim, s.kv_dim
    mats = (q + 2 * kvd) * d + d * q + 3 * d * f
    layer_bytes = mats * (2.0 if case["weights"] == "bf16" else 0.5 + 2.0 / 128)
    kv_row = 2.0 * kvd * 2  # keys and values of one position of one layer
    if case["op"] == "prefill":
        n = case["prompt"] - 1
        flops = B * n * 2.0 * L * mats + B * L * 4.0 * q * (n * (n + 1) / 2)
        return {"bytes": L * (layer_bytes + B * n * kv_row) + B * n * d * 2.0, "flops": flops}
    lens = _lengths(case)
    if case["op"] == "verify":
        passes = [(B * (case["gamma"] + 1), B * (case["gamma"] + 1), [n + case["gamma"] + 1 for n in lens])]
    else:
        passes = [(2 * B if t == 0 else B, B, [n + 2 + t for n in lens]) for t in range(case["first"], case["last"] + 1)]
    nbytes = flops = 0.0
    for rows, outs, ctx in passes:
        nbytes += L * (layer_bytes + sum(ctx) * kv_row) + V * d * 2.0 + rows * d * 2.0 + outs * V * 4.0
        flops += 2.0 * rows * (L * mats) + 2.0 * outs * V * d + L * 4.0 * q * sum(ctx) * rows / B
        if case["op"] == "draft" and case["temperature"] > 0:
            nbytes += B * V * 4.0
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    if case["op"] == "accept":
        # a decision may fall on the other side of a boundary that lies within the softmax's rounding
        return {"rel": 0.0, "differ": min(0.99, 1.5 / case["batch"])}
    if case["op"] == "prefill":
        # keys and values stored in bf16: a changed rounding moves single values by one unit in the last place
        # (7.4e-4 from the 64-bit result over four 7B layers)
        return {"rel": 3e-3}
    # float32 results behind keys and values stored in bf16: 1e-5 to 4e-5 from the 64-bit result with bf16 weights
    # (4 to 32 layers), 6e-5 to 1.1e-4 with INT4 weights
    t = {"rel": 5e-4 if case["weights"] == "int4" else 2e-4}
    if case["op"] == "draft":
        t["differ"] = 1.5 / (case["batch"] * case["gamma"]) if case["batch"] * case["gamma"] > 1 else 0.99
    return t


# ---------------------------------------------------------------- 64-bit results
def _bf16(x):
    return x.to(torch.float32).to(torch.bfloat16).double()


def _matrix(w, case):
    """The effective matrix in 64 bits: the bf16 weights, or codes times scales of 128-column groups."""
    if case["weights"] != "int4":
        return w.double()
    N, K = w.shape
    G = (K + 127) // 128
    x = torch.zeros((N, G * 128), dtype=torch.float32, device=w.device)
    x[:, :K] = w.float()
    x = x.reshape(N, G, 128)
    s = (x.abs().amax(-1, keepdim=True) / 7.0).to(torch.bfloat16).float()
    c = torch.where(s == 0, torch.zeros_like(x), torch.clamp(torch.round(x / s), -8, 7))
    return (c.double() * s.double()).reshape(N, G * 128)[:, :K].contiguous()


def _norm(x, g, eps):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + eps) * g.double()


def _rope(x, pos, shape):
    """x [n, heads, hd], pos [n]."""
    half = shape.head_dim // 2
    j = torch.arange(half, dtype=torch.float64, device=x.device)
    ang = pos.double()[:, None] * torch.pow(torch.tensor(shape.rope_base, dtype=torch.float64, device=x.device),
                                            -2.0 * j / shape.head_dim)[None]
    c, s = torch.cos(ang)[:, None], torch.sin(ang)[:, None]
    a, b = x[..., :half], x[..., half:]
    return torch.cat([a * c - b * s, b * c + a * s], -1)


def _attend(q, k, v, pos, shape):
    """q [n, H, hd] at positions pos, k and v [m, G, hd] in 64 bits; keys 0..pos are seen."""
    H, G, hd = shape.n_heads, shape.n_kv_heads, shape.head_dim
    n, m = q.shape[0], k.shape[0]
    qg = q.reshape(n, G, H // G, hd).permute(1, 2, 0, 3).reshape(G, (H // G) * n, hd).contiguous()
    out = torch.empty_like(qg)
    seen = (torch.arange(m, device=q.device)[None] <= pos[:, None]).repeat(H // G, 1)
    for g in range(G):
        sc = torch.mm(qg[g], k[:, g].t().contiguous()) / math.sqrt(hd)
        p = torch.softmax(sc.masked_fill(~seen, -math.inf), -1)
        out[g] = torch.mm(p, v[:, g].contiguous())
    return out.reshape(G, H // G, n, hd).permute(2, 0, 1, 3).reshape(n, H * hd)


class _Reference:
    """The decoder in 64 bits; keys and values are rounded to bf16 where they
    are stored.  layer(l) gives layer l's matrices, drawn again when needed."""

    def __init__(self, case, seed):
        self.case, self.gen = case, _Gen(seed)
        self.shape = SHAPES[case["shape"]]
        self.top = _top_weights(self.shape, self.gen)
        n = [0] * case["batch"] if case["op"] == "prefill" else _resident(case)
        self.kv = [[[t.double() for t in _context(self.shape, self.gen, l, b, n[b])] if n[b] else
                    [torch.zeros((0, self.shape.n_kv_heads, self.shape.head_dim), dtype=torch.float64, device=DEV)] * 2
                    for b in range(case["batch"])] for l in range(case["layers"])] if case["op"] != "verify" else None
        self.n = n

    def forward(self, tokens, pos, head=True):
        """tokens, pos: per sequence lists of tensors; appends the rows to the
        caches and returns the logits per sequence."""
        s, case = self.shape, self.case
        rows = [len(t) for t in tokens]
        x = self.top["embed"][torch.cat(tokens).long()].double()
        allpos = torch.cat(pos)
        for l in range(case["layers"]):
            w = _layer_weights(s, self.gen, l)
            y = _norm(x, w["attn_norm"], s.rms_eps)
            q = _rope((y @ _matrix(w["wq"], case).t()).reshape(-1, s.n_heads, s.head_dim), allpos, s)
            k = _bf16(_rope((y @ _matrix(w["wk"], case).t()).reshape(-1, s.n_kv_heads, s.head_dim), allpos, s))
            v = _bf16((y @ _matrix(w["wv"], case).t()).reshape(-1, s.n_kv_heads, s.head_dim))
            o, at = [], 0
            for b, r in enumerate(rows):
                if self.kv is not None:
                    old = self.kv[l][b]
                else:  # (a single pass: the contexts are drawn when needed)
                    old = [t.double() for t in _context(s, self.gen, l, b, self.n[b])]
                kb, vb = torch.cat([old[0], k[at:at + r]]), torch.cat([old[1], v[at:at + r]])
                if self.kv is not None:
                    self.kv[l][b] = [kb, vb]
                o.append(_attend(q[at:at + r], kb, vb, pos[b], s))
                at += r
            x = x + torch.cat(o) @ _matrix(w["wo"], case).t()
            y = _norm(x, w["ffn_norm"], s.rms_eps)
            gate, up = y @ _matrix(w["w_gate"], case).t(), y @ _matrix(w["w_up"], case).t()
            x = x + (gate * torch.sigmoid(gate) * up) @ _matrix(w["w_down"], case).t()
        if not head:
            return None
        lg = _norm(x, self.top["final_norm"], s.rms_eps) @ self.top["lm_head"].double().t()
        return list(lg.split(rows))


def _kv_image(case, shape, kv, cap):
    """The cache's storage: per (layer, sequence, kv head) a K block, then a V
    block, in fragments of 16 positions x 32 dims (K) and 32 positions x 16
    dims (V) with eight consecutive dims (K) or positions (V) innermost."""
    G, hd, out = shape.n_kv_heads, shape.head_dim, []
    for l in range(case["layers"]):
        for b in range(case["batch"]):
            k, v = (torch.cat([t, torch.zeros((cap - t.shape[0], G, hd), dtype=t.dtype, device=t.device)])
                    for t in kv[l][b])
            kf = k.reshape(cap // 16, 16, G, hd // 32, 4, 8).permute(2, 0, 3, 4, 1, 5).reshape(G, -1)
            vf = v.reshape(cap // 32, 4, 8, G, hd // 16, 16).permute(3, 0, 4, 1, 5, 2).reshape(G, -1)
            out.append(torch.cat([kf, vf], 1).reshape(-1))
    return torch.cat(out)


def exact(case, seed):
    if case["op"] == "accept":
        return None  # whole numbers, decided by integer sums
    ref = _Reference(case, seed)
    gen, V, B = _Gen(seed), ref.shape.vocab, case["batch"]
    ints = lambda lo, n: torch.arange(lo, lo + n, device=DEV)  # noqa: E731
    if case["op"] == "prefill":
        n = case["prompt"] - 1
        tok = gen.ints(12, (B, case["prompt"]), V)
        ref.forward([tok[b, :n] for b in range(B)], [ints(0, n)] * B, head=False)
        return {"kv": _kv_image(case, ref.shape, ref.kv, (case["prompt"] + 63) // 64 * 64), "state": None}
    pend, n_pend, d = _tokens(case, gen, V)
    lens = _lengths(case)
    if case["op"] == "verify":
        rows = case["gamma"] + 1
        lg = ref.forward([torch.cat([pend[b, 1:], d[b]]) for b in range(B)], [ints(lens[b], rows) for b in range(B)])
        return {"logits": torch.stack(lg)}
    d, T, logits, q = d.clone(), case["temperature"], [], None
    if T > 0:
        q = torch.zeros((B, case["gamma"], V), dtype=torch.float64, device=DEV)
    for s in range(case["first"], case["last"] + 1):
        if s == 0:
            lg = ref.forward([pend[b, 2 - n_pend[b]:] for b in range(B)], [ints(lens[b], n_pend[b]) for b in range(B)])
        else:
            lg = ref.forward([d[b, s - 1:s] for b in range(B)], [ints(lens[b] + n_pend[b] + s - 1, 1) for b in range(B)])
        last = torch.stack([x[-1] for x in lg])
        logits.append(last)
        if T > 0:
            q[:, s] = torch.softmax(last / T, -1)
        else:
            d[:, s] = last.argmax(-1).to(torch.int32)
    out = {"logits": logits, "d": None}
    if q is not None:
        out["q"] = q
    return out
