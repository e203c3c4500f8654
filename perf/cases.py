"""The work a user of this library has it do, as cases that can be timed: decode steps of the shared decode module
over a mixed batch (bf16 and 4-bit weights, from one request to a full batch), a multi-step run of the fp32
configuration, prefill of a prompt (whole, and as the continuation of a cached one) and the ingest of a cache that was
computed elsewhere.

Shapes are the repository's own (8B, 14B and tiny).  Most cases hold eight of the backbone's layers: every layer is the
same launches on weights and caches of its own (nothing stays in a cache of the chip from one layer to the next), and
eight of them can be prepared and checked against 64 bits in seconds.  Two cases hold the 8B backbone whole.

A case is a dict of plain values:
  op "step":    one decode step of `batch` requests whose cached lengths lie in [lo, hi] ("uniform": uniformly, "long_tail":
                log-normally around median with sigma 1, as the serving workload with a skewed length distribution)
  op "run":     `steps` decode steps in a row with greedy feedback
  op "prefill": `tokens` prompt positions behind `first` cached ones
  op "ingest":  a cache of `tokens` positions placed behind `first` cached ones
`weights` is "f32", "bf16" or "w4" (4-bit codes in groups of 128, fp16 scales and zero points)."""
import dataclasses
import math

import numpy as np
import torch

from paper_2603_02599_amd import binding as sun
from paper_2603_02599_amd import workloads as wl

DEV = "cuda:0"
PAGE = 16
GROUP = 128
MATS = ("wq", "wk", "wv", "wo", "wg", "wu", "wd")


def listed():
    return [
        # the fp32 configuration, a handful of short requests: the smallest calls, launches and latency are all there is
        {"name": "run_tiny_f32", "op": "run", "shape": "tiny", "layers": 2, "weights": "f32", "batch": 8, "lo": 16, "hi": 128, "steps": 16},
        # one user, one short conversation: interactive latency, weight streaming
        {"name": "step_8b_b1_bf16", "op": "step", "shape": "llama8b", "layers": 8, "weights": "bf16", "batch": 1, "lo": 1024, "hi": 1024, "dist": "uniform"},
        # a few users on 4-bit weights
        {"name": "step_8b_b5_w4", "op": "step", "shape": "llama8b", "layers": 8, "weights": "w4", "batch": 5, "lo": 256, "hi": 2048, "dist": "uniform"},
        # a lightly loaded worker
        {"name": "step_8b_b16_bf16", "op": "step", "shape": "llama8b", "layers": 8, "weights": "bf16", "batch": 16, "lo": 512, "hi": 4096, "dist": "uniform"},
        # the benchmark's default batch: 64 requests of four source models, the whole backbone, bf16 and 4-bit
        {"name": "step_8b_full_b64_bf16", "op": "step", "shape": "llama8b", "layers": 32, "weights": "bf16", "batch": 64, "lo": 512, "hi": 4096, "dist": "uniform"},
        {"name": "step_8b_full_b64_w4", "op": "step", "shape": "llama8b", "layers": 32, "weights": "w4", "batch": 64, "lo": 512, "hi": 4096, "dist": "uniform"},
        # a full batch with the skewed lengths of the heavy-traffic workload
        {"name": "step_8b_b256_bf16", "op": "step", "shape": "llama8b", "layers": 8, "weights": "bf16", "batch": 256, "lo": 64, "hi": 16384, "dist": "long_tail", "median": 1024},
        {"name": "step_8b_b150_w4", "op": "step", "shape": "llama8b", "layers": 8, "weights": "w4", "batch": 150, "lo": 64, "hi": 16384, "dist": "long_tail", "median": 1024},
        # the 14B backbone with long contexts: five query heads per kv head, attention is most of the step
        {"name": "step_14b_b24_w4", "op": "step", "shape": "qwen14b", "layers": 8, "weights": "w4", "batch": 24, "lo": 2048, "hi": 32768, "dist": "uniform"},
        # a prompt from its first token
        {"name": "prefill_8b_1024", "op": "prefill", "shape": "llama8b", "layers": 8, "weights": "bf16", "tokens": 1024, "first": 0},
        # a long prompt continued: the next turn of a conversation whose history is cached, ragged on both sides
        {"name": "prefill_8b_3000_at_1003", "op": "prefill", "shape": "llama8b", "layers": 8, "weights": "bf16", "tokens": 3000, "first": 1003},
        # the receiving end of disaggregated serving: a whole prompt's cache of all layers, bytes in bytes out
        {"name": "ingest_8b_4096", "op": "ingest", "shape": "llama8b", "layers": 32, "weights": "bf16", "tokens": 4096, "first": 0},
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    op = rng.choice(["step", "step", "step", "step", "prefill", "prefill", "run", "ingest"])
    if op == "run":
        lo = _log_int(rng, 1, 64)
        return {"op": "run", "shape": "tiny", "layers": 2, "weights": "f32", "batch": _log_int(rng, 1, 48), "lo": lo, "hi": lo + _log_int(rng, 1, 200), "steps": rng.randint(2, 16)}
    shape = rng.choice(["llama8b", "llama8b", "qwen14b"])
    if op == "ingest":
        return {"op": "ingest", "shape": shape, "layers": rng.choice([8, 32]) if shape == "llama8b" else 8, "weights": "bf16",
                "tokens": _log_int(rng, 16, 4096), "first": rng.choice([0, 0, rng.randint(1, 2000)])}
    if op == "prefill":
        tokens = _log_int(rng, 20, 2500 if shape == "llama8b" else 1200)
        return {"op": "prefill", "shape": shape, "layers": 8 if shape == "llama8b" else 4, "weights": "bf16", "tokens": tokens,
                "first": rng.choice([0, 0, rng.randint(1, 1500)])}
    batch = _log_int(rng, 1, 256)
    weights = rng.choice(["bf16", "w4"])
    if rng.random() < 0.3:
        return {"op": "step", "shape": shape, "layers": 8, "weights": weights, "batch": batch, "lo": 64, "hi": 16384, "dist": "long_tail", "median": rng.randint(256, 1024)}
    hi = _log_int(rng, 256, max(512, min(16384, 400000 // batch)))
    return {"op": "step", "shape": shape, "layers": 8, "weights": weights, "batch": batch, "lo": rng.randint(1, hi), "hi": hi, "dist": "uniform"}


# ------------------------------------------------------------------ inputs
def _shape(case):
    return dataclasses.replace(wl.SHAPES[case["shape"]], n_layers=int(case["layers"]))


def _gen(seed, what):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1000003 + what) & 0x7FFFFFFFFFFF)
    return g


def _mats(shape, dtype, seed, layer):
    """The matrices of one layer, N(0, 0.02^2), and its two gains, 1 + N(0, 0.1^2)."""
    g = _gen(seed, 100 + layer)
    h, q, kv, f = shape.hidden, shape.q_dim, shape.kv_dim, shape.ffn
    dims = {"wq": (q, h), "wk": (kv, h), "wv": (kv, h), "wo": (h, q), "wg": (f, h), "wu": (f, h), "wd": (h, f)}
    out = {k: torch.empty(d, dtype=dtype, device=DEV).normal_(0.0, 0.02, generator=g) for k, d in dims.items()}
    for k in ("g1", "g2"):
        out[k] = torch.empty(h, device=DEV).normal_(1.0, 0.1, generator=g).to(dtype)
    return out


def _ends(shape, dtype, seed):
    g = _gen(seed, 1)
    out = {k: torch.empty((shape.vocab, shape.hidden), dtype=dtype, device=DEV).normal_(0.0, 0.02, generator=g) for k in ("embed", "wlm")}
    out["gf"] = torch.empty(shape.hidden, device=DEV).normal_(1.0, 0.1, generator=g).to(dtype)
    return out


def _quantise(w):
    """Round to nearest on a grid per row and 128 inputs: codes two a byte (low nibble first), fp16 scale and zero point."""
    rows, cols = w.shape
    x = w.float().view(rows, cols // GROUP, GROUP)
    lo, hi = x.amin(2, keepdim=True), x.amax(2, keepdim=True)
    s = ((hi - lo) / 15).half()
    z = torch.round(-lo / s.float()).clamp_(0, 15)
    q = (torch.round(x / s.float()) + z).clamp_(0, 15).to(torch.uint8).view(rows, cols)
    return (q[:, 0::2] | (q[:, 1::2] << 4)).contiguous(), s.view(rows, -1).contiguous(), z.half().view(rows, -1).contiguous()


def _dequantise(q, s, z):
    rows = q.shape[0]
    codes = torch.stack([q & 15, q >> 4], 2).view(rows, -1, GROUP).double()
    return ((codes - z.double().unsqueeze(2)) * s.double().unsqueeze(2)).view(rows, -1)


def _weights(case, shape, cfg, seed):
    dtype = torch.float32 if case["weights"] == "f32" else torch.bfloat16
    w = _ends(shape, dtype, seed)
    layers = [_mats(shape, dtype, seed, i) for i in range(shape.n_layers)] if case["weights"] != "w4" else None
    if layers is not None:
        for k in MATS + ("g1", "g2"):
            w[k] = [m[k] for m in layers]
        del layers
        return sun.sun_weights_create(cfg, w, keep_sources=False)
    quant = {k: [] for k in MATS}
    w["g1"], w["g2"] = [], []
    for i in range(shape.n_layers):
        m = _mats(shape, dtype, seed, i)
        for k in MATS:
            quant[k].append(_quantise(m[k]))
        w["g1"].append(m["g1"])
        w["g2"].append(m["g2"])
    return sun.sun_qweights_create(cfg, w, quant, GROUP)


def _requests(case, shape, seed):
    """Lengths, page tables, token ids and source-model ids of the batch (host), and the pool's page count.  The lengths
    belong to the case (the pool has the same size for every seed), the rest to the seed."""
    batch, grow = int(case["batch"]), int(case.get("steps", 0))
    r = np.random.default_rng([7, batch, int(case["lo"]), int(case["hi"])])
    if case.get("dist") == "long_tail":
        lens = np.clip(np.rint(np.exp(math.log(case["median"]) + r.standard_normal(batch))), case["lo"], case["hi"])
    else:
        lens = r.integers(case["lo"], case["hi"] + 1, size=batch)
    r = np.random.default_rng([int(seed), 7])
    lens = np.asarray(lens, dtype=np.int32)
    need = (lens + grow) // PAGE + 1
    have = lens // PAGE + 1            # a run takes the further pages from the free list
    n_pages = int(need.sum()) + batch // 4 + 4
    perm = r.permutation(n_pages).astype(np.int32)
    tables = np.full((batch, int(need.max())), -1, dtype=np.int32)
    o = 0
    for i in range(batch):
        tables[i, : have[i]] = perm[o : o + have[i]]
        o += int(have[i])
    tokens = r.integers(0, shape.vocab, size=batch).astype(np.int32)
    ids = r.integers(0, 4, size=batch).astype(np.int32)
    return {"lens": lens, "tables": tables, "tokens": tokens, "ids": ids, "free": perm[o:], "n_pages": n_pages}


def _prompt(case, shape, seed):
    """The page-table row of one request, its prompt tokens and the pool's page count."""
    r = np.random.default_rng([int(seed), 8])
    n = (int(case["first"]) + int(case["tokens"]) + PAGE - 1) // PAGE
    n_pages = n + 5
    return {"row": r.permutation(n_pages)[:n].astype(np.int32), "tokens": r.integers(0, shape.vocab, size=int(case["tokens"])).astype(np.int32), "n_pages": n_pages}


def _pool_mem(shape, cfg, n_pages, seed):
    mem = torch.empty(sun.sun_kv_pool_bytes(cfg, n_pages) // 2, dtype=torch.bfloat16, device=DEV)
    return mem.normal_(0.0, 1.0, generator=_gen(seed, 2)) if mem.numel() < 1 << 31 else _fill(mem, _gen(seed, 2))


def _fill(mem, g):
    for o in range(0, mem.numel(), 1 << 30):
        mem[o : o + (1 << 30)].normal_(0.0, 1.0, generator=g)
    return mem


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def _source_cache(case, shape, seed):
    g = _gen(seed, 3)
    dims = (shape.n_layers, int(case["tokens"]), shape.n_kv_heads, shape.head_dim)
    return [torch.empty(dims, dtype=torch.bfloat16, device=DEV).normal_(0.0, 1.0, generator=g) for _ in range(2)]


def prepare(case, seed):
    shape = _shape(case)
    cfg = sun.make_cfg(shape, "f32" if case["weights"] == "f32" else "bf16")
    s = {"op": case["op"], "cfg": cfg, "w4": case["weights"] == "w4"}
    if case["op"] in ("step", "run"):
        req = _requests(case, shape, seed)
        batch = len(req["lens"])
        s["weights"] = _weights(case, shape, cfg, seed)
        s["mem"] = _pool_mem(shape, cfg, req["n_pages"], seed)
        s["pool"] = sun.sun_kv_pool_create(cfg, s["mem"], PAGE, 4)
        for k in ("lens", "tables", "tokens", "ids", "free"):
            s[k] = _dev(req[k])
        s["host_lens"] = req["lens"]
        s["ws"] = torch.empty(sun.sun_workspace_bytes(cfg, batch, req["tables"].shape[1]), dtype=torch.uint8, device=DEV)
        s["logits"] = torch.empty((batch, shape.vocab), device=DEV)
        s["next"] = torch.empty(batch, dtype=torch.int32, device=DEV)
        if case["op"] == "run":
            s["steps"] = int(case["steps"])
            s["out"] = torch.empty((s["steps"], batch), dtype=torch.int32, device=DEV)
            s["head0"] = torch.zeros(1, dtype=torch.int32, device=DEV)
            s["status"] = torch.zeros(1, dtype=torch.int32, device=DEV)
        return s
    p = _prompt(case, shape, seed)
    s["mem"] = _pool_mem(shape, cfg, p["n_pages"], seed)
    s["pool"] = sun.sun_kv_pool_create(cfg, s["mem"], PAGE, 4)
    s["row"], s["first"] = _dev(p["row"]), int(case["first"])
    if case["op"] == "ingest":
        s["k"], s["v"] = _source_cache(case, shape, seed)
        return s
    s["weights"] = _weights(case, shape, cfg, seed)
    s["tokens"] = _dev(p["tokens"])
    s["ws"] = torch.empty(sun.sun_prefill_workspace_bytes(cfg, int(case["tokens"]), len(p["row"])), dtype=torch.uint8, device=DEV)
    s["logits"] = torch.empty(shape.vocab, device=DEV)
    s["next"] = torch.empty(1, dtype=torch.int32, device=DEV)
    return s


def run(s):
    if s["op"] == "step":
        step = sun.sun_qdecode_step if s["w4"] else sun.sun_decode_step
        step(s["pool"], s["weights"], s["tokens"], s["tables"], s["lens"], s["ids"], s["logits"], s["next"], s["ws"], seq_lens_host=s["host_lens"])
        # The next tokens are the logits' argmax.  They are left out: two correct sums differ by about 1e-4 of a logit's size
        # and the two largest of 128 256 lie some 0.2 apart, so that every tenth batch or so has a row that ties.
        # A pool of more than 16 GiB is left out as well, only for its size.
        return {"logits": s["logits"], "cache": s["mem"] if s["mem"].numel() < 1 << 33 else None}
    if s["op"] == "run":
        tokens, tables, lens, head = s["tokens"].clone(), s["tables"].clone(), s["lens"].clone(), s["head0"].clone()
        sun.sun_decode_run(s["pool"], s["weights"], s["steps"], tokens, tables, lens, s["ids"], s["free"], head, s["status"], s["out"], s["logits"], s["ws"])
        return {"tokens": s["out"], "logits": s["logits"], "tables": tables, "lens": lens, "head": head, "status": s["status"], "cache": s["mem"]}
    if s["op"] == "prefill":
        sun.sun_prefill(s["pool"], s["weights"], s["tokens"], s["row"], s["first"], 1, s["logits"], s["next"], s["ws"])
        return {"cache": s["mem"], "logits": s["logits"]}
    sun.sun_kv_pool_ingest(s["pool"], 1, s["k"], s["v"], s["first"], s["row"])
    return {"cache": s["mem"]}


# ------------------------------------------------------------------ what a pass cannot do without
def work(case):
    sh = _shape(case)
    wb = {"f32": 4.0, "bf16": 2.0, "w4": 0.53125}[case["weights"]]
    dense = 4.0 if case["weights"] == "f32" else 2.0
    body, head = sh.body_params, sh.vocab * sh.hidden
    kv = sh.kv_bytes_per_token()
    attn = 4.0 * sh.n_layers * sh.q_dim   # per query and cached position
    if case["op"] == "ingest":
        return {"bytes": 2.0 * kv * case["tokens"], "flops": 0.0}
    if case["op"] == "prefill":
        n, first = int(case["tokens"]), int(case["first"])
        pairs = n * first + n * (n + 1) / 2
        return {"bytes": body * wb + head * dense + kv * (first + n) + n * sh.hidden * dense + sh.vocab * 4.0, "flops": 2.0 * body * n + 2.0 * head + attn * pairs}
    batch, steps = int(case["batch"]), int(case.get("steps", 1))
    lens = _requests(case, sh, 0)["lens"].astype(np.float64)
    cached = float(lens.sum()) + batch * (steps - 1) / 2
    one = {"bytes": body * wb + head * dense + kv * (cached + batch) + batch * (sh.hidden * dense + sh.vocab * 4.0), "flops": 2.0 * (body + head) * batch + attn * (cached + batch)}
    if case["op"] == "run":  # weights and caches of all steps, the logits of the last
        one["bytes"] -= batch * sh.vocab * 4.0 * (1 - 1 / steps)
    return {k: v * steps for k, v in one.items()}


def tolerance(case):
    """About four times the distance of two correct implementations: 1.4 times the error against 64 bits that was
    measured (bf16 weights 2e-5 to 9e-5 of the logits; 4-bit weights 2.5e-4 to 1e-3, their activations have 16 bits a
    group; prefill 2e-4 to 1e-3, where a new cache entry that falls on the other side of a bf16 rounding is attended
    to by all later rows).  An entry of the cache may differ by a rounding step of bf16, 1/128 of its value."""
    if case["op"] == "ingest":
        return "exact"
    if case["op"] == "run":
        return {"rel": 1e-4, "max": 1e-2}
    if case["op"] == "step" and case["weights"] == "bf16":
        return {"rel": 5e-4, "max": 2e-2}
    return {"rel": 5e-3, "max": 0.1}


# ------------------------------------------------------------------ the same in 64 bits
def _rms(x, g, eps):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + eps) * g.double()


def _rope(x, pos, shape):
    """x [rows, heads, dim], pos [rows]"""
    half = shape.head_dim // 2
    theta = float(shape.rope_base) ** (-2.0 * torch.arange(half, dtype=torch.float64, device=DEV) / shape.head_dim)
    ang = pos.double()[:, None] * theta[None, :]
    c, s = torch.cos(ang)[:, None, :], torch.sin(ang)[:, None, :]
    lo, hi = x[..., :half], x[..., half:]
    return torch.cat([lo * c - hi * s, hi * c + lo * s], -1)


class _Exact:
    """The block in float64; new K and V are rounded to bf16, the type they are stored in."""

    def __init__(self, case, seed):
        self.case, self.seed, self.shape = case, seed, _shape(case)
        self.cfg = sun.make_cfg(self.shape, "f32" if case["weights"] == "f32" else "bf16")
        self.dtype = torch.float32 if case["weights"] == "f32" else torch.bfloat16
        self.ends = _ends(self.shape, self.dtype, seed)
        self.kept = {}

    def layer(self, i):
        if i in self.kept:
            return self.kept[i]
        m = _mats(self.shape, self.dtype, self.seed, i)
        for k in MATS:
            m[k] = _dequantise(*_quantise(m[k])) if self.case["weights"] == "w4" else m[k].double()
        if self.case["op"] == "run":
            self.kept[i] = m
        return m

    def cache(self, n_pages):
        """The pool as K [layer, page, head, token, dim] and V [layer, page, head, dim, token] views of one buffer."""
        mem = _pool_mem(self.shape, self.cfg, n_pages, self.seed)
        lay = sun.sun_kv_pool_create(self.cfg, mem, PAGE, 4).layout()
        dims = (self.shape.n_layers, n_pages, self.shape.n_kv_heads)
        k = mem.as_strided(dims + (PAGE, self.shape.head_dim), (lay.k_layer, lay.k_page, lay.k_head, lay.k_token, lay.k_dim), lay.k_off)
        v = mem.as_strided(dims + (PAGE, self.shape.head_dim), (lay.v_layer, lay.v_page, lay.v_head, lay.v_token, lay.v_dim), lay.v_off)
        return mem, k, v

    def put(self, view, layer, pages, slots, x):
        view[layer][pages.long(), :, slots.long()] = x.to(torch.bfloat16)

    def gather(self, view, layer, pages, n):
        """[head, n, dim] of one request"""
        t = view[layer][pages.long()].transpose(0, 1)
        return t.reshape(t.shape[0], -1, t.shape[-1])[:, :n].double()

    def qkv(self, m, x, pos):
        sh = self.shape
        h = _rms(x, m["g1"], sh.rms_eps)
        q = _rope((h @ m["wq"].t()).view(-1, sh.n_q_heads, sh.head_dim), pos, sh)
        k = _rope((h @ m["wk"].t()).view(-1, sh.n_kv_heads, sh.head_dim), pos, sh)
        return q, k, (h @ m["wv"].t()).view(-1, sh.n_kv_heads, sh.head_dim)

    def rest(self, m, x, a):
        x = x + a @ m["wo"].t()
        h = _rms(x, m["g2"], self.shape.rms_eps)
        g = h @ m["wg"].t()
        return x + (g * torch.sigmoid(g) * (h @ m["wu"].t())) @ m["wd"].t()

    def head(self, x):
        h = _rms(x, self.ends["gf"], self.shape.rms_eps)
        return torch.cat([h @ w.double().t() for w in self.ends["wlm"].split(16384)], 1)

    def step(self, k, v, tokens, tables, lens):
        sh, grp = self.shape, self.shape.n_q_heads // self.shape.n_kv_heads
        x = self.ends["embed"][tokens.long()].double()
        at = torch.arange(len(lens), device=DEV)
        pages, slots, host = tables[at, (lens // PAGE).long()], lens % PAGE, lens.tolist()
        for i in range(sh.n_layers):
            m = self.layer(i)
            q, kn, vn = self.qkv(m, x, lens)
            self.put(k, i, pages, slots, kn)
            self.put(v, i, pages, slots, vn)
            out = torch.empty((len(host), sh.n_kv_heads, grp, sh.head_dim), dtype=torch.float64, device=DEV)
            for b, n in enumerate(host):
                own = tables[b, : n // PAGE + 1]
                kc, vc = self.gather(k, i, own, n + 1), self.gather(v, i, own, n + 1)
                p = torch.softmax(q[b].view(sh.n_kv_heads, grp, -1) @ kc.transpose(1, 2) / math.sqrt(sh.head_dim), -1)
                out[b] = p @ vc
            x = self.rest(m, x, out.view(len(host), -1))
        return self.head(x)

    def prefill(self, k, v, tokens, row, first):
        sh, grp, n = self.shape, self.shape.n_q_heads // self.shape.n_kv_heads, len(tokens)
        x = self.ends["embed"][tokens.long()].double()
        pos = first + torch.arange(n, device=DEV)
        pages, slots = row[(pos // PAGE)], pos % PAGE
        for i in range(sh.n_layers):
            m = self.layer(i)
            q, kn, vn = self.qkv(m, x, pos)
            self.put(k, i, pages, slots, kn)
            self.put(v, i, pages, slots, vn)
            kc, vc = self.gather(k, i, row, first + n), self.gather(v, i, row, first + n)
            a = torch.empty((n, sh.n_q_heads, sh.head_dim), dtype=torch.float64, device=DEV)
            hidden = torch.arange(first + n, device=DEV)[None, :] > pos[:, None]
            for h in range(sh.n_q_heads):
                sc = (q[:, h] @ kc[h // grp].t() / math.sqrt(sh.head_dim)).masked_fill_(hidden, -math.inf)
                a[:, h] = torch.softmax(sc, -1) @ vc[h // grp]
            x = self.rest(m, x, a.view(n, -1))
        return self.head(x[-1:])[0]


def exact(case, seed):
    sh = _shape(case)
    if case["op"] == "ingest":
        return None  # bytes
    e = _Exact(case, seed)
    if case["op"] == "prefill":
        p = _prompt(case, sh, seed)
        mem, k, v = e.cache(p["n_pages"])
        logits = e.prefill(k, v, _dev(p["tokens"]), _dev(p["row"]), int(case["first"]))
        return {"cache": mem.double(), "logits": logits}
    req = _requests(case, sh, seed)
    mem, k, v = e.cache(req["n_pages"])
    tokens, tables, lens = _dev(req["tokens"]), _dev(req["tables"]), _dev(req["lens"])
    if case["op"] == "step":
        return {"logits": e.step(k, v, tokens, tables, lens), "cache": None}  # a handful of new entries among the old
    free, head = req["free"].tolist(), 0
    for _ in range(int(case["steps"])):
        logits = e.step(k, v, tokens, tables, lens)
        tokens, lens = logits.argmax(1).to(torch.int32), lens + 1
        for b in range(len(lens)):
            n = int(lens[b])
            if n % PAGE == 0 and n // PAGE < tables.shape[1] and int(tables[b, n // PAGE]) < 0:
                tables[b, n // PAGE], head = free[head], head + 1
    return {"tokens": None, "logits": logits, "tables": None, "lens": None, "head": None, "status": None, "cache": None}
