"""Performance cases of the denoising-step library.

What a program that generates text with this library has the GPU do: a block decoded by a
small model (launch latency), stacks of transformer layers over decoding windows of
several widths, prefixes, weight types and model shapes, one whole step of the 8B model
up to its logits, the step that also appends a finished block and refreshes revised
positions, and prompts.  Every pass goes through the public entry points; weights, token
ids and the cached prefix are random, of the distributions a random-init model has.

A case is a dict of plain values:
  kind     "block" (a whole block of a small model: steps and commits), "layers" (a
           window through `layers` layers, residual stream out), "logits" (a whole step,
           logits out), "merged" (refresh + append + window in one step), "prefill"
  model    a shape of synth.PRESETS, cut to `layers` layers; "layers" cases, which never
           reach the LM head, also cut its vocabulary
  dtype    "f32", "bf16", "w8" or "q4" weights
  prefix   positions already cached; rows: window rows (prompt ids for "prefill")
"""
import math
import weakref

import torch

import paper_2606_13740_amd as dl
import synth

STD = synth.WEIGHT_STD
WBYTES = {"f32": 4.0, "bf16": 2.0, "w8": 1.0, "q4": 18.0 / 32.0}


def listed():
    return [
        # a small fp32 model decodes a 32-row block in 4 steps of 8 commits: launches and latency
        {"name": "block_tiny_f32", "kind": "block", "model": "tiny", "layers": 2, "dtype": "f32", "prefix": 64,
         "rows": 32, "steps": 4},
        # the usual denoising step: one 32-token block behind a 512-token prefix
        {"name": "layers_bf16_w32_p512", "kind": "layers", "model": "llada8b", "layers": 4, "dtype": "bf16",
         "prefix": 512, "rows": 32},
        # current block + speculative draft block
        {"name": "layers_bf16_w64_p1024", "kind": "layers", "model": "llada8b", "layers": 4, "dtype": "bf16",
         "prefix": 1024, "rows": 64},
        # the same with int8 weights behind a long prefix
        {"name": "layers_w8_w64_p4096", "kind": "layers", "model": "llada8b", "layers": 4, "dtype": "w8",
         "prefix": 4096, "rows": 64},
        # Q4_0 weights
        {"name": "layers_q4_w32_p512", "kind": "layers", "model": "llada8b", "layers": 4, "dtype": "q4",
         "prefix": 512, "rows": 32},
        # grouped-query attention and biases (Dream-7B), a window that has slid to an odd size
        {"name": "layers_dream_w29_p777", "kind": "layers", "model": "dream7b", "layers": 4, "dtype": "bf16",
         "prefix": 777, "rows": 29},
        # a wide lookahead window, ragged
        {"name": "layers_bf16_w200_p1500", "kind": "layers", "model": "llada8b", "layers": 4, "dtype": "bf16",
         "prefix": 1500, "rows": 200},
        # one whole step of the 8B model, logits out
        {"name": "logits_bf16_w32_p512", "kind": "logits", "model": "llada8b", "layers": 32, "dtype": "bf16",
         "prefix": 512, "rows": 32},
        # block boundary: 4 revised positions, the finished block appended, the next window
        {"name": "merged_bf16_w28_p544", "kind": "merged", "model": "llada8b", "layers": 4, "dtype": "bf16",
         "prefix": 544, "rows": 28, "block": 32, "refresh": 4},
        # prompts: the ordinary one, a ragged one on Q4_0 weights, a long one on int8 weights
        {"name": "prefill_bf16_512", "kind": "prefill", "model": "llada8b", "layers": 32, "dtype": "bf16",
         "prefix": 0, "rows": 512},
        {"name": "prefill_q4_473", "kind": "prefill", "model": "llada8b", "layers": 32, "dtype": "q4",
         "prefix": 0, "rows": 473},
        {"name": "prefill_w8_4096", "kind": "prefill", "model": "llada8b", "layers": 32, "dtype": "w8",
         "prefix": 0, "rows": 4096},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["block", "layers", "layers", "layers", "layers", "logits", "merged", "prefill", "prefill"])
    if kind == "block":
        return {"kind": kind, "model": rng.choice(["tiny", "tiny_gqa"]), "layers": 2, "dtype": "f32",
                "prefix": _log_int(rng, 16, 160), "rows": rng.randint(8, 48), "steps": rng.choice([2, 4, 8])}
    model = rng.choice(["llada8b", "llada8b", "dream7b"])
    dtype = rng.choice(["bf16", "bf16", "w8", "q4"])
    case = {"kind": kind, "model": model, "layers": 4, "dtype": dtype, "prefix": _log_int(rng, 16, 4096)}
    if kind == "layers":
        case["rows"] = _log_int(rng, 1, 256)
    elif kind == "logits":
        case.update(layers=synth.PRESETS[model].n_layers, rows=_log_int(rng, 1, 64))
    elif kind == "merged":
        # the refreshed positions are those of the last whole block of the prefix
        case.update(prefix=32 * rng.randint(1, 64), rows=_log_int(rng, 1, 64), block=32, refresh=rng.randint(1, 8))
    else:
        top = {"bf16": 4096, "w8": 3000, "q4": 1024}[dtype]
        case.update(layers=synth.PRESETS[model].n_layers, prefix=0, rows=_log_int(rng, 40, top))
    return case


# ----------------------------------------------------------------------------
# Inputs
# ----------------------------------------------------------------------------


def _shape(case):
    import dataclasses

    sh = synth.PRESETS[case["model"]].with_layers(case["layers"])
    if case["kind"] == "layers":
        sh = dataclasses.replace(sh, vocab=4096, mask_id=4095)
    return sh


def _gen(seed, stream):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 1000003 + stream)
    return g


def _weights(case, sh, seed, name, layer=-1):
    """One tensor as the caller holds it: fp32 or bf16 matrices, fp32 gains and biases."""
    names = ("embed", "lm_head", "final_norm", "wq", "wk", "wv", "wo", "wg", "wu", "wd", "attn_norm", "ffn_norm",
             "bq", "bk", "bv")
    g = _gen(seed, 100 + 32 * (layer + 1) + names.index(name))
    shp = synth.tensor_shape(sh, name)
    if name.endswith("norm"):
        return torch.empty(shp, device="cuda").normal_(1.0, 0.1, generator=g)
    if name.startswith("b"):
        return torch.empty(shp, device="cuda").normal_(0.0, STD, generator=g)
    dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    return torch.empty(shp, device="cuda", dtype=dt).normal_(0.0, STD, generator=g)


def _layer_names(sh):
    return synth.LAYER_TENSORS + synth.LAYER_GAINS + (synth.LAYER_BIASES if sh.qkv_bias else ())


def _tokens(case, sh, seed):
    """Ids of the window (or prompt), its mask flags, the block to append, the refresh picks."""
    n = case["rows"]
    g = _gen(seed, 1)
    t = {"tok": torch.randint(0, sh.mask_id, (n,), device="cuda", dtype=torch.int32, generator=g)}
    mask = torch.zeros(n, device="cuda", dtype=torch.uint8)
    if case["kind"] != "prefill":
        mask[n // 4:] = 1          # a quarter of the block is committed
        if case["kind"] == "block":
            mask[:] = 1
    t["mask"] = mask
    if case["kind"] == "merged":
        P, nb, nr = case["prefix"], case["block"], case["refresh"]
        t["block"] = torch.randint(0, sh.mask_id, (nb,), device="cuda", dtype=torch.int32, generator=g)
        t["ref_pos"] = (P - 32 + torch.randperm(32, device="cuda", generator=g)[:nr]).to(torch.int32)
        t["ref_id"] = torch.randint(0, sh.mask_id, (nr,), device="cuda", dtype=torch.int32, generator=g)
    return t


def _cache_rows(case):
    return case["prefix"] + case["rows"] + case.get("block", 0)


def _prefix_kv(case, sh, seed, layer):
    """Cached K [Hkv, P, Dh] and V [Hkv, P, Dh] of one layer: the spread K and V rows of a
    normalised input have."""
    g = _gen(seed, 50000 + layer)
    dt = torch.float32 if case["dtype"] == "f32" else torch.float16
    shp = (sh.kv_heads, case["prefix"], sh.head_dim)
    std = STD * math.sqrt(sh.d_model)
    return tuple(torch.empty(shp, device="cuda").normal_(0.0, std, generator=g).to(dt) for _ in range(2))


class _Handle:
    """A library handle destroyed with its holder."""

    def __init__(self, value, destroy):
        self.value = value
        weakref.finalize(self, destroy, value).atexit = False


def _model(case, sh, seed):
    dtype = case["dtype"]
    rows = 64 if case["kind"] == "prefill" else case["rows"] + case.get("block", 0) + case.get("refresh", 0)
    cfg = dl.make_config(sh, dtype, max_window=max(64, rows), max_pos=_cache_rows(case) + 64)
    keep = []
    layers = (dl.dllm_layer_weights * sh.n_layers)()
    for l in range(sh.n_layers):
        t = {k: _weights(case, sh, seed, k, l) for k in _layer_names(sh)}
        keep.append(t)
        layers[l] = dl.dllm_layer_weights(*[t[k].data_ptr() if k in t else None
                                            for k in ("wq", "wk", "wv", "wo", "wg", "wu", "wd", "attn_norm",
                                                      "ffn_norm", "bq", "bk", "bv")])
    top = {k: _weights(case, sh, seed, k) for k in ("embed", "lm_head", "final_norm")}
    w = dl.dllm_weights(top["embed"].data_ptr(), top["lm_head"].data_ptr(), top["final_norm"].data_ptr(), layers)
    handle = dl.dllm_model_create(cfg, w)
    del keep, top
    torch.cuda.empty_cache()       # the library keeps its own packed copy
    return _Handle(handle, dl.dllm_model_destroy)


def prepare(case, seed):
    sh = _shape(case)
    s = dict(_tokens(case, sh, seed))
    s["case"], s["shape"] = case, sh
    s["model"] = _model(case, sh, seed)
    n, P = case["rows"], case["prefix"]
    cap = _cache_rows(case)
    s["cap"], s["kv_bytes"] = cap, dl.dllm_kv_bytes(s["model"].value, cap)
    el = 4 if case["dtype"] == "f32" else 2
    s["kv_buf"] = torch.zeros(s["kv_bytes"] // el, device="cuda", dtype=torch.float32 if el == 4 else torch.float16)
    Cs, H, Dh = (cap + 31) // 32 * 32, sh.kv_heads, sh.head_dim
    plane = s["kv_buf"].view(sh.n_layers, 2, H * Cs * Dh)
    s["K"] = plane[:, 0].view(sh.n_layers, H, Cs, Dh)
    s["V"] = plane[:, 1].view(sh.n_layers, H, Dh, Cs)
    for l in range(sh.n_layers if P else 0):
        k, v = _prefix_kv(case, sh, seed, l)
        s["K"][l, :, :P] = k
        s["V"][l, :, :, :P] = v.transpose(1, 2)
    if case["kind"] != "prefill":  # a prompt starts its own cache
        s["kv"] = _Handle(dl.dllm_kv_create(s["model"].value, s["kv_buf"], s["kv_bytes"], cap), dl.dllm_kv_destroy)
        dl.dllm_kv_set_prefix_len(s["kv"].value, P)
    s["out_id"] = torch.empty(n, device="cuda", dtype=torch.int32)
    s["out_conf"] = torch.empty(n, device="cuda")
    if case["kind"] == "layers":
        s["x"] = torch.empty(n, sh.d_model, device="cuda")
    elif case["kind"] == "logits":
        s["logits"] = torch.empty(n, sh.vocab, device="cuda")
    elif case["kind"] == "merged":
        s["ref_out_id"] = torch.empty(case["refresh"], device="cuda", dtype=torch.int32)
        s["ref_out_conf"] = torch.empty(case["refresh"], device="cuda")
    elif case["kind"] == "block":
        s["w_tok"], s["w_mask"] = s["tok"].clone(), s["mask"].clone()
    return s


# ----------------------------------------------------------------------------
# One pass
# ----------------------------------------------------------------------------


def run(s):
    case, m = s["case"], s["model"].value
    n, P, kind = case["rows"], case["prefix"], case["kind"]
    if kind == "prefill":
        kv = dl.dllm_kv_create(m, s["kv_buf"], s["kv_bytes"], s["cap"])
        try:
            dl.dllm_prefill(m, kv, s["tok"], n)
        finally:
            dl.dllm_kv_destroy(kv)
        return {"k": s["K"][:, :, :n], "v": s["V"][:, :, :, :n]}
    kv = s["kv"].value
    rows = {"k": s["K"][:, :, P:P + n], "v": s["V"][:, :, :, P:P + n]}
    if kind == "layers":
        dl.dllm_debug_hidden(m, kv, s["tok"], s["mask"], n, case["layers"], s["x"])
        return {"x": s["x"], **rows}
    if kind == "logits":
        # The ids are the logits' argmax: near-ties make them incomparable between roundings.
        dl.dllm_debug_logits(m, kv, s["tok"], s["mask"], n, s["logits"], s["out_id"], s["out_conf"])
        return {"logits": s["logits"], "conf": s["out_conf"], **rows}
    if kind == "merged":
        # the refresh gives the same rows each time: its ids and what they attend to stay
        nb, nr = case["block"], case["refresh"]
        dl.dllm_kv_set_prefix_len(kv, P)
        dl.dllm_step_merged(m, kv, s["ref_pos"], s["ref_id"], nr, s["block"], nb, s["tok"], s["mask"], n,
                            s["out_id"], s["out_conf"], s["ref_out_id"], s["ref_out_conf"])
        lo, hi = P - 32, P + nb + n
        return {"conf": s["out_conf"], "ref_conf": s["ref_out_conf"], "k": s["K"][:, :, lo:hi],
                "v": s["V"][:, :, :, lo:hi]}
    s["w_tok"].copy_(s["tok"])     # a fresh block
    s["w_mask"].copy_(s["mask"])
    per = -(-n // case["steps"])
    for _ in range(case["steps"]):
        dl.dllm_denoise_step(m, kv, s["w_tok"], s["w_mask"], n, s["out_id"], s["out_conf"])
        dl.dllm_commit(s["out_conf"], s["out_id"], s["w_tok"], s["w_mask"], 0, n, per)
    return {"tok": s["w_tok"], "mask": s["w_mask"], "conf": s["out_conf"], **rows}


# ----------------------------------------------------------------------------
# What a pass cannot do without
# ----------------------------------------------------------------------------


def work(case):
    sh = _shape(case)
    n, P = case["rows"], case["prefix"]
    steps = case.get("steps", 1)
    M = n + case.get("block", 0) + case.get("refresh", 0)
    keys = P + case.get("block", 0) + n
    wb, kvb = WBYTES[case["dtype"]], 4 if case["dtype"] == "f32" else 2
    head = 0 if case["kind"] in ("layers", "prefill") else sh.vocab * sh.d_model
    params = sh.n_layers * sh.params_per_layer + head
    lm_rows = n + case.get("refresh", 0)
    # cached rows read; K/V rows written; embedding rows; residual or logits out
    nbytes = params * wb + sh.n_layers * 2 * sh.d_kv * kvb * (P + M) + M * sh.d_model * (4 if wb == 4 else 2)
    if case["kind"] == "layers":
        nbytes += n * sh.d_model * 4
    if case["kind"] == "logits":
        nbytes += n * sh.vocab * 4
    flops = 2.0 * M * sh.n_layers * sh.params_per_layer + 2.0 * lm_rows * head
    flops += 4.0 * M * keys * sh.d_model * sh.n_layers
    return {"bytes": float(nbytes) * steps, "flops": flops * steps}


def tolerance(case):
    """About four times the distance from the 64-bit values that these paths show: fp32
    models differ in summation order only (3e-7); the others store K and V in fp16 (2^-12 of
    a value) and split activations into two bf16 halves, and each layer passes on what the
    layers before it rounded (4 layers 2e-4 to 4e-4, confidences 6e-4; 32 layers: a step
    8e-4, a prompt 2e-3)."""
    if case["kind"] == "block":
        return {"rel": 1.5e-6, "max": 3e-5}
    return {"rel": {"layers": 1.5e-3, "merged": 2.5e-3, "logits": 4e-3, "prefill": 8e-3}[case["kind"]]}


# ----------------------------------------------------------------------------
# The same in 64 bits
# ----------------------------------------------------------------------------


def _exact_matrix(case, w):
    """The weight values a matrix product uses: the caller's, or those its quantised form stands for."""
    if case["dtype"] == "w8":
        w = w.float()
        amax = w.abs().amax(dim=1, keepdim=True)
        s = amax / torch.full_like(amax, 127.0)        # (a scalar divisor would become a reciprocal)
        q = torch.where(s > 0, torch.round(w / s), torch.zeros_like(w)).clamp_(-127, 127)
        return q.double() * s.double()
    if case["dtype"] == "q4":
        b = w.float().view(w.shape[0], -1, 32)
        a = b.abs()
        hit = a == a.amax(dim=2, keepdim=True)
        first = hit & (hit.int().cumsum(2) == 1)       # the first of largest magnitude
        d = (b * first).sum(2, keepdim=True) / -8.0
        inv = torch.where(d != 0, 1.0 / d, torch.zeros_like(d))
        t = b * inv
        q = torch.trunc(t + 8.5).clamp_(max=15.0)
        return ((q.double() - 8.0) * d.half().double()).view(w.shape)
    return w.double()


class _Exact:
    def __init__(self, case, seed):
        self.case, self.seed, self.sh = case, seed, _shape(case)
        sh = self.sh
        n = _cache_rows(case)
        ang = torch.arange(n, device="cuda", dtype=torch.float64)[:, None] * \
            sh.rope_base ** (-2.0 * torch.arange(sh.head_dim // 2, device="cuda", dtype=torch.float64) / sh.head_dim)
        self.cos, self.sin = ang.cos(), ang.sin()
        self.embed = _weights(case, sh, seed, "embed")
        self.kept = {}

    def norm(self, x, g):
        return x / torch.sqrt((x * x).mean(dim=1, keepdim=True) + self.sh.eps) * g.double()

    def rope(self, x, pos):        # x [H, M, Dh]
        c, s = self.cos[pos], self.sin[pos]
        a, b = x.chunk(2, dim=2)
        return torch.cat((a * c - b * s, a * s + b * c), dim=2)

    def layer(self, l):
        if l not in self.kept:
            w = {}
            for k in _layer_names(self.sh):
                t = _weights(self.case, self.sh, self.seed, k, l)
                w[k] = _exact_matrix(self.case, t) if k in synth.LAYER_TENSORS else t.double()
            if self.case["kind"] != "block":
                return w
            self.kept[l] = w
        return self.kept[l]

    def forward(self, ids, pos, lim, cache):
        """Residual stream of rows `ids` at `pos` [M], row i seeing keys [0, lim[i]); `cache`:
        per layer [K, V] of [Hkv, C, Dh], the rows' own written at `pos`."""
        sh = self.sh
        M, H, Hk, Dh = len(ids), sh.n_heads, sh.kv_heads, sh.head_dim
        x = self.embed[ids.long()].double()
        top = int(lim.max())
        hide = torch.arange(top, device="cuda")[None, :] >= lim[:, None]
        for l in range(sh.n_layers):
            w = self.layer(l)
            h = self.norm(x, w["attn_norm"])

            def proj(name, heads):
                y = h @ w["w" + name].t()
                if sh.qkv_bias:
                    y = y + w["b" + name]
                return y.view(M, heads, Dh).transpose(0, 1)

            q = self.rope(proj("q", H), pos)
            K, V = cache[l]
            K[:, pos] = self.rope(proj("k", Hk), pos)
            V[:, pos] = proj("v", Hk)
            o = torch.empty(M, H, Dh, device="cuda", dtype=torch.float64)
            for i in range(H):
                j = i // (H // Hk)
                sc = q[i] @ K[j, :top].t() / math.sqrt(Dh)
                sc.masked_fill_(hide, -math.inf)
                o[:, i] = torch.softmax(sc, dim=1) @ V[j, :top]
            x = x + o.view(M, H * Dh) @ w["wo"].t()
            h = self.norm(x, w["ffn_norm"])
            gate = h @ w["wg"].t()
            x = x + (gate * torch.sigmoid(gate) * (h @ w["wu"].t())) @ w["wd"].t()
        return x

    def logits(self, x):
        c, sh = self.case, self.sh
        if "head" not in self.kept:
            self.kept["head"] = (_exact_matrix(c, _weights(c, sh, self.seed, "lm_head")),
                                 _weights(c, sh, self.seed, "final_norm"))
        head, g = self.kept["head"]
        y = self.norm(x, g) @ head.t()
        y[:, sh.mask_id] = -math.inf
        return y


def exact(case, seed):
    e = _Exact(case, seed)
    sh, t = e.sh, _tokens(case, e.sh, seed)
    n, P, kind = case["rows"], case["prefix"], case["kind"]
    C = _cache_rows(case)
    cache = []
    for l in range(sh.n_layers):
        kv = [torch.zeros(sh.kv_heads, C, sh.head_dim, device="cuda", dtype=torch.float64) for _ in range(2)]
        if P:
            for dst, src in zip(kv, _prefix_kv(case, sh, seed, l)):
                dst[:, :P] = src.double()
        cache.append(kv)

    def rows(lo, hi):
        return {"k": torch.stack([c[0][:, lo:hi] for c in cache]),
                "v": torch.stack([c[1][:, lo:hi].transpose(1, 2) for c in cache])}

    def fed(tok, mask):
        return torch.where(mask != 0, torch.full_like(tok, sh.mask_id), tok)

    def ar(lo, k):
        return torch.arange(lo, lo + k, device="cuda")

    full = torch.full((n,), C, device="cuda")
    if kind == "prefill":
        e.forward(t["tok"], ar(0, n), full, cache)
        return rows(0, n)
    if kind == "merged":
        nb, nr = case["block"], case["refresh"]
        ref = t["ref_pos"].long()
        blk = sh.block
        ids = torch.cat((t["ref_id"], t["block"], fed(t["tok"], t["mask"])))
        pos = torch.cat((ref, ar(P, nb + n)))
        lim = torch.cat(((blk * (1 + ref // blk)).clamp(max=P), torch.full((nb,), P + nb, device="cuda"), full))
        conf = e.logits(e.forward(ids, pos, lim, cache)).softmax(dim=1).amax(dim=1)
        return {"conf": conf[nr + nb:], "ref_conf": conf[:nr], **rows(P - 32, C)}
    pos = ar(P, n)
    if kind == "block":
        tok, mask = t["tok"].clone(), t["mask"].clone()
        per = -(-n // case["steps"])
        for _ in range(case["steps"]):
            p = e.logits(e.forward(fed(tok, mask), pos, full, cache)).softmax(dim=1)
            conf, best = p.max(dim=1)
            for i in torch.where(mask != 0, conf, -1.0).argsort(descending=True, stable=True)[:per].tolist():
                if mask[i]:
                    tok[i] = best[i].to(torch.int32)
                    mask[i] = 0
        return {"tok": tok, "mask": mask, "conf": conf, **rows(P, P + n)}
    x = e.forward(fed(t["tok"], t["mask"]), pos, full, cache)
    if kind == "layers":
        return {"x": x, **rows(P, P + n)}
    y = e.logits(x)
    return {"logits": y, "conf": y.softmax(dim=1).amax(dim=1), **rows(P, P + n)}
