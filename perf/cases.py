"""Cases of the gated decode path, timed through the entry points that a serving program calls.

Kinds (the "kind" of a case; every call goes through mg.Engine, GatedDecoder or the gate's
allocation-free form):
  gate      the margin gate over a batch of LM-head logits
  step      the BF16 decode step of a batch: embedding, decoder layers over the paged cache
            with the tentative K/V append, final norm and LM head
  verify    the canonical verifier on the gated rows of a batch
  verify_mc the matrix-core verifier on the gated rows of a batch
  prefill   one call of the canonical prompt prefill: consecutive positions of all prompts of
            a batch, in the order in which prefill_rows issues them
  gated     one whole gated step of GatedDecoder: decode, gate, verify, commit

The models are the repository's shapes.  All kinds but "gated" run a few of their layers (a
decoder's layers are alike) with a small vocabulary, so that a case stands for its layers and
a change of rounding passes through few of them; the weights of a pass still exceed the
chip's caches, as a full-depth model's do.  "gated" is a quarter of the Llama-8B-shaped model,
8 of 32 layers and a quarter of the vocabulary: over 32 layers two correct orders of the BF16
path's sums already lie 0.036 apart (relative error of the logits; 0.0055 over 2 layers), which
would let nothing else be seen.
Weights N(0, 0.02), caches N(0, 1), both bf16; page tables are random permutations.
"""
import dataclasses
import math

import numpy as np
import torch

from paper_2605_30218_amd import mg, synth
from paper_2605_30218_amd.runtime import GatedDecoder

MODELS = {"llama8b": synth.LLAMA8B, "qwen7b": synth.QWEN7B, "qwen14b": synth.QWEN14B}
SPARE = 64  # positions of capacity past the longest context, as a serving program keeps


def listed():
    return [
        # a single request's gate: two launches' latency
        {"name": "gate_1", "kind": "gate", "rows": 1, "vocab": 128256},
        # one request decoded alone: every launch is small, the weights are all that is read
        {"name": "step_1", "kind": "step", "model": "llama8b", "layers": 2, "vocab": 4096, "rows": 1, "lo": 512,
         "hi": 512},
        # the benchmark's batch of 64 at contexts of 512 and up
        {"name": "step_64", "kind": "step", "model": "llama8b", "layers": 2, "vocab": 4096, "rows": 64, "lo": 512,
         "hi": 768},
        # the Qwen2.5-14B workload: 128 ragged contexts, 5 query heads per KV head, biases
        {"name": "step_128_ragged", "kind": "step", "model": "qwen14b", "layers": 2, "vocab": 4096, "rows": 128,
         "lo": 128, "hi": 2048},
        # nearly the largest batch the library takes, an odd count, short contexts
        {"name": "step_251", "kind": "step", "model": "qwen7b", "layers": 2, "vocab": 4096, "rows": 251, "lo": 40,
         "hi": 700},
        # long contexts at a small batch: the cache is most of what is read
        {"name": "step_9_long", "kind": "step", "model": "llama8b", "layers": 2, "vocab": 4096, "rows": 9, "lo": 4096,
         "hi": 16384},
        # few gated rows: a low trigger rate, or a small batch
        {"name": "verify_5", "kind": "verify", "model": "llama8b", "layers": 2, "vocab": 4096, "batch": 32, "rows": 5,
         "lo": 512, "hi": 768},
        # about a seventh of a batch of 128 gated
        {"name": "verify_18", "kind": "verify", "model": "qwen14b", "layers": 2, "vocab": 4096, "batch": 128,
         "rows": 18, "lo": 128, "hi": 2048},
        # the always-on baseline: every row of the batch is verified
        {"name": "verify_64", "kind": "verify", "model": "llama8b", "layers": 2, "vocab": 4096, "batch": 64,
         "rows": 64, "lo": 512, "hi": 768},
        # the matrix-core verifier on half of a batch of 32
        {"name": "verify_mc_17", "kind": "verify_mc", "model": "qwen7b", "layers": 2, "vocab": 4096, "batch": 32,
         "rows": 17, "lo": 1024, "hi": 1536},
        # a prefill call of 1000 items in the middle of the prompts of 40 requests
        {"name": "prefill_1000", "kind": "prefill", "model": "llama8b", "layers": 2, "vocab": 4096, "rows": 40,
         "items": 1000, "start": 240},
        # the headline workload's whole step: 64 rows, 12 of them protected and gated
        {"name": "gated_64", "kind": "gated", "model": "llama8b", "layers": 8, "vocab": 32064, "rows": 64,
         "protected": 12, "lo": 512, "hi": 536},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choices(["gate", "step", "verify", "verify_mc", "prefill"], [1, 4, 3, 1, 1])[0]
    if kind == "gate":
        return {"kind": kind, "rows": _log_int(rng, 1, 256), "vocab": rng.randint(32000, 152064)}
    c = {"kind": kind, "model": rng.choice(sorted(MODELS)), "layers": 2, "vocab": 16 * rng.randint(128, 1024)}
    if kind == "prefill":
        return dict(c, rows=_log_int(rng, 1, 64), items=_log_int(rng, 48, 800), start=rng.randint(0, 600))
    if kind == "step":
        c["rows"] = _log_int(rng, 1, 256)
    else:
        c["rows"] = _log_int(rng, 1, 64)
        c["batch"] = rng.randint(c["rows"], 128)
    # the longer the contexts, the fewer rows hold them
    longest = min(16384, 200000 // max(c["rows"], c.get("batch", 0)))
    a, b = _log_int(rng, 16, longest), _log_int(rng, 16, longest)
    return dict(c, lo=min(a, b), hi=max(a, b))


# ---------------------------------------------------------------- inputs


def _shape(case):
    return dataclasses.replace(MODELS[case["model"]], n_layers=case["layers"], vocab=case["vocab"])


def _inputs(case, seed):
    """Weights, page table, tokens, positions (and the rows concerned) of a case, from the seed."""
    s = _shape(case)
    rng = np.random.RandomState(seed % (1 << 32))
    w = synth.make_weights(s, seed=seed, device="cuda")
    d = {"shape": s, "weights": w}
    if case["kind"] == "prefill":
        # items in increasing position order; row r's prompt reaches past the last item
        n, R = case["items"], case["rows"]
        pos = case["start"] + np.arange(n) // R
        d["item_rows"], d["positions"] = (np.arange(n) % R).astype(np.int32), pos.astype(np.int32)
        d["tokens"] = rng.randint(0, s.vocab, n).astype(np.int32)
        caps = [int(pos[-1]) + 1 + SPARE] * R
    else:
        B = case.get("batch", case["rows"])
        ctx = rng.permutation(np.linspace(case["lo"], case["hi"], B).astype(np.int64))  # evenly over the range
        d["positions"] = (ctx - 1).astype(np.int32)  # the step attends to ctx positions, its own among them
        d["tokens"] = rng.randint(0, s.vocab, B).astype(np.int32)
        caps = [case["hi"] + SPARE] * B
        k = case.get("protected", case["rows"])
        d["rows"] = np.sort(rng.permutation(B)[:k]).astype(np.int32)
    maxp = -(-max(caps) // s.page_size)
    d["page_table"], d["n_pages"] = synth.make_page_table(caps, s.page_size, maxp, seed=seed % (1 << 31))
    return d


def _fill_cache(kv_view, n_pages, seed):
    synth.fill_synthetic_kv(kv_view, np.arange(n_pages), seed=seed + 77)


def _logits(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randn((case["rows"], case["vocab"]), generator=g, device="cuda") * 1.28


def prepare(case, seed):
    kind = case["kind"]
    dev = "cuda"
    if kind == "gate":
        B = case["rows"]
        i32 = dict(dtype=torch.int32, device=dev)
        return {"case": case, "logits": _logits(case, seed), "top1": torch.empty(B, **i32),
                "margin": torch.empty(B, device=dev), "gate": torch.empty(B, dtype=torch.uint8, device=dev),
                "gated_rows": torch.full((B,), -1, **i32), "n_gated": torch.zeros(1, **i32)}
    d = _inputs(case, seed)
    s = d["shape"]
    B = len(d["page_table"])
    eng = mg.Engine(s, d["weights"], B, d["page_table"].shape[1], d["n_pages"])
    _fill_cache(eng.kv_view(), d["n_pages"], seed)
    st = {"case": case, "eng": eng}
    if kind == "gated":
        prot = np.zeros(B, np.uint8)
        prot[d["rows"]] = 1
        st["dec"] = GatedDecoder(eng, d["page_table"], prot, tau=1e30)  # every protected row fires
        st["tokens"], st["positions"] = d["tokens"], d["positions"]
        return st

    def i32(a):
        return torch.as_tensor(np.ascontiguousarray(a)).to(dev)

    st.update(tokens=i32(d["tokens"]), positions=i32(d["positions"]), page_table=i32(d["page_table"]))
    if kind == "prefill":
        st["item_rows"] = i32(d["item_rows"])
    else:
        n = case["rows"]
        st["rows"] = i32(d["rows"])
        st["logits"] = torch.empty((n, s.vocab), dtype=torch.float32, device=dev)
        st["v_tok"] = torch.empty(n, dtype=torch.int32, device=dev)
        st["v_kvcol"] = torch.empty((n, eng.col_elems), dtype=torch.int16, device=dev)
    return st


def _bf16(t):
    return t.view(torch.bfloat16)


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "gate":
        mg.margin_gate_noalloc(case["rows"], case["vocab"], st["logits"], None, 0.5, st["top1"], st["margin"],
                               st["gate"], st["gated_rows"], st["n_gated"])
        return {k: st[k] for k in ("top1", "margin", "gate", "gated_rows", "n_gated")}
    eng = st["eng"]
    if kind == "step":
        eng.decode_step(case["rows"], st["tokens"], st["positions"], st["page_table"], st["logits"])
        return {"logits": st["logits"], "cache": _bf16(eng.kv_pool)}
    if kind == "verify":
        eng.verify_rows(case["rows"], st["rows"], None, st["tokens"], st["positions"], st["page_table"], st["logits"],
                        st["v_tok"], st["v_kvcol"])
        return {"logits": st["logits"], "v_tok": st["v_tok"], "v_kvcol": _bf16(st["v_kvcol"])}
    if kind == "verify_mc":
        eng.verify_rows_mfma(case["rows"], st["rows"], st["tokens"], st["positions"], st["page_table"], st["logits"],
                             st["v_tok"], st["v_kvcol"])
        return {"logits": st["logits"], "v_kvcol": _bf16(st["v_kvcol"])}
    if kind == "prefill":
        eng.prefill(case["items"], st["tokens"], st["positions"], st["item_rows"], st["page_table"])
        return {"cache": _bf16(eng.kv_pool)}
    dec = st["dec"]
    dec.set_state(st["tokens"], st["positions"])
    n = dec.step("gated")
    return {"logits": dec.logits, "n": n, "gated_rows": dec.gated_rows[:n], "v_tok": dec.v_tok[:n],
            "v_kvcol": _bf16(dec.v_kvcol)[:n], "cache": _bf16(eng.kv_pool)}


# ---------------------------------------------------------------- work and tolerance


def _layer_params(s):
    nq, nk = s.n_q_heads * s.head_dim, s.n_kv_heads * s.head_dim
    return s.d_model * (nq + 2 * nk) + nq * s.d_model + 3 * s.d_model * s.d_ffn


def _forward_work(s, ctxs, kv_positions, head=True):
    """Work of one forward over rows attending ctxs positions, reading kv_positions positions of K/V."""
    n, L = len(ctxs), s.n_layers
    w = L * _layer_params(s) + (s.vocab * s.d_model if head else 0)
    kv_col = 2 * s.n_kv_heads * s.head_dim * 2
    return {"bytes": 2.0 * w + L * kv_col * (float(kv_positions) + n) + n * (2.0 * s.d_model + 4.0 * s.vocab * head),
            "flops": 2.0 * n * w + 4.0 * L * s.n_q_heads * s.head_dim * float(np.sum(ctxs))}


def work(case):
    kind = case["kind"]
    if kind == "gate":
        return {"bytes": 4.0 * case["rows"] * (case["vocab"] + 4), "flops": 0.0}
    s = _shape(case)
    if kind == "prefill":
        ctx = case["start"] + np.arange(case["items"]) // case["rows"] + 1
        return _forward_work(s, ctx, case["rows"] * case["start"], head=False)
    mean = (case["lo"] + case["hi"]) / 2
    w = _forward_work(s, np.full(case["rows"], mean), case["rows"] * mean)
    if kind == "gated":
        v = _forward_work(s, np.full(case["protected"], mean), case["protected"] * mean)
        w = {k: w[k] + v[k] for k in w}
    return w


def tolerance(case):
    # the gate compares and the canonical arithmetic has one order: the same bits.  The BF16 path's
    # values are rounded to bf16 some ten times a layer and its sums may take another order: its
    # logits against the canonical order's on the same rows differ by rel 0.0055 and max 0.033 over
    # 2 layers (all models, 1 to 251 rows); four times that, and what 8 layers give, at most 0.03
    return {"gate": "exact", "verify": "exact", "prefill": "exact",
            "step": {"rel": 2e-2, "max": 0.13}, "verify_mc": {"rel": 2e-2, "max": 0.13},
            "gated": {"rel": 3e-2, "max": 0.3}}[case["kind"]]


# ---------------------------------------------------------------- the same in 64 bits


def _rms(x, g, eps):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + eps) * g


def _rope(x, pos, theta):
    """Rotate-half RoPE of x [n][heads][hd] at positions pos [n]."""
    hd = x.shape[-1]
    inv = theta ** (-torch.arange(0, hd, 2, dtype=torch.float64, device=x.device) / hd)
    a = (pos.double()[:, None] * inv)[:, None, :]
    lo, hi = x[..., :hd // 2], x[..., hd // 2:]
    return torch.cat([lo * a.cos() - hi * a.sin(), hi * a.cos() + lo * a.sin()], -1)


def _forward64(s, weights, cache, page_table, rows, tokens, positions, head=True):
    """One forward of the listed items (batch row, token, position) in float64 over a cache
    [L][pages][2][Hkv][page][hd]; every item's K/V is placed before any attends.  Returns the
    logits (or None) and each item's column [n][L][2][Hkv][hd]."""
    w = [None if t is None else t.view(torch.bfloat16) for t in weights]
    n, hd, Hq, Hk = len(rows), s.head_dim, s.n_q_heads, s.n_kv_heads
    rows, pt = torch.as_tensor(rows).long().cuda(), torch.as_tensor(page_table).long().cuda()
    pos = torch.as_tensor(positions).long().cuda()
    page, slot = pt[rows, pos // s.page_size], pos % s.page_size
    x = w[0][torch.as_tensor(tokens).long().cuda()].double()
    cols = torch.empty((n, s.n_layers, 2, Hk, hd), dtype=torch.float64, device="cuda")
    for l in range(s.n_layers):
        an, wq, wk, wv, bq, bk, bv, wo, fn, wg, wu, wd = [None if t is None else t.double()
                                                          for t in w[1 + 12 * l:13 + 12 * l]]
        h = _rms(x, an, s.rms_eps)
        q, k, v = [h @ m.T + (0 if b is None else b) for m, b in ((wq, bq), (wk, bk), (wv, bv))]
        q = _rope(q.view(n, Hq, hd), pos, s.rope_theta).view(n, Hk, Hq // Hk, hd)
        cols[:, l, 0], cols[:, l, 1] = _rope(k.view(n, Hk, hd), pos, s.rope_theta), v.view(n, Hk, hd)
        layer = cache[l].double()
        layer[page, :, :, slot] = cols[:, l]
        att = torch.empty((n, Hk, Hq // Hk, hd), dtype=torch.float64, device="cuda")
        for r in torch.unique(rows).tolist():
            at = (rows == r).nonzero()[:, 0]
            T = int(pos[at].max()) + 1
            kv = layer[pt[r, :-(-T // s.page_size)]]
            kv = kv.permute(1, 2, 0, 3, 4).reshape(2, Hk, -1, hd)[:, :, :T]
            sc = torch.matmul(q[at].transpose(0, 1).reshape(Hk, -1, hd), kv[0].transpose(1, 2).contiguous())
            sc = sc.view(Hk, len(at), Hq // Hk, T) / math.sqrt(hd)
            late = torch.arange(T, device="cuda")[None, :] > pos[at][:, None]
            sc = torch.softmax(sc.masked_fill(late[None, :, None, :], -math.inf), -1)
            att[at] = torch.matmul(sc.view(Hk, -1, T), kv[1].contiguous()).view(Hk, len(at), -1, hd).transpose(0, 1)
        x = x + att.view(n, Hq * hd) @ wo.T
        h = _rms(x, fn, s.rms_eps)
        g = h @ wg.T
        x = x + (g * torch.sigmoid(g) * (h @ wu.T)) @ wd.T
    if not head:
        return None, cols
    return _rms(x, w[1 + 12 * s.n_layers].double(), s.rms_eps) @ w[2 + 12 * s.n_layers].double().T, cols


def exact(case, seed):
    kind = case["kind"]
    if kind == "gate":
        top = torch.topk(_logits(case, seed).double(), 2).values
        return {"top1": None, "margin": top[:, 0] - top[:, 1], "gate": None, "gated_rows": None, "n_gated": None}
    d = _inputs(case, seed)
    s, pt = d["shape"], d["page_table"]
    cache = torch.zeros((s.n_layers, d["n_pages"], 2, s.n_kv_heads, s.page_size, s.head_dim), dtype=torch.int16,
                        device="cuda")
    _fill_cache(cache, d["n_pages"], seed)
    cache = _bf16(cache)

    def appended(rows, pos, cols):
        c = cache.double()
        page = torch.as_tensor(pt[rows, pos // s.page_size]).long().cuda()
        c[:, page, :, :, torch.as_tensor(pos % s.page_size).long().cuda()] = cols
        return c.reshape(-1)

    if kind == "prefill":
        _, cols = _forward64(s, d["weights"], cache, pt, d["item_rows"], d["tokens"], d["positions"], head=False)
        return {"cache": appended(d["item_rows"], d["positions"], cols)}
    rows = d["rows"] if kind in ("verify", "verify_mc") else np.arange(len(pt))
    tok, pos = d["tokens"][rows], d["positions"][rows]
    logits, cols = _forward64(s, d["weights"], cache, pt, rows, tok, pos)
    if kind == "step":
        return {"logits": logits, "cache": appended(rows, pos, cols)}
    if kind == "verify":
        return {"logits": logits, "v_tok": None, "v_kvcol": cols.reshape(len(rows), -1)}
    if kind == "verify_mc":
        return {"logits": logits, "v_kvcol": cols.reshape(len(rows), -1)}
    return {"logits": logits, "n": None, "gated_rows": None, "v_tok": None,
            "v_kvcol": cols[torch.as_tensor(d["rows"]).long().cuda()].reshape(len(d["rows"]), -1),
            "cache": appended(rows, pos, cols)}
