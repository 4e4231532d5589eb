"""The work that users of this framework have it do, as measurable cases: one pass of a case is one round (or one step)
of a decoding program through the public session calls.

  verify   a draft block proposed elsewhere: ee_draft_inject, ee_verify_intermediate, ee_verify_full
  round    the whole loop of the method: ee_draft (k sequential rows), then the two verifications
  decode   vanilla greedy steps (ee_decode_ar)
  prefill  a request arrives: ee_prefill of the prompts and the first decoding step
  sample   the round under the rejection-sampling acceptance (ee_draft_sample, the two *_rs verifications)

After the pass kv_rollback puts the sequences back to their contexts, as a program does with rejected tokens, so that the
pass can be repeated.  A pass ends with what the calls return on the host (accept counts, tokens) and the hidden rows of
its exits; where `logits` is set it also returns the logits (for `sample` the distributions) of its last head.

Shapes: the repository's tiny fp32 and small bf16 test models, and the Llama-3-8B / 70B layer widths of its benchmark, at
full depth with the full vocabulary where the whole model counts and otherwise with fewer layers and a 32000-token
vocabulary, which keeps the share of the exit heads about what it is in the full model.

Weights: the library's seeded generator with the residual writes damped (gamma) to the size of the embeddings, and the LM
head tied to the embedding table with a shift of one token, so that every exit is confident and its next token is t + 1.
That is what trained early-exit models look like to this path: the exits mostly agree, and which token wins does not hang
on the last bit.  A block's first wrong token sits where `accept` says.
"""
from __future__ import annotations

import math
import random
from types import SimpleNamespace

import numpy as np
import torch

import paper_2510_01336_amd as hs

#          d_model, q heads, kv heads, head_dim, d_ffn, theta, sigma
WIDTHS = {
    "tiny": (256, 4, 4, 64, 688, 1e4, 0.08),          # the fp32 test model
    "small": (256, 8, 2, 64, 688, 1e4, 0.08),         # the bf16 test model
    "8b": (4096, 32, 8, 128, 14336, 5e5, 0.02),
    "70b": (8192, 64, 8, 128, 28672, 5e5, 0.02),
}
BASE = {"dtype": "bf16", "ragged": False, "accept": 0, "head_rank": 0, "bonus_full": 1, "logits": False, "spread": 2.0}


def listed():
    cases = [
        # the smallest calls, bound by launches and latency: the fp32 reference model, and a small bf16 model of two sequences
        dict(name="tiny_f32_round", kind="round", width="tiny", dtype="f32", layers=4, exit_d=1, exit_i=2, vocab=1024, batch=1, ctx=32,
             k=4, accept=4, logits=True, spread=1.0),
        dict(name="small_bf16_verify", kind="verify", width="small", layers=6, exit_d=2, exit_i=4, vocab=1000, batch=2, ctx=150, k=8,
             accept=5, logits=True, spread=1.0),
        # the benchmark's own step: one sequence, 2048 cached tokens, a block of eight of which six are right
        dict(name="verify_8b", kind="verify", width="8b", layers=32, exit_d=4, exit_i=16, vocab=128256, batch=1, ctx=2048, k=8, accept=6),
        # the decoding loop as it runs best end to end (short blocks, no catch-up row), low-rank heads at the early exits
        dict(name="round_8b_heads", kind="round", width="8b", layers=16, exit_d=2, exit_i=8, vocab=128256, batch=1, ctx=1000, k=6,
             accept=6, head_rank=1024, bonus_full=0),
        # vanilla decoding of eight requests in one batch, two steps per call
        dict(name="decode_8b_b8", kind="decode", width="8b", layers=8, exit_d=1, exit_i=4, vocab=32000, batch=8, ctx=1024, ragged=True,
             k=2, logits=True),
        # a serving batch: sixteen requests with contexts of very different lengths, nine block rows each
        dict(name="verify_8b_b16_ragged", kind="verify", width="8b", layers=8, exit_d=1, exit_i=4, vocab=32000, batch=16, ctx=1024,
             ragged=True, k=8, accept=5),
        # the wide model with four requests (36 rows)
        dict(name="verify_70b_b4", kind="verify", width="70b", layers=4, exit_d=1, exit_i=2, vocab=32000, batch=4, ctx=1024, k=8, accept=5),
        # long context, deep speculation: attention carries the step (17 rows, an odd context length)
        dict(name="verify_8b_ctx32k", kind="verify", width="8b", layers=8, exit_d=2, exit_i=4, vocab=32000, batch=1, ctx=32001, k=16,
             accept=14),
        # context build: the benchmark's prompt through the whole model
        dict(name="prefill_8b_2048", kind="prefill", width="8b", layers=32, exit_d=4, exit_i=16, vocab=128256, batch=1, ctx=2048, k=1,
             logits=True),
        # ... a long document, where causal attention weighs in
        dict(name="prefill_8b_8k", kind="prefill", width="8b", layers=8, exit_d=1, exit_i=4, vocab=32000, batch=1, ctx=8190, k=1,
             logits=True),
        # ... and a batch of short prompts of odd lengths that share passes
        dict(name="prefill_8b_ragged", kind="prefill", width="8b", layers=8, exit_d=1, exit_i=4, vocab=32000, batch=12, ctx=120,
             ragged=True, k=1, logits=True),
        # the sampling acceptance, four requests
        dict(name="sample_8b_b4", kind="sample", width="8b", layers=8, exit_d=1, exit_i=4, vocab=32000, batch=4, ctx=500, ragged=True,
             k=5, accept=5, logits=True, spread=3.5),
    ]
    return [{**BASE, **c} for c in cases]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    width = rng.choice(["8b", "8b", "8b", "8b", "70b", "small"])
    kind = rng.choice(["verify", "verify", "verify", "round", "decode", "prefill", "prefill", "sample"])
    c = dict(BASE, kind=kind, width=width)
    if width == "small":
        c.update(layers=6, exit_d=2, exit_i=4, vocab=rng.choice([1000, 1024]))
        if rng.random() < 0.4:
            c.update(width="tiny", dtype="f32", layers=4, exit_d=1, exit_i=2)
    else:
        c["layers"] = rng.randint(3, 8 if width == "8b" else 4)
        c["exit_d"] = rng.randint(1, max(1, c["layers"] // 3))
        c["exit_i"] = rng.randint(c["exit_d"] + 1, c["layers"] - 1)
        c["vocab"] = 32000
    c["batch"] = 1 if rng.random() < 0.3 else _log_int(rng, 1, 20)
    # tokens of all contexts together; prompts that a pass builds cost at most what the listed ones do
    most = 600 if width == "small" else 32768
    if kind == "prefill":
        most = min(most, 60000 // c["layers"] // (4 if width == "70b" else 1))
    c["ctx"] = _log_int(rng, 16, max(17, most // c["batch"]))
    c["ragged"] = rng.random() < 0.6
    c["k"] = {"decode": rng.randint(1, 4), "prefill": 1, "sample": rng.randint(2, 8), "round": rng.randint(2, 8)}.get(kind, rng.randint(2, 16))
    c["accept"] = c["k"] if kind in ("round", "sample") else rng.randint(0, c["k"])
    c["head_rank"] = 1024 if width == "8b" and rng.random() < 0.2 else 0
    c["bonus_full"] = rng.randint(0, 1)
    c["logits"] = kind in ("decode", "prefill", "sample")
    c["spread"] = (0.7 if kind == "sample" else 1.0) if c["vocab"] < 2000 else (3.5 if kind == "sample" else 2.0)
    return c


# ---- shapes and token streams of a case -----------------------------------------------------------------------------

def _lens(c):
    """Context lengths; ragged ones spread over a quarter to almost twice the nominal length, the same for every seed."""
    if not c["ragged"]:
        return [c["ctx"]] * c["batch"]
    r = np.random.default_rng(c["ctx"] * 31 + c["batch"])
    return [int(max(2, min(2 * c["ctx"] - 1, round(c["ctx"] * x)))) for x in np.exp(r.normal(-0.15, 0.5, c["batch"]))]


def _accepts(c):
    """First wrong position of every sequence's block (k: none)."""
    if c["kind"] != "verify" or not c["ragged"]:
        return [c["accept"]] * c["batch"]
    return [(c["accept"] + 3 * b) % (c["k"] + 1) for b in range(c["batch"])]


def _inputs(c, seed):
    """Prompts, draft blocks and uniform numbers, from the seed alone."""
    r = np.random.default_rng([seed, 0x5EED])
    V, k = c["vocab"], c["k"]
    prompts = [r.integers(0, V, n).astype(np.int32) for n in _lens(c)]
    blocks = np.empty((c["batch"], k), np.int32)
    for b, a in enumerate(_accepts(c)):
        first = (int(prompts[b][-1]) + 1) % V
        blocks[b] = r.integers(0, V, k)
        blocks[b, :a] = (first + 1 + np.arange(a)) % V
        if a < k:
            blocks[b, a] = (first + 1 + a + int(r.integers(1, V))) % V
    u = r.uniform(0.05, 0.9, (4, c["batch"], 64)).astype(np.float32)      # (away from the ends: no draw hangs on a last bit)
    return prompts, blocks, u


def _config(c):
    d, hq, hkv, D, F, theta, sigma = WIDTHS[c["width"]]
    g = c["spread"] / (0.43 * sigma * sigma * d * math.sqrt(F * c["layers"]))      # all layers' writes: `spread` times the embedding
    return SimpleNamespace(n_layers=c["layers"], d_model=d, n_q_heads=hq, n_kv_heads=hkv, head_dim=D, d_ffn=F, vocab=c["vocab"],
                           exit_draft=c["exit_d"], exit_inter=c["exit_i"], rope_theta=theta, rms_eps=1e-5, dtype=c["dtype"], sigma=sigma,
                           gamma=(g, g, g), head_rank=c["head_rank"])


def prepare(case, seed):
    c = {**BASE, **case}
    cfg = _config(c)
    model = hs.Model(cfg, seed, 1, c["bonus_full"])
    emb = torch.from_numpy(model.tensor_rows("emb", 0, 0, c["vocab"], cfg.d_model))
    model.set_tensor("head", 0, torch.roll(emb, 1, 0).numpy())            # head row t + 1 = embedding of t
    del emb
    prompts, blocks, u = _inputs(c, seed)
    rows = 2 * (c["k"] + 1) + 3
    sess = hs.Session(model, c["batch"], max(_lens(c)) + rows + 8, rows)
    if c["kind"] == "sample":
        sess.enable_sampling()
    if c["logits"]:
        sess.enable_logits(True)
    if c["kind"] != "prefill":
        sess.prefill(prompts)
    full_rows = sum(a + 1 for a in _accepts(c)) + c["bonus_full"] * c["batch"]
    return SimpleNamespace(c=c, sess=sess, prompts=prompts, blocks=blocks, u=u, lens=[len(p) for p in prompts], full_rows=full_rows)


def run(s):
    c, sess, k = s.c, s.sess, s.c["k"]
    B, kind = c["batch"], c["kind"]
    out = {}
    if kind == "prefill":
        out["first"] = sess.prefill(s.prompts)
        out["token"] = sess.decode_ar(1)
        out["hidden"] = sess.last_hidden(B)
        out["logits"] = sess.last_logits(B)
        return out
    if kind == "decode":
        out["tokens"] = sess.decode_ar(k)
        out["hidden"] = sess.last_hidden(B)
        out["logits"] = sess.last_logits(B)
    else:
        if kind == "verify":
            sess.draft_inject(s.blocks)
        elif kind == "round":
            out["draft"] = sess.draft(k)
        else:
            out["draft"] = sess.draft_sample(k, s.u[0, :, :k])
        if kind == "sample":
            out["accept_i"], out["next_i"] = sess.verify_intermediate_rs(s.u[1, :, :k], s.u[2, :, 0])
        else:
            out["accept_i"], out["next_i"] = sess.verify_intermediate()
        out["hidden_i"] = sess.last_hidden(B * (k + 1))
        if kind == "sample":
            f = sess.verify_full_rs(s.u[3, :, :sess.max_rows], s.u[2, :, 1])
        else:
            f = sess.verify_full()
        out["accept_f"], out["next_f"], out["committed"] = f[0], f[1], np.concatenate([np.asarray(x, np.int32) for x in f[2]])
        out["hidden_f"] = sess.last_hidden(s.full_rows)
        if c["logits"]:
            out["logits"] = sess.last_logits(s.full_rows)
    for b, n in enumerate(s.lens):
        sess.rollback(b, 0b111, n)
    return out


# ---- what a pass cannot do without ----------------------------------------------------------------------------------

def work(case):
    """Weights of every layer and head that a pass runs, once per sequential pass over them (a drafted row needs the row
    before it), the cached K and V once per layer pass, rows written; 2 flop per weight and row, 4 * head_dim per query head
    and visible position."""
    c = {**BASE, **case}
    d, hq, hkv, D, F, _, _ = WIDTHS[c["width"]]
    es = 2 if c["dtype"] == "bf16" else 4
    layer, head, L = (hq + 2 * hkv) * D * d + d * hq * D + 3 * F * d, c["vocab"] * d, c["layers"]
    aux = 2 * c["head_rank"] * d
    lens, B, k = _lens(c), c["batch"], c["k"]
    kv = 2 * hkv * D * es
    nbytes = flops = 0.0

    def layers(n, rows, seen):                 # rows per sequence, positions each sequence's rows see in all
        nonlocal nbytes, flops
        nbytes += n * (layer * es + sum(seen) * kv + sum(rows) * kv) + sum(rows) * d * 4
        flops += n * (2.0 * layer * sum(rows) + sum(4.0 * hq * D * r * s for r, s in zip(rows, seen)))

    def exit_(rows, early):
        nonlocal nbytes, flops
        w = head + (aux if early else 0)
        nbytes += w * es
        flops += 2.0 * w * rows

    one = [1] * B
    if c["kind"] == "prefill":
        nbytes += L * layer * es + sum(lens) * (L * kv + d * 4)
        flops += L * sum(2.0 * layer * n + 2.0 * hq * D * n * n for n in lens)
        exit_(B, False)
        layers(L, one, lens)
        exit_(B, False)
    elif c["kind"] == "decode":
        for _ in range(k):
            layers(L, one, lens)
            exit_(B, False)
    else:
        block, m = [k + 1] * B, [a + 1 for a in _accepts(c)]
        if c["kind"] == "verify":
            layers(c["exit_d"], block, lens)
        else:
            for j in range(k + 1):
                layers(c["exit_d"], one, lens)
                if j < k:
                    exit_(B, True)
        layers(c["exit_i"] - c["exit_d"], block, lens)
        exit_(B * (k + 1), True)
        if c["bonus_full"]:
            layers(c["exit_i"], one, lens)
        rows = [x + c["bonus_full"] for x in m]
        layers(L - c["exit_i"], rows, lens)
        exit_(sum(rows), False)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Largest relative difference (2-norm) that another correct implementation at the same precision shows.  With the
    attention's splits and the row-tiled projections' sums cut another way the bf16 outputs of the listed cases differ by
    0.004 to 0.0095 (largest single difference 0.04 of the root mean square), and both are 0.004 to 0.008 off the 64-bit
    values; the fp32 ones are 3e-7 off them."""
    if case.get("dtype") == "f32":
        return {"rel": 2e-6, "max": 2e-5}
    return {"rel": 0.025, "max": 0.15}


# ---- the same in 64 bits --------------------------------------------------------------------------------------------

_IDS = {"emb": 0, "gfinal": 2, "g1": 3, "wq": 4, "wk": 5, "wv": 6, "wo": 7, "g2": 8, "wgate": 9, "wup": 10, "wdown": 11,
        "aux_g": 12, "aux_a": 13, "aux_b": 14}


def _signed(x):
    x &= (1 << 64) - 1
    return x - (1 << 64) if x >> 63 else x


def _mix(z):
    """The generator's 64-bit mix on an int64 tensor (wrapping products, logical shifts) or on a Python integer."""
    if isinstance(z, int):
        z &= (1 << 64) - 1
        z = ((z ^ (z >> 30)) * 0xBF58476D1CE4E5B9) & ((1 << 64) - 1)
        z = ((z ^ (z >> 27)) * 0x94D049BB133111EB) & ((1 << 64) - 1)
        return z ^ (z >> 31)
    z = (z ^ ((z >> 30) & ((1 << 34) - 1))) * _signed(0xBF58476D1CE4E5B9)
    z = (z ^ ((z >> 27) & ((1 << 37) - 1))) * _signed(0x94D049BB133111EB)
    return z ^ ((z >> 31) & ((1 << 33) - 1))


def _weights(cfg, seed, name, layer, rows, cols):
    """The tensor of this name as include/hispec.h and its generator define it, in 64 bits on the GPU."""
    gold = 0x9E3779B97F4A7C15
    key = _mix(_mix(seed) ^ ((_IDS[name] << 32) | layer))
    damp = cfg.gamma[0] if name in ("wo", "wdown", "aux_b") else 1.0
    scale = float(np.float32(np.float32(cfg.sigma) * np.float32(damp)) * np.float32(2.0 ** -16))
    out = torch.empty(rows * cols, dtype=torch.float64, device="cuda")
    step = 1 << 24
    for e0 in range(0, rows * cols, step):
        e = torch.arange(e0, min(rows * cols, e0 + step), dtype=torch.int64, device="cuda")
        base = (3 * e + 1) * _signed(gold) + _signed(key)
        s = torch.zeros_like(e)
        for j in range(3):
            w = _mix(base + _signed(j * gold))
            s += (w & 0xFFFF) + ((w >> 16) & 0xFFFF) + ((w >> 32) & 0xFFFF) + ((w >> 48) & 0xFFFF)
        v = (s - 393210).to(torch.float32) * scale
        if name in ("gfinal", "g1", "g2", "aux_g"):
            v = 1.0 + v
        if cfg.dtype == "bf16":
            v = v.to(torch.bfloat16)
        out[e0:e0 + len(e)] = v.to(torch.float64)
    return out.view(rows, cols) if cols > 1 else out


def _norm(x, g):
    return x * torch.rsqrt((x * x).mean(-1, keepdim=True) + float(np.float32(1e-5))) * g


def _rope(x, pos, theta):
    """x [rows, heads, D], half-split pairs."""
    h = x.shape[-1] // 2
    ang = pos.to(torch.float64)[:, None] * (float(np.float32(theta)) ** (-torch.arange(h, dtype=torch.float64, device="cuda") / h))
    c, s = ang.cos()[:, None], ang.sin()[:, None]
    return torch.cat([x[..., :h] * c - x[..., h:] * s, x[..., h:] * c + x[..., :h] * s], -1)


def _attend(q, k, v, q_pos):
    """q [n, Hq, D] at positions q_pos over keys [m, Hkv, D] at 0..m-1, causal."""
    n, hq, D = q.shape
    m, hkv, _ = k.shape
    out = torch.empty_like(q)
    kt, vt = k.permute(1, 2, 0).contiguous(), v.permute(1, 0, 2).contiguous()
    for i in range(0, n, 512):
        qi = q[i:i + 512]
        r, top = len(qi), int(q_pos[i:i + 512].max()) + 1
        a = qi.view(r, hkv, hq // hkv, D).permute(1, 2, 0, 3).reshape(hkv, -1, D)
        s = torch.matmul(a, kt[:, :, :top]).view(hkv, hq // hkv, r, top) / math.sqrt(D)
        s.masked_fill_(torch.arange(top, device="cuda")[None, :] > q_pos[i:i + r, None], -math.inf)
        o = torch.matmul(torch.softmax(s, -1).view(hkv, -1, top), vt[:, :top])
        out[i:i + r] = o.view(hkv, hq // hkv, r, D).permute(2, 0, 1, 3).reshape(r, hq, D)
    return out


def _forward(cfg, seed, ctxs, tails):
    """Hidden rows behind every layer of the wanted tails: ctxs[b] tokens first, then each tail (b, tokens, layer) on its
    own behind its context; returns the tail's hidden rows behind `layer`."""
    d, hq, hkv, D, F = cfg.d_model, cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim, cfg.d_ffn
    emb = _weights(cfg, seed, "emb", 0, cfg.vocab, d)
    parts = [(b, list(t)) for b, t in enumerate(ctxs)] + [(b, list(t)) for b, t, _ in tails]
    starts = [0] * len(ctxs) + [len(ctxs[b]) for b, _, _ in tails]
    x = emb[torch.tensor([t for _, p in parts for t in p], device="cuda")]
    at = np.cumsum([0] + [len(p) for _, p in parts])
    pos = torch.cat([torch.arange(s, s + len(p), device="cuda") for s, (_, p) in zip(starts, parts)])
    nc, got = len(ctxs), [None] * len(tails)
    for l in range(cfg.n_layers):
        w = lambda name, r, c: _weights(cfg, seed, name, l, r, c)  # noqa: E731
        n = _norm(x, w("g1", d, 1))
        q = _rope((n @ w("wq", hq * D, d).T).view(-1, hq, D), pos, cfg.rope_theta)
        k = _rope((n @ w("wk", hkv * D, d).T).view(-1, hkv, D), pos, cfg.rope_theta)
        v = (n @ w("wv", hkv * D, d).T).view(-1, hkv, D)
        lo = 0
        if l + 1 == cfg.n_layers:              # only the tails are wanted behind the last layer
            lo = int(at[nc])
        o = torch.empty_like(q[lo:])
        for i, (b, p) in enumerate(parts):
            a, e = int(at[i]), int(at[i + 1])
            if a < lo:
                continue
            kk, vv = k[a:e], v[a:e]
            if i >= nc:
                c0, c1 = int(at[b]), int(at[b + 1])
                kk, vv = torch.cat([k[c0:c1], kk]), torch.cat([v[c0:c1], vv])
            o[a - lo:e - lo] = _attend(q[a:e], kk, vv, pos[a:e])
        del q, k, v, n
        full, x = x, x[lo:] + o.reshape(-1, hq * D) @ w("wo", d, hq * D).T
        n = _norm(x, w("g2", d, 1))
        wg, wu, wd = w("wgate", F, d), w("wup", F, d), w("wdown", d, F)
        for i in range(0, len(x), 4096):
            x[i:i + 4096] += (torch.nn.functional.silu(n[i:i + 4096] @ wg.T) * (n[i:i + 4096] @ wu.T)) @ wd.T
        del n, wg, wu, wd, o, full
        for j, (_, _, layer) in enumerate(tails):
            if layer == l + 1:
                got[j] = x[int(at[nc + j]) - lo:int(at[nc + j + 1]) - lo].clone()
    return got, emb


def exact(case, seed):
    c = {**BASE, **case}
    cfg = _config(c)
    prompts, blocks, _ = _inputs(c, seed)
    V, k, kind, L = c["vocab"], c["k"], c["kind"], c["layers"]
    chain = lambda t, n: [(t + j) % V for j in range(n)]  # noqa: E731
    firsts = [(int(p[-1]) + 1) % V for p in prompts]
    out = {}
    if kind in ("prefill", "decode"):
        tails = [(b, chain(f, k), L) for b, f in enumerate(firsts)]
        got, emb = _forward(cfg, seed, prompts, tails)
        last = torch.cat([g[-1:] for g in got])
        out["hidden"] = last
    else:
        tails = [(b, [f] + (blocks[b].tolist() if kind == "verify" else chain(f + 1, k)), c["exit_i"]) for b, f in enumerate(firsts)]
        tails += [(b, chain(f, a + 1 + c["bonus_full"]), L) for b, (f, a) in enumerate(zip(firsts, _accepts(c)))]
        got, emb = _forward(cfg, seed, prompts, tails)
        B = c["batch"]
        out["hidden_i"], last = torch.cat(got[:B]), torch.cat(got[B:])
        out["hidden_f"] = last
    if c["logits"]:
        lg = _norm(last, _weights(cfg, seed, "gfinal", 0, cfg.d_model, 1)) @ torch.roll(emb, 1, 0).T
        out["logits"] = torch.softmax(lg, -1) if kind == "sample" else lg
    return out
