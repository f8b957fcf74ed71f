"""The work a user of this framework has it do, as timed cases with a 64-bit reference.

A case is one request (or one batch of requests) through the public binding: ``reset``, ``prefill`` of the prompts, a run
of decode steps with given input tokens, ``logits``; or one whole-sequence scoring call (``masked_forward``); or a run of
decode steps that continues a context which ``prepare`` has already filled (long contexts, where the prompt is paid for
once and many tokens follow).  The input tokens of the decode steps are given (teacher forcing), so that the logits of two
correct implementations stay comparable; the steps, the kernels and the token selection are those of free-running
decoding.  Two cases are whole models (the 0.6B- and 4B-shaped configurations of the benchmark); the others are models of
a few layers with the same layer shapes, where rounding has less depth to travel through.

Weights are N(0, 0.02), norm gains 1 + 0.2 N(0, 1), prompts uniform over the vocabulary.
"""
import math

import numpy as np
import torch

import paper_2510_11958_amd as pkg

EPS, THETA = 1e-6, 1e6

# layer shapes: hidden, query heads, KV heads, head dim, SwiGLU width
_TINY = dict(hidden=256, q_heads=4, kv_heads=2, head_dim=64, ffn=768)
_W1024 = dict(hidden=1024, q_heads=16, kv_heads=8, head_dim=128, ffn=3072)
_W2560 = dict(hidden=2560, q_heads=32, kv_heads=8, head_dim=128, ffn=9728)
_VOCAB = 151936


def _case(name, shape, layers, **kw):
    c = dict(kind="request", dtype="bf16", vocab=_VOCAB, batch=1, prompt=64, ragged=False, steps=0, tau=1, n_late=1,
             n_early=0, api="decode", temperature=0.0, top_k=0, layers=layers, **shape)
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest model and the smallest calls there are: a tiny fp32 model, a short prompt, a few tokens
        _case("tiny fp32 request", _TINY, 4, dtype="fp32", vocab=1024, prompt=32, steps=16, tau=2, n_late=1),
        # a small model serving one user: every launch is a few microseconds long
        _case("0.6B request", _W1024, 28, prompt=256, steps=64, tau=2, n_late=4),
        # the benchmark's own configuration: one user, 1024-token prompt, cycles of three tokens
        _case("4B request", _W2560, 36, prompt=1024, steps=63, tau=3, n_late=8),
        # one user's prompt through the layers, odd length (time to first token)
        _case("prompt of 1003", _W2560, 4, prompt=1003),
        # one long document as a prompt: attention over the growing context weighs in
        _case("prompt of 8192", _W2560, 2, prompt=8192),
        # prefill of a large batch at the batched configuration's prompt length
        _case("prompts 32 x 2048", _W2560, 2, batch=32, prompt=2048),
        # ordinary decoding (tau = 1), one user: what the method is compared with
        _case("tau 1, one user", _W2560, 8, prompt=130, steps=48, tau=1, n_late=8),
        # a batch of the speed-test grid whose tokens are drawn (temperature, top-k) instead of taken greedily
        _case("batch of 8, sampled", _W2560, 8, batch=8, prompt=40, steps=48, tau=3, n_late=4, temperature=0.8, top_k=50),
        # the batched configuration: 32 sequences, cycles of four tokens (128 rows in the front layers of a full step)
        _case("batch of 32", _W2560, 6, batch=32, prompt=64, steps=48, tau=4, n_late=2),
        # prompts of different lengths in one batch, one cycle length per sequence
        _case("ragged, cycles per sequence", _W2560, 6, batch=5, prompt=301, ragged=True, steps=24, tau=4, n_late=2, api="per_seq"),
        # long contexts: tokens for 8 sequences that already hold 16k tokens each
        _case("8 x 16k context", _W2560, 4, kind="continue", batch=8, prompt=16384, steps=24, tau=3, n_late=2),
        # teacher-forced scoring of whole sequences (per-position cross entropy)
        _case("scoring 3 x 701", _W2560, 4, kind="score", batch=3, prompt=701, tau=3, n_late=2),
    ]


def _cost(c):
    """Rough time of a pass in seconds, for keeping drawn cases within the listed ones."""
    w = work(c)
    if c["dtype"] == "fp32":      # the tiny model: cache resident, a few rows per pass over its weights
        return c["layers"] * (c["batch"] * c["prompt"] + 2 * c["batch"] * c["steps"]) * 1e-5 + w["bytes"] / 1e12
    return w["bytes"] / 2.5e12 + w["flops"] / 1.0e14 + c["steps"] * c["layers"] * 4e-5


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    shape = rng.choice([
        _TINY, _W1024, _W2560, _W2560, _W2560,
        dict(hidden=2048, q_heads=16, kv_heads=8, head_dim=128, ffn=6144),
        dict(hidden=1536, q_heads=12, kv_heads=2, head_dim=128, ffn=8960),
        dict(hidden=896, q_heads=14, kv_heads=2, head_dim=64, ffn=4864),
    ])
    limit = max(_cost(c) for c in listed())
    while True:
        kind = rng.choice(["prompt", "decode", "decode", "decode", "batch", "score", "continue"])
        layers = rng.randint(2, 8)
        c = _case("", shape, layers, vocab=rng.choice([_VOCAB, _log(rng, 1000, _VOCAB)]))
        c["n_late"] = rng.randint(1, layers)
        c["tau"] = rng.randint(1, 6)
        c["prompt"] = _log(rng, 8, 3000)
        if kind == "prompt":
            c.update(batch=_log(rng, 1, 40), ragged=rng.random() < 0.3)
        elif kind == "score":
            c.update(kind="score", batch=_log(rng, 1, 8), prompt=_log(rng, 20, 1200))
        elif kind == "continue":
            c.update(kind="continue", batch=_log(rng, 1, 12), prompt=_log(rng, 2000, 16384), steps=rng.randint(16, 32), tau=rng.randint(1, 4))
        else:
            c.update(batch=_log(rng, 2, 40) if kind == "batch" else 1, steps=rng.randint(16, 63), prompt=_log(rng, 8, 600))
            c["api"] = rng.choice(["decode", "decode", "cycle", "per_seq"] if c["batch"] > 1 else ["decode", "decode", "cycle", "noalloc"])
            c["ragged"] = c["batch"] > 1 and rng.random() < 0.3
            if rng.random() < 0.3:
                c.update(temperature=round(rng.uniform(0.5, 1.2), 2), top_k=rng.choice([0, 20, 50]))
            if c["api"] != "per_seq" and c["n_late"] < layers and rng.random() < 0.2:
                c["n_early"] = rng.randint(1, layers - c["n_late"])
        if shape is _TINY:
            c["dtype"] = "fp32"
            c["vocab"] = min(c["vocab"], 32000)
        if c["ragged"] and c["batch"] < 2:
            c["ragged"] = False
        # room in memory for several states, and no dearer than the listed cases
        kv = 2 * c["layers"] * c["batch"] * (c["prompt"] + 4096) * c["kv_heads"] * c["head_dim"] * (4 if c["dtype"] == "fp32" else 2)
        if _cost(c) <= 0.8 * limit and kv < 16e9:
            return c


# ------------------------------------------------------------------------------------------------ inputs

def _tensors(c):
    """(name, dims, is gain) of the weight blob, in the order the library documents."""
    d, hd, ff = c["hidden"], c["head_dim"], c["ffn"]
    qd, kd = c["q_heads"] * hd, c["kv_heads"] * hd
    out = [("embed", (c["vocab"], d), False)]
    for l in range(c["layers"]):
        out += [((l, "attn_norm"), (d,), True), ((l, "q"), (qd, d), False), ((l, "k"), (kd, d), False), ((l, "v"), (kd, d), False),
                ((l, "q_norm"), (hd,), True), ((l, "k_norm"), (hd,), True), ((l, "o"), (d, qd), False), ((l, "mlp_norm"), (d,), True),
                ((l, "gate"), (ff, d), False), ((l, "up"), (ff, d), False), ((l, "down"), (d, ff), False)]
    return out + [("final_norm", (d,), True)]


def _weights(c, seed):
    """The flat weight blob on the GPU, and views of its tensors by name."""
    specs = _tensors(c)
    blob = torch.empty(sum(math.prod(s) for _, s, _ in specs), dtype=torch.float32 if c["dtype"] == "fp32" else torch.bfloat16, device="cuda")
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    views, off = {}, 0
    for name, dims, gain in specs:
        t = blob[off:off + math.prod(dims)].view(dims)
        off += t.numel()
        t.normal_(1.0 if gain else 0.0, 0.2 if gain else 0.02, generator=g)
        views[name] = t
    return blob, views


def _tokens(c, seed):
    """Prompts [batch, prompt], their lengths, cycle lengths per sequence, and the decode steps' input tokens."""
    rng = np.random.RandomState(seed % (1 << 31))
    b, p = c["batch"], c["prompt"]
    prompts = rng.randint(0, c["vocab"], (b, p)).astype(np.int32)
    lengths = np.full(b, p, np.int32)
    if c["ragged"]:
        lengths = rng.randint(max(1, p // 3), p + 1, b).astype(np.int32)
        lengths[rng.randint(b)] = p
    taus = np.full(b, c["tau"], np.int32)
    if c["api"] == "per_seq":
        taus = rng.randint(1, c["tau"] + 1, b).astype(np.int32)
    forced = rng.randint(0, c["vocab"], (b, max(1, c["steps"]))).astype(np.int32)
    return prompts, lengths, taus, forced


_ROOM = 4096      # "continue": tokens a context can grow by before the state starts over


def _fill(s):
    c = s["case"]
    s["eng"].prefill(s["prompts"], lengths=s["lengths"] if c["ragged"] else None)
    s["at"] = c["prompt"]


def prepare(case, seed):
    c = dict(case)
    blob, _ = _weights(c, seed)
    prompts, lengths, taus, forced = _tokens(c, seed)
    room = _ROOM if c["kind"] == "continue" else c["steps"] + 8
    cfg = pkg.ModelConfig(c["layers"], c["hidden"], c["q_heads"], c["kv_heads"], c["head_dim"], c["ffn"], c["vocab"], dtype=c["dtype"],
                          rms_eps=EPS, rope_theta=THETA, max_batch=c["batch"], max_seq_len=c["prompt"] + room)
    eng = pkg.Engine(cfg, blob)
    if c["n_early"]:
        eng.set_n_early(c["n_early"])
    if c["temperature"] > 0:
        eng.set_sampling(c["temperature"], c["top_k"], seed)
    s = dict(case=c, eng=eng, prompts=prompts, lengths=lengths, taus=taus, forced=forced)
    if c["kind"] == "score":
        s["mask"] = _score_mask(c)
    if c["kind"] == "continue":
        _fill(s)
    if c["api"] == "noalloc":
        s["forced_dev"] = [torch.from_numpy(np.ascontiguousarray(forced[:, i:i + n])).cuda() for i, n in _cycles(c)]
        s["out_dev"] = torch.empty((c["batch"], c["tau"]), dtype=torch.int32, device="cuda")
    return s


def _cycles(c):
    """(first step, steps) of each decode_cycle call: the prefill's token is the first of cycle 1."""
    out, i, n = [], 0, c["tau"] - 1 if c["tau"] > 1 else 1
    while i < c["steps"]:
        n = min(n, c["steps"] - i)
        out.append((i, n))
        i, n = i + n, c["tau"]
    return out


def run(s):
    c, eng = s["case"], s["eng"]
    if c["kind"] == "score":
        r = eng.masked_forward(s["prompts"], s["mask"], c["n_late"])
        return {"nll": r["nll"], "loss": r["loss"]}
    if c["kind"] == "request" or s["at"] + c["steps"] > c["prompt"] + _ROOM:
        eng.reset()
        _fill(s)
    tau, n_late, forced, tokens = c["tau"], c["n_late"], s["forced"], None
    if c["steps"]:
        s["at"] += c["steps"]
        if c["api"] == "decode":
            tokens = eng.decode(tau, n_late, c["steps"], forced=forced)
        elif c["api"] == "per_seq":
            tokens = eng.decode_per_seq(s["taus"], n_late, c["steps"], forced=forced)
        elif c["api"] == "cycle":
            tokens = np.concatenate([eng.decode_cycle(tau, n_late, n, forced=forced[:, i:i + n]) for i, n in _cycles(c)], 1)
        else:
            for f, (i, n) in zip(s["forced_dev"], _cycles(c)):
                eng.decode_cycle_noalloc(tau, n_late, s["out_dev"], n, forced_dev=f)
    out = {"logits": eng.logits()}
    # in 16 bits a near-tie between the two largest of 150,000 logits may go either way: the logits are the output there
    if c["dtype"] == "fp32" and tokens is not None and c["temperature"] == 0:
        out["tokens"] = tokens
    return out


# ---------------------------------------------------------------------------------------- bytes, flops, limits

def _schedule(c, taus, b):
    """For each decode step of sequence b: True where its cycle starts (all layers), else the late layers only."""
    full, phase = [], 1
    for _ in range(c["steps"]):
        full.append(phase >= taus[b])
        phase = 1 if full[-1] else phase + 1
    return full


def work(case):
    """Weights once for the prompt pass and once per decode step (they exceed every cache), the table's rows once per step for
    the LM head, each sequence's live keys and values once per step, logits written once; two operations per weight and row."""
    c = case
    e = 4 if c["dtype"] == "fp32" else 2
    d, hd, ff, V, L = c["hidden"], c["head_dim"], c["ffn"], c["vocab"], c["layers"]
    qd, kd = c["q_heads"] * hd, c["kv_heads"] * hd
    wl = d * (qd + 2 * kd) + qd * d + 3 * d * ff
    B, P, nl, ne = c["batch"], c["prompt"], c["n_late"], c["n_early"]
    kv, bytes_, flops = 2 * kd * e, 0, 0
    if c["kind"] != "continue":
        rows = B * P
        bytes_ += L * (wl * e + rows * kv) + V * d * e
        flops += 2 * rows * L * wl + 4 * qd * L * B * P * (P + 1) // 2
        heads = rows if c["kind"] == "score" else B
        flops += 2 * heads * V * d
        bytes_ += rows * d * e + (rows * 4 if c["kind"] == "score" else 0)
    # the schedule of the largest cycle length; sequences with shorter cycles of their own add front passes
    pending = 0
    for i, full in enumerate(_schedule(c, [c["tau"]], 0)):
        ctx = P + i + 1
        layers = L if full else nl + ne
        rows = (L - nl - ne) * (pending + 1) + nl + ne if full else layers
        bytes_ += layers * (wl * e + B * ctx * kv) + V * d * e + B * V * 4
        flops += B * (2 * rows * wl + 4 * qd * rows * ctx + 2 * V * d)
        pending = 0 if full else pending + 1
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    # fp32: sums in another order, through a few layers (measured against exact: 2.5e-7 with 4 layers).  bf16: weights and KV
    # cache are bf16, everything between carries at least 16 mantissa bits, so two correct implementations differ where a key
    # or value rounds the other way (measured against exact: 3e-3 to 6e-3 up to 8 layers and in the 28-layer 1024-wide model,
    # 1.2e-2 in the 36-layer 2560-wide one; cross entropies, whose size comes from the vocabulary, 3e-4 to 4e-4).
    c = case
    if c["dtype"] == "fp32":
        return {"rel": 5e-6, "differ": 0.01}
    if c["kind"] == "score":
        return {"rel": 2e-3}
    return {"rel": 1e-2 if c["layers"] <= 28 else 3e-2}


# ------------------------------------------------------------------------------------------- 64-bit reference

def _norm(x, g):
    return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + EPS) * g


def _layer(c, w, l, h):
    """One transformer block over a whole sequence h [T, hidden], float64."""
    T, hd, nh, nk = h.shape[0], c["head_dim"], c["q_heads"], c["kv_heads"]
    W = {n: w[(l, n)].double() for n in ("attn_norm", "q", "k", "v", "q_norm", "k_norm", "o", "mlp_norm", "gate", "up", "down")}
    x = _norm(h, W["attn_norm"])
    q = _norm((x @ W["q"].t()).view(T, nh, hd), W["q_norm"])
    k = _norm((x @ W["k"].t()).view(T, nk, hd), W["k_norm"])
    v = (x @ W["v"].t()).view(T, nk, hd)
    ang = torch.arange(T, device=h.device, dtype=torch.float64)[:, None] * THETA ** (-torch.arange(0, hd, 2, device=h.device, dtype=torch.float64) / hd)
    cos, sin = ang.cos()[:, None], ang.sin()[:, None]

    def rope(t):
        a, b = t[..., :hd // 2], t[..., hd // 2:]
        return torch.cat([a * cos - b * sin, b * cos + a * sin], -1)

    q, k = rope(q).transpose(0, 1).contiguous(), rope(k).permute(1, 2, 0).contiguous()     # [heads, T, hd], [kv heads, hd, T]
    v = v.transpose(0, 1).contiguous()
    out = torch.empty((T, nh, hd), dtype=torch.float64, device=h.device)
    step = max(1, min(T, (1 << 27) // (T * (nh // nk))))
    for g in range(nk):
        for t0 in range(0, T, step):
            t1 = min(T, t0 + step)
            qq = q[g * (nh // nk):(g + 1) * (nh // nk), t0:t1].reshape(-1, hd)
            sc = ((qq @ k[g][:, :t1]) / math.sqrt(hd)).view(nh // nk, t1 - t0, t1)
            sc.masked_fill_(torch.arange(t1, device=h.device)[None, :] > torch.arange(t0, t1, device=h.device)[:, None], -math.inf)
            o = torch.softmax(sc, -1).view(-1, t1) @ v[g][:t1]
            out[t0:t1, g * (nh // nk):(g + 1) * (nh // nk)] = o.view(nh // nk, t1 - t0, hd).transpose(0, 1)
    h = h + out.view(T, nh * hd) @ W["o"].t()
    x = _norm(h, W["mlp_norm"])
    return h + (torch.nn.functional.silu(x @ W["gate"].t()) * (x @ W["up"].t())) @ W["down"].t()


def _forward(c, w, tokens, full):
    """The final norm's output [T, hidden] of the masked whole-sequence form: late layers read the front output at full
    positions, the embedding (with early layers: their output) elsewhere."""
    emb = w["embed"][torch.from_numpy(tokens.astype(np.int64)).cuda()].double()
    h, masked = emb, emb
    first_late = c["layers"] - c["n_late"]
    for l in range(c["layers"]):
        if l == c["n_early"] and l > 0:
            masked = h
        if l == first_late:
            if l > 0 and l == c["n_early"]:
                masked = h
            h = torch.where(torch.from_numpy(full).cuda()[:, None], h, masked)
        h = _layer(c, w, l, h)
    return _norm(h, w["final_norm"].double())


def _score_mask(c):
    """First half of the positions full, then every tau-th."""
    i, half = np.arange(c["prompt"]), c["prompt"] // 2
    return ((i < half) | ((i - half) % c["tau"] == 0)).astype(np.uint8)


def exact(case, seed):
    c = dict(case)
    _, w = _weights(c, seed)
    prompts, lengths, taus, forced = _tokens(c, seed)
    table = w["embed"]
    if c["kind"] == "score":
        mask = _score_mask(c).astype(bool)
        nll = np.zeros((c["batch"], c["prompt"]))
        for b in range(c["batch"]):
            h = _forward(c, w, prompts[b], mask)
            z = torch.cat([_head(h[t:t + 256], table) for t in range(0, c["prompt"], 256)])
            target = torch.from_numpy(prompts[b, 1:].astype(np.int64)).cuda()
            nll[b, :-1] = torch.nn.functional.cross_entropy(z[:-1], target, reduction="none").cpu().numpy()
        return {"nll": nll, "loss": nll[:, :-1].mean(1)}
    logits = np.empty((c["batch"], c["vocab"]))
    for b in range(c["batch"]):
        seq = np.concatenate([prompts[b, :lengths[b]], forced[b, :c["steps"]]])
        full = np.array([True] * int(lengths[b]) + _schedule(c, taus, b))
        logits[b] = _head(_forward(c, w, seq, full)[-1:], table)[0].cpu().numpy()
    return {"logits": logits, "tokens": None} if c["dtype"] == "fp32" and c["steps"] and c["temperature"] == 0 and c["api"] != "noalloc" else {"logits": logits}


def _head(h, table):
    return torch.cat([h @ table[v:v + 32768].double().t() for v in range(0, table.shape[0], 32768)], 1)
