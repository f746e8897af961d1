"""The work whose speed is measured: calls of the verification step as a serving or training program makes them.

Sizes are those of the benchmark's workloads (Llama-3-8B and Qwen3-8B shapes: 32 query heads over 8 KV heads of 128, hidden
size 4096, vocabularies of 128 256 and 151 936; the stress shape 48/8/128, 6144, 200 064; the tiny float32 chain) and, for the
drawn cases, odd and ragged sizes around them: batches from one request to a full server, contexts from a short prompt to
tens of thousands of tokens, chains and draft trees, greedy and sampled, 16-bit and 8-bit caches and LM heads.

Every input is made on the GPU from the seed alone.  A case's sequence lengths are spread evenly over its range (and dealt to
the requests by the seed), so that the work of a case does not depend on the seed.
"""
import math
import random

import torch

import paper_2602_06932_amd as av

DEV = "cuda"


# ---------------------------------------------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------------------------------------------
def _attn(batch, nq, lo, hi, tree=False, kv8=False, hq=32, hkv=8, d=128, page=16, dtype="bf16"):
    return {"batch": batch, "nq": nq, "hq": hq, "hkv": hkv, "d": d, "page": page, "len_lo": lo, "len_hi": hi, "dtype": dtype,
            "kv8": kv8, "tree": tree}


def _head(batch, nq, hidden=4096, vocab=128256, head="bf16"):
    return {"batch": batch, "nq": nq, "hidden": hidden, "vocab": vocab, "head": head}


def _sample(temperature=1.0, mixed=False, draft_vocab=0):
    return {"temperature": temperature, "mixed": mixed, "draft_vocab": draft_vocab}


def listed():
    return [
        # the smallest call: the tiny float32 chain, one whole step (what a first program or a unit test of a server runs)
        {"name": "verify_tiny_f32", "kind": "verify", **_attn(4, 5, 256, 256, hq=8, hkv=2, d=64, page=256, dtype="f32"),
         **_head(4, 5, 256, 1024, "f32"), **_sample()},
        # the step a server of a Llama-3-8B-shaped target runs all day: 32 requests, lookahead 4, sampled at T = 1
        {"name": "verify_chain_b32", "kind": "verify", **_attn(32, 5, 1024, 4096), **_head(32, 5), **_sample()},
        # one user: the attention of a single request in the middle of a conversation
        {"name": "attn_one_request", "kind": "attn", **_attn(1, 5, 2777, 2777)},
        # a full server with ragged contexts and lookahead 6 (the Qwen3-8B-shaped greedy workload)
        {"name": "attn_chain_b64", "kind": "attn", **_attn(64, 7, 512, 8192)},
        # draft trees: 32 nodes per request under their ancestor mask
        {"name": "attn_tree_b16", "kind": "attn", **_attn(16, 32, 4096, 4096, tree=True)},
        # the headline batch on an 8-bit KV cache
        {"name": "attn_chain_b32_kv8", "kind": "attn", **_attn(32, 5, 1024, 4096, kv8=True)},
        # one user: the vocabulary sweep for five token rows
        {"name": "lmhead_one_request", "kind": "lmhead", **_head(1, 5)},
        # the largest call: the vocabulary sweep of the stress batch, 1280 token rows
        {"name": "lmhead_b256", "kind": "lmhead", **_head(256, 5, 6144, 200064)},
        # the 8-bit LM head under draft trees, 512 token rows
        {"name": "lmhead_tree_b16_fp8", "kind": "lmhead", **_head(16, 32, head="fp8")},
        # what follows the vocabulary sweep on the serving side: the sampled tree walk and the trace records of the step
        {"name": "accept_trace_tree_b16", "kind": "accept", **_head(16, 32), "tree": True, **_sample(), "top_k": 1024},
        # the training side: forward and backward of the tree attention
        {"name": "train_attn_tree_b16", "kind": "train", **_attn(16, 32, 4096, 4096, tree=True)},
        # the training side: loss and gradient of 4096 trace rows over a 32K-entry draft vocabulary
        {"name": "draft_loss_4096", "kind": "loss", "rows": 4096, "draft_vocab": 32000, "top_k": 1024, "discard_top_k": 64},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_chunk(rng):
    """Query positions of a drawn case: a chain of 1 to 10 drafts or a tree of 8 to 48 nodes."""
    tree = rng.random() < 0.4
    return (rng.randint(8, 48) if tree else rng.randint(2, 11)), tree


def _draw_attn(rng, most_tokens, kv8=None):
    nq, tree = _draw_chunk(rng)
    batch = _log_int(rng, 1, 128)
    hi = min(_log_int(rng, 200, 20000), max(200, most_tokens // batch))
    lo = rng.choice([hi, max(nq, hi // 2), max(nq, hi // 8)])
    hq, hkv = rng.choice([(32, 8), (32, 8), (48, 8), (40, 8), (16, 8), (28, 4)])
    return _attn(batch, nq, lo, hi, tree=tree, hq=hq, hkv=hkv, page=rng.choice([16, 16, 32, 64]),
                 kv8=rng.random() < 0.3 if kv8 is None else kv8)


def _draw_head(rng, nq=None, most_rows=1024):
    nq = _draw_chunk(rng)[0] if nq is None else nq
    batch = max(1, min(_log_int(rng, 1, 192), most_rows // nq))
    hidden, vocab = rng.choice([(4096, 128256), (4096, 151936), (3584, 152064), (2048, 128256), (5120, 151936), (4096, 32003)])
    return _head(batch, nq, hidden, vocab, rng.choice(["bf16", "bf16", "fp8"]))


def _draw_sample(rng, vocab):
    return _sample(rng.choice([0.0, 0.6, 1.0, 1.0]), rng.random() < 0.2, 32000 if rng.random() < 0.25 and vocab > 64000 else 0)


def draw(rng):
    kind = rng.choice(["verify", "verify_f32", "attn", "attn", "attn", "lmhead", "lmhead", "lmhead", "accept", "train", "loss"])
    if kind == "attn":
        return {"kind": kind, **_draw_attn(rng, 400000)}
    if kind == "lmhead":
        return {"kind": kind, **_draw_head(rng)}
    if kind == "train":
        a = _draw_attn(rng, 80000, kv8=False)
        a["nq"] = min(a["nq"], 128 // (a["hq"] // a["hkv"]))  # a training tree of at most 32 nodes of four heads
        return {"kind": kind, **a}
    if kind == "loss":
        k = rng.choice([64, 256, 1000, 1024])
        return {"kind": kind, "rows": _log_int(rng, 100, 5000), "draft_vocab": rng.choice([32000, 32000, 24576, 16001, 32768]),
                "top_k": k, "discard_top_k": rng.choice([0, 32, 64])}
    if kind == "accept":
        nq, tree = _draw_chunk(rng)
        h = _draw_head(rng, nq, 600)
        return {"kind": kind, **h, "tree": tree, **_draw_sample(rng, h["vocab"]), "top_k": rng.choice([256, 1000, 1024])}
    if kind == "verify_f32":
        batch, nq = rng.randint(1, 8), rng.randint(2, 8)
        hi = _log_int(rng, 64, 1024)
        return {"kind": "verify", **_attn(batch, nq, max(nq, hi // 2), hi, hq=8, hkv=2, d=64, page=256, dtype="f32"),
                **_head(batch, nq, rng.choice([256, 512]), rng.choice([1024, 2003, 4096]), "f32"), **_sample()}
    a = _draw_attn(rng, 160000)
    h = _draw_head(rng, a["nq"], 600)
    a["batch"] = h["batch"] = min(a["batch"], h["batch"])
    return {"kind": "verify", **a, **h, **_draw_sample(rng, h["vocab"])}


# ---------------------------------------------------------------------------------------------------------------
# inputs, from the seed alone
# ---------------------------------------------------------------------------------------------------------------
def _seq_lens(c, rnd):
    n, lo, hi = c["batch"], c["len_lo"], c["len_hi"]
    lens = [lo + (hi - lo) * i // max(1, n - 1) for i in range(n)] if n > 1 else [(lo + hi) // 2]
    rnd.shuffle(lens)
    return [max(c["nq"], x) for x in lens]


def _tree_parents(rnd, batch, nodes, max_children=4, max_depth=6):
    out = []
    for _ in range(batch):
        par, depth, kids = [-1], [0], [0]
        for n in range(1, nodes):
            m = rnd.choice([i for i in range(n) if depth[i] < max_depth and kids[i] < max_children])
            par.append(m)
            depth.append(depth[m] + 1)
            kids.append(0)
            kids[m] += 1
        out.append(par)
    return out


def _normal(shape, dtype, g, std=1.0):
    """N(0, std^2) in float32, rounded once to `dtype`, in pieces that keep the temporary small."""
    out = torch.empty(shape, dtype=dtype, device=DEV)
    flat, step = out.view(-1), 1 << 26
    for o in range(0, flat.numel(), step):
        n = min(step, flat.numel() - o)
        flat[o:o + n] = torch.randn(n, device=DEV, generator=g) * std
    return out


def _to_e4m3(x, dims):
    """E4M3 codes of a float tensor and one float32 scale for all but `dims`."""
    scale = x.abs().amax(dim=dims, keepdim=True).float() / 448.0
    return (x.float() / scale).to(torch.float8_e4m3fn).view(torch.uint8), scale.reshape(-1).contiguous()


def _codes(x):
    return x.view(torch.float8_e4m3fn)


def _attn_inputs(c, rnd, g):
    lens = _seq_lens(c, rnd)
    dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    per = [-(-x // c["page"]) for x in lens]
    used, width = sum(per), max(per)
    pool = used + used // 10
    ids = torch.randperm(pool, device=DEV, generator=g)[:used].to(torch.int32).tolist()
    table, o = [], 0
    for n in per:
        table.append(ids[o:o + n] + [-1] * (width - n))
        o += n
    shape = (pool, c["hkv"], c["page"], c["d"])
    s = {"lens": lens, "pool": pool, "q": _normal((c["batch"], c["nq"], c["hq"], c["d"]), dt, g),
         "k": _normal(shape, dt, g), "v": _normal(shape, dt, g),
         "table": torch.tensor(table, dtype=torch.int32, device=DEV), "seq": torch.tensor(lens, dtype=torch.int32, device=DEV),
         "k_scale": None, "v_scale": None}
    if c["kv8"]:
        # heads of different magnitudes, as a per-head scale is there for
        gain = (2.0 ** (torch.arange(c["hkv"], device=DEV) % 3 - 1)).view(1, -1, 1, 1)
        for n in ("k", "v"):
            s[n], s[n + "_scale"] = _to_e4m3(s[n] * gain.to(dt), (0, 2, 3))
    return s


def _head_inputs(c, g):
    rows, fp8 = c["batch"] * c["nq"], c["head"] == "fp8"
    dt = torch.float32 if c["head"] == "f32" else torch.bfloat16
    s = {"hidden": _normal((rows, c["hidden"]), dt, g), "w": _normal((c["vocab"], c["hidden"]), dt, g, 0.02),
         "hidden_scale": None, "w_scale": None}
    if fp8:
        for n in ("hidden", "w"):
            s[n], s[n + "_scale"] = _to_e4m3(s[n], (1,))
    return s


def _sample_inputs(c, s, rnd, g):
    """Draft tokens and probabilities of a drafter that agrees with the target up to noise, and the uniforms."""
    B, nq, V = c["batch"], c["nq"], c["vocab"]
    par = s["parents_list"] or [list(range(-1, nq - 1))] * B
    par_t = torch.tensor(par, device=DEV)
    deq = lambda n: s[n] if c["head"] != "fp8" else (_codes(s[n]).to(torch.bfloat16) * s[n + "_scale"][:, None].to(torch.bfloat16))
    z = torch.matmul(deq("hidden"), deq("w").T).float().view(B, nq, V)  # what the drafter imitates: no more than an input
    tokens = torch.zeros((B, nq), dtype=torch.int32, device=DEV)
    s.update(temps=None, probs=None, uniforms=None, t2d=None)
    at = torch.arange(B, device=DEV)
    if c["temperature"] == 0.0 and not c["mixed"]:
        top = z.argmax(-1)
        for n in range(1, nq):
            hit = torch.rand(B, device=DEV, generator=g) < 0.7
            rand = torch.randint(0, V, (B,), device=DEV, generator=g)
            tokens[:, n] = torch.where(hit, top[at, par_t[:, n]], rand).to(torch.int32)
        s["tokens"] = tokens
        return
    T = torch.full((B,), c["temperature"] or 1.0, device=DEV)
    if c["mixed"]:  # a batch of requests with their own settings, greedy ones among them
        s["temps"] = torch.tensor([[0.0, 0.6, 1.0, 0.8][i % 4] for i in range(B)], device=DEV)
        T = torch.where(s["temps"] > 0, s["temps"], 1.0)
    d2t = None
    if c["draft_vocab"]:
        d2t = torch.randperm(V, device=DEV, generator=g)[:c["draft_vocab"]].sort().values
        s["t2d"] = torch.full((V,), -1, dtype=torch.int32, device=DEV)
        s["t2d"][d2t] = torch.arange(len(d2t), dtype=torch.int32, device=DEV)
        z = z[..., d2t].contiguous()
    z += torch.randn(z.shape, device=DEV, generator=g)
    z /= T.view(B, 1, 1)
    s["probs"] = torch.softmax(z, -1)
    for n in range(1, nq):
        pick = torch.multinomial(s["probs"][at, par_t[:, n]], 1, generator=g)[:, 0]
        tokens[:, n] = (d2t[pick] if d2t is not None else pick).to(torch.int32)
    s["tokens"] = tokens
    s["uniforms"] = torch.randint(0, 1 << 24, (B, nq, 2), device=DEV, generator=g).float() * 2.0 ** -24


def _loss_inputs(c, g):
    rows, vd, k = c["rows"], c["draft_vocab"], c["top_k"]
    ids = torch.empty((rows, k), dtype=torch.int32, device=DEV)
    for o in range(0, rows, 512):  # distinct tokens of every row
        ids[o:o + 512] = torch.rand((min(512, rows - o), vd), device=DEV, generator=g).topk(k, dim=1).indices.to(torch.int32)
    kept = (torch.randn((rows, k), device=DEV, generator=g) * 2).sort(dim=1, descending=True).values.to(torch.bfloat16)
    z = torch.randn((rows, vd), device=DEV, generator=g) - 3.0
    z.scatter_(1, ids.long(), kept.float() + torch.randn((rows, k), device=DEV, generator=g))
    u = torch.rand(rows, device=DEV, generator=g)
    traj = torch.where(u < 0.45, 1, torch.where(u < 0.8, 2, 0)).to(torch.int8)
    return {"z": z, "ids": ids, "kept": kept, "traj": traj}


def _inputs(c, seed):
    """Every input of a case; nothing of the package is called here."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    rnd = random.Random(seed)
    s = {"parents": None, "parents_list": None}
    if c["kind"] == "loss":
        return {**s, **_loss_inputs(c, g)}
    if c.get("tree"):
        s["parents_list"] = _tree_parents(rnd, c["batch"], c["nq"])
        s["parents"] = torch.tensor(s["parents_list"], dtype=torch.int32, device=DEV)
    if c["kind"] in ("attn", "train", "verify"):
        s.update(_attn_inputs(c, rnd, g))
    if c["kind"] in ("lmhead", "accept", "verify"):
        s.update(_head_inputs(c, g))
    if c["kind"] in ("accept", "verify"):
        _sample_inputs(c, s, rnd, g)
    if c["kind"] == "train":
        s["dout"] = _normal(s["q"].shape, s["q"].dtype, g)
    return s


# ---------------------------------------------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------------------------------------------
def _ptr(t):
    return None if t is None else t.data_ptr()


def _empty(shape, dtype=torch.float32):
    return torch.empty(shape, dtype=dtype, device=DEV)


def prepare(case, seed):
    c = case
    s = _inputs(c, seed)
    s["case"] = c
    if c["kind"] == "loss":
        s["desc"] = av.aurora_loss_desc(rows=c["rows"], draft_vocab=c["draft_vocab"], top_k=c["top_k"],
                                        discard_top_k=c["discard_top_k"], lambda_discard=0.5)
        s["row_kl"], s["loss"], s["grad"] = _empty(c["rows"]), _empty(5), _empty((c["rows"], c["draft_vocab"]))
        s["kept_bits"] = s["kept"].view(torch.int16)
        return s
    B, nq = c["batch"], c["nq"]
    s["ad"] = s["cd"] = None
    if "hq" in c:
        s["ad"] = av.aurora_attn_desc(batch=B, num_q=nq, num_q_heads=c["hq"], num_kv_heads=c["hkv"], head_dim=c["d"],
                                      page_size=c["page"], max_pages_per_seq=s["table"].shape[1], num_pages=s["pool"],
                                      dtype=av.AURORA_BF16 if c["dtype"] == "bf16" else av.AURORA_F32, sm_scale=0.0,
                                      kv_fp8=int(c["kv8"]), k_scale=_ptr(s["k_scale"]), v_scale=_ptr(s["v_scale"]))
        s["out"] = torch.empty_like(s["q"])
    if "vocab" in c:
        dt = {"bf16": av.AURORA_BF16, "f32": av.AURORA_F32, "fp8": av.AURORA_FP8_E4M3}[c["head"]]
        s["cd"] = av.aurora_accept_desc(batch=B, num_q=nq, hidden=c["hidden"], vocab=c["vocab"], dtype=dt,
                                        temperature=c.get("temperature", 1.0), draft_vocab=c.get("draft_vocab", 0) if s.get("t2d") is not None else 0,
                                        target_to_draft=_ptr(s.get("t2d")), hidden_scale=_ptr(s["hidden_scale"]),
                                        lm_head_scale=_ptr(s["w_scale"]), temperatures=_ptr(s.get("temps")))
    ws = av.aurora_verify_workspace_bytes(s["ad"], s["cd"])
    if c["kind"] == "train":
        ws = max(ws, av.aurora_attn_backward_workspace_bytes(s["ad"]))
        s["lse"], s["dq"] = _empty(s["q"].shape[:3]), _empty(s["q"].shape)
        s["dk"], s["dv"] = (torch.zeros(s["k"].shape, device=DEV) for _ in range(2))
    s["ws"] = _empty(ws, torch.uint8)
    if s["cd"] is not None:
        off = av.aurora_verify_logits_ptr(s["ad"], s["cd"], s["ws"]) - s["ws"].data_ptr()
        s["logits"] = s["ws"][off:off + 4 * B * nq * c["vocab"]].view(torch.float32).view(B * nq, c["vocab"])
    if c["kind"] in ("accept", "verify"):
        s["accept_len"], s["next_token"] = _empty(B, torch.int32), _empty(B, torch.int32)
        s["mask"] = _empty((B, nq), torch.uint8)
        s["p_at_draft"], s["row_lse"] = _empty((B, nq)), _empty((B, nq))
    if c["kind"] == "accept":
        av.aurora_verify_lmhead(s["cd"], s["hidden"], s["w"], s["ws"])  # the logits that the walk and the records work on
        gptr, n_groups = av.aurora_verify_group_max_ptr(None, s["cd"], s["ws"])
        s["td"] = av.aurora_trace_desc(batch=B, num_q=nq, vocab=c["vocab"], top_k=c["top_k"], n_groups=n_groups,
                                       group_max=gptr or None)
        s["topk_ids"], s["topk_logits"] = _empty((B * nq, c["top_k"]), torch.int32), _empty((B * nq, c["top_k"]), torch.int16)
        s["y_out"], s["traj"] = _empty((B, nq), torch.int32), _empty((B, nq), torch.int8)
    return s


def run(s):
    kind = s["case"]["kind"]
    if kind == "loss":
        av.aurora_draft_loss(s["desc"], s["z"], s["ids"], s["kept_bits"], s["traj"], s["row_kl"], s["loss"], s["grad"])
        return {n: s[n] for n in ("row_kl", "loss", "grad")}
    if kind == "attn":
        av.aurora_verify_attn(s["ad"], s["q"], s["k"], s["v"], s["table"], s["seq"], s["parents"], s["out"], s["ws"])
        return {"out": s["out"]}
    if kind == "lmhead":
        av.aurora_verify_lmhead(s["cd"], s["hidden"], s["w"], s["ws"])
        return {"logits": s["logits"]}
    if kind == "train":
        av.aurora_attn_forward(s["ad"], s["q"], s["k"], s["v"], s["table"], s["seq"], s["parents"], s["out"], s["lse"], s["ws"])
        av.aurora_attn_backward_saved(s["ad"], s["q"], s["k"], s["v"], s["table"], s["seq"], s["parents"], s["out"], s["lse"],
                                      s["dout"], s["dq"], s["dk"], s["dv"], s["ws"])
        return {n: s[n] for n in ("out", "lse", "dq", "dk", "dv")}
    outs = (s["accept_len"], s["next_token"], s["mask"], s["p_at_draft"], s["row_lse"], s["ws"])
    got = {n: s[n] for n in ("accept_len", "next_token", "mask", "p_at_draft", "row_lse")}
    if kind == "accept":
        av.aurora_verify_accept_logits(s["cd"], s["tokens"], s["probs"], s["uniforms"], s["parents"], *outs)
        av.aurora_trace_emit(s["td"], s["logits"], s["tokens"], s["parents"], s["next_token"], s["mask"], s["topk_ids"],
                             s["topk_logits"], s["y_out"], s["traj"])
        return {**got, "topk_ids": s["topk_ids"], "topk_logits": s["topk_logits"].view(torch.bfloat16), "y_out": s["y_out"],
                "traj": s["traj"]}
    av.aurora_verify(s["ad"], s["cd"], s["q"], s["k"], s["v"], s["table"], s["seq"], s["parents"], s["out"], s["hidden"], s["w"],
                     s["tokens"], s["probs"], s["uniforms"], *outs)
    return {**got, "attn": s["out"], "logits": s["logits"]}


# ---------------------------------------------------------------------------------------------------------------
# the work of one pass, the tolerances, and the results in 64 bits
# ---------------------------------------------------------------------------------------------------------------
def work(case):
    c = case
    if c["kind"] == "loss":
        n = c["rows"] * c["draft_vocab"]
        return {"bytes": 8 * n + 6 * c["rows"] * c["top_k"] + 5 * c["rows"], "flops": 8 * n}
    b = f = 0
    rows = c["batch"] * c["nq"]
    if "hq" in c:
        tokens = sum(_seq_lens(c, random.Random(0)))
        e = 4 if c["dtype"] == "f32" else 2
        kv, qo = tokens * c["hkv"] * c["d"], rows * c["hq"] * c["d"]
        b += 2 * kv * (1 if c["kv8"] else e) + 2 * qo * e
        f += 4 * tokens * c["nq"] * c["hq"] * c["d"]
        if c["kind"] == "train":  # K, V and q are needed by both passes, but once is enough to read them in principle
            b += 2 * kv * 4 + qo * (e + 4)
            f += 10 * tokens * c["nq"] * c["hq"] * c["d"]
    if c["kind"] in ("lmhead", "verify"):
        e = {"f32": 4, "bf16": 2, "fp8": 1}[c["head"]]
        b += (c["vocab"] + rows) * c["hidden"] * e + 4 * rows * c["vocab"]
        f += 2 * rows * c["vocab"] * c["hidden"]
    if c["kind"] in ("accept", "verify"):
        # the walk reads the row it stops at: its logits, and the draft distribution where it samples
        sampled = c["temperature"] > 0 or c["mixed"]
        row = (c["draft_vocab"] or c["vocab"]) + (c["vocab"] if c["kind"] == "accept" else 0)
        b += (c["batch"] * 4 * row if sampled else 0) + 32 * rows
        f += 4 * c["batch"] * c["vocab"]
    if c["kind"] == "accept":
        b += 4 * rows * c["vocab"] + 6 * rows * c["top_k"]
        f += rows * c["vocab"]
    return {"bytes": b, "flops": f}


def tolerance(case):
    """About four times the error that the path shows against 64 bits at these sizes (in brackets), which is what another
    order of its sums may differ by."""
    c = case
    if c["kind"] == "loss":  # float32 exponentials, sums in 64 bits (4e-7)
        return {"rel": 2e-6, "max": 1e-3}
    if c["kind"] == "lmhead":  # exact products, float32 sums over the hidden dimension (5e-7; 1.5e-5 in the 8-bit instruction)
        return {"rel": 6e-5, "max": 1e-3} if c["head"] == "fp8" else {"rel": 2e-6, "max": 1e-4}
    if c["kind"] == "accept":  # tokens and ids are whole values; the kept logits are bfloat16, where a rounding may tip
        return {"rel": 1e-4, "max": 1e-2, "differ": 0.005}
    if c.get("dtype") == "f32":  # (3e-7)
        return {"rel": 2e-6, "max": 1e-4, "differ": 0.005}
    # bfloat16 outputs and probabilities: attention and its gradients (2.3e-3)
    return {"rel": 9e-3, "max": 0.2, "differ": 0.005}


def _gather(c, s, name, b):
    """K or V of request b as float64 [Hkv, L, D]."""
    L = s["lens"][b]
    ids = s["table"][b, :-(-L // c["page"])].long()
    x = s[name][ids]
    x = _codes(x).double() if c["kv8"] else x.double()
    if c["kv8"]:
        x = x * s[name + "_scale"].double().view(1, -1, 1, 1)
    return x.permute(1, 0, 2, 3).reshape(c["hkv"], -1, c["d"])[:, :L].contiguous()


def _seen(c, s, b):
    """[nq, L] truth values: the prefix, the node itself and its ancestors."""
    nq, L = c["nq"], s["lens"][b]
    own = [[False] * nq for _ in range(nq)]
    for n in range(nq):
        a = n
        while a >= 0:
            own[n][a] = True
            a = s["parents_list"][b][a] if s["parents_list"] else a - 1
    return torch.cat([torch.ones((nq, L - nq), dtype=torch.bool, device=DEV), torch.tensor(own, device=DEV)], 1)


def _exact_attn(c, s):
    B, nq, hq, hkv, d = c["batch"], c["nq"], c["hq"], c["hkv"], c["d"]
    G, scale, train = hq // hkv, 1.0 / math.sqrt(d), c["kind"] == "train"
    r = {"out": _empty((B, nq, hq, d), torch.float64)}
    if train:
        r.update(lse=_empty((B, nq, hq), torch.float64), dq=_empty((B, nq, hq, d), torch.float64),
                 dk=torch.zeros(s["k"].shape, dtype=torch.float64, device=DEV), dv=torch.zeros(s["v"].shape, dtype=torch.float64, device=DEV))
    rows = lambda x, b: x[b].double().view(nq, hkv, G, d).permute(1, 0, 2, 3).reshape(hkv, nq * G, d).contiguous()
    back = lambda x: x.view(hkv, nq, G, -1).permute(1, 0, 2, 3).reshape(nq, hq, -1)
    for b in range(B):
        K, V, q = _gather(c, s, "k", b), _gather(c, s, "v", b), rows(s["q"], b)
        seen = _seen(c, s, b).repeat_interleave(G, 0)
        z = torch.bmm(q, K.transpose(1, 2).contiguous()) * scale
        z.masked_fill_(~seen, -math.inf)
        lse = torch.logsumexp(z, -1, keepdim=True)
        p = torch.exp(z - lse)
        o = torch.bmm(p, V)
        r["out"][b] = back(o)
        if train:
            do = rows(s["dout"], b)
            ds = p * (torch.bmm(do, V.transpose(1, 2).contiguous()) - (do * o).sum(-1, keepdim=True)) * scale
            r["lse"][b] = back(lse)[..., 0]
            r["dq"][b] = back(torch.bmm(ds, K))
            L, page = s["lens"][b], c["page"]
            pos = torch.arange(L, device=DEV)
            pid, off = s["table"][b].long()[pos // page], pos % page
            r["dk"][pid, :, off] = torch.bmm(ds.transpose(1, 2).contiguous(), q).permute(1, 0, 2)
            r["dv"][pid, :, off] = torch.bmm(p.transpose(1, 2).contiguous(), do).permute(1, 0, 2)
    return r


def _exact_logits(c, s):
    h, w, V = s["hidden"], s["w"], c["vocab"]
    out = _empty((h.shape[0], V), torch.float64)
    deq = lambda x, sc: x.double() if sc is None else _codes(x).double() * sc.double()[:, None]
    hd = deq(h, s["hidden_scale"])
    for o in range(0, V, 16384):
        out[:, o:o + 16384] = hd @ deq(w[o:o + 16384], None if s["w_scale"] is None else s["w_scale"][o:o + 16384]).T
    return out


def _exact_rows(c, s, logits):
    """p_at_draft and row_lse in 64 bits; greedy requests have 1 / 0 at the draft, which is a decision and left out."""
    B, nq = c["batch"], c["nq"]
    T = torch.full((B,), c["temperature"] or 1.0, dtype=torch.float64, device=DEV)
    if s["temps"] is not None:
        T = torch.where(s["temps"] > 0, s["temps"], 1.0).double()
    lse = _empty(B * nq, torch.float64)
    for m in range(B * nq):
        lse[m] = torch.logsumexp(logits[m] / T[m // nq], 0)
    lse = lse.view(B, nq)
    if c["temperature"] == 0.0 or c["mixed"]:
        return lse, None
    par = torch.tensor(s["parents_list"] or [list(range(-1, nq - 1))] * B, device=DEV).clamp(min=0)
    at = torch.arange(B, device=DEV)[:, None]
    z = logits.view(B, nq, -1)[at, par, s["tokens"].long()] / T[:, None]
    p = torch.exp(z - lse[at, par])
    p[:, 0] = 0.0
    return lse, p


def _exact_loss(c, s):
    rows, k = c["rows"], c["top_k"]
    traj = s["traj"].long()
    lim = torch.where(traj == 2, c["discard_top_k"] or k, k)
    zt = s["kept"].double().masked_fill(torch.arange(k, device=DEV)[None] >= lim[:, None], -math.inf)
    n_acc, n_dis = int((traj == 1).sum()), int((traj == 2).sum())
    wt = torch.where(traj == 1, 1.0 / max(1, n_acc), torch.where(traj == 2, 0.5 / max(1, n_dis), 0.0)).double()
    row_kl, grad = _empty(rows, torch.float64), _empty(s["z"].shape, torch.float64)
    for o in range(0, rows, 512):
        e = slice(o, min(rows, o + 512))
        lp = torch.log_softmax(s["z"][e].double(), -1)
        lt = torch.log_softmax(zt[e], -1)
        pt, ids = torch.exp(lt), s["ids"][e].long()
        row_kl[e] = torch.where(pt > 0, pt * (lt - lp.gather(1, ids)), 0.0).sum(1)
        grad[e] = torch.exp(lp).scatter_add_(1, ids, -pt) * wt[e, None]
    acc = row_kl[traj == 1].sum() / max(1, n_acc)
    dis = row_kl[traj == 2].sum() / max(1, n_dis)
    return {"row_kl": row_kl, "loss": torch.stack([acc + 0.5 * dis, acc, dis, acc * 0 + n_acc, acc * 0 + n_dis]), "grad": grad}


def exact(case, seed):
    c = case
    s = _inputs(c, seed)
    if c["kind"] == "loss":
        return _exact_loss(c, s)
    if c["kind"] in ("attn", "train"):
        return _exact_attn(c, s)
    logits = _exact_logits(c, s)
    if c["kind"] == "lmhead":
        return {"logits": logits}
    lse, p = _exact_rows(c, s, logits)
    r = {"accept_len": None, "next_token": None, "mask": None, "p_at_draft": p, "row_lse": lse}
    if c["kind"] == "accept":
        top = logits.topk(c["top_k"], dim=1).values
        return {**r, "topk_ids": None, "topk_logits": top, "y_out": None, "traj": None}
    return {**r, "attn": _exact_attn(c, s)["out"], "logits": logits}
