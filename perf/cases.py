"""The work that a video-LLM serving program has this library do, as cases that can be timed and compared.

One request of such a program: the text-prompt queries score the visual tokens of the prefilled caches (once per
request, over one or several layers), the best-scored tokens' K/V rows are gathered into the draft cache, and then
decoding rounds follow -- verification attention over every layer's full cache beside draft attention over the
pruned ones, and the speculative-sampling verdict.  Caches may be contiguous, paged, or quantised to 8 bits.
The configurations are those of synth_inputs.py (832, 4K, 16K, 33K and 4 x 37K visual-token caches), ragged
ones around them come from `draw`.

Calls that happen once per request are made eagerly and let the library allocate what it returns; the decoding
rounds, whose kernels take a few microseconds each, are captured in a HIP graph with outputs and workspaces kept,
which is how such a loop is run.
"""
from __future__ import annotations

import math

import torch

import paper_2601_08273_amd as h

# (query heads, KV heads, head dim) of the configurations
HEADS = {"4/2x64": (4, 2, 64), "14/2x64": (14, 2, 64), "28/4x128": (28, 4, 128), "64/8x128": (64, 8, 128)}
TORCH_DTYPE = {"fp32": torch.float32, "bf16": torch.bfloat16}
ELEM_BYTES = {"fp32": 4, "bf16": 2, "fp8": 1}
CROP = 5              # the method's 5 x 5 crops
PAGE = 16             # tokens per page of the paged caches
VOCAB = 152064        # rows of the LM head of a 7B-class model


def _video(name, op, dtype, batch, heads, frames, grid_h, grid_w, prefix, suffix, **more):
    return dict(name=name, op=op, dtype=dtype, batch=batch, heads=heads, frames=frames, grid_h=grid_h, grid_w=grid_w,
                prefix=prefix, suffix=suffix, **more)


def listed():
    return [
        # the smallest call: one verification of a short fp32 cache, launched by itself (latency and launches)
        _video("verify_fp32_832", "round", "fp32", 1, "4/2x64", 4, 12, 16, 32, 32, gamma=4, layers=1, cache="plain",
               draft_pct=0, graph=False),
        # scoring an fp32 cache of short video on a 14 x 14 grid, whose crops are cut at the edges
        _video("score_fp32_3k", "score", "fp32", 1, "14/2x64", 16, 14, 14, 64, 64, layers=1, emb_dim=0),
        # scoring with a small model's cache: little work per launch
        _video("score_4k", "score", "bf16", 1, "14/2x64", 16, 16, 16, 64, 64, layers=1, emb_dim=0),
        # scoring one layer of a 7B-class cache, the ordinary request
        _video("score_16k", "score", "bf16", 1, "28/4x128", 64, 16, 16, 128, 128, layers=1, emb_dim=0),
        # scoring a long video with the attention mass summed over four layers
        _video("score_33k_4layers", "score", "bf16", 1, "28/4x128", 128, 16, 16, 256, 256, layers=4, emb_dim=0),
        # scoring a batch of a large model: the most arithmetic, embeddings of 1024 channels
        _video("score_4x37k", "score", "bf16", 4, "64/8x128", 64, 24, 24, 128, 128, layers=1, emb_dim=0),
        # top-k and construction of the draft cache of the ordinary request
        _video("select_16k", "select", "bf16", 1, "28/4x128", 64, 16, 16, 128, 128, keep_pct=10),
        # one decoding round of the ordinary request: 28 layers verified (their new rows appended by the call)
        # beside the draft model's decode over the pruned caches
        _video("round_16k", "round", "bf16", 1, "28/4x128", 64, 16, 16, 128, 128, gamma=5, layers=28, cache="append",
               draft_pct=10, graph=True),
        # the first verification of a long video: the 12 tokens that the draft model buffered during prefill,
        # over paged caches
        _video("verify_33k_paged", "round", "bf16", 1, "28/4x128", 128, 16, 16, 256, 256, gamma=12, layers=8,
               cache="paged", draft_pct=0, graph=True),
        # verification of a batch of a large model: the most bytes
        _video("verify_4x37k", "round", "bf16", 4, "64/8x128", 64, 24, 24, 128, 128, gamma=5, layers=4, cache="plain",
               draft_pct=0, graph=True),
        # the same batch kept in 8 bits: a layer's cache is quantised after prefill, then verified from its codes
        _video("fp8_4x37k", "fp8", "bf16", 4, "64/8x128", 64, 24, 24, 128, 128, gamma=5),
        # the verdict of a round by sampling, for a batch of four sequences
        dict(name="verdict_152k", op="verdict", dtype="bf16", batch=4, gamma=5, vocab=VOCAB, temperature=1.0),
    ]


# ---------------------------------------------------------------------------------------------------------------
# drawn cases
# ---------------------------------------------------------------------------------------------------------------

def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_once(rng):
    op = rng.choice(["score", "score", "score", "select", "round", "round", "round", "fp8", "verdict"])
    if op == "verdict":
        return dict(op=op, dtype=rng.choice(["bf16", "bf16", "fp32"]), batch=rng.choice([1, 1, 2, 4, 7]),
                    gamma=rng.randint(1, 12), vocab=_log_int(rng, 32000, VOCAB) // 8 * 8,
                    temperature=rng.choice([0.0, 0.7, 1.0]))
    dtype = "bf16" if op == "fp8" else rng.choice(["bf16", "bf16", "bf16", "fp32"])
    case = dict(op=op, dtype=dtype, batch=rng.choice([1, 1, 1, 2, 3, 4]), heads=rng.choice(sorted(HEADS)),
                frames=_log_int(rng, 4, 128), grid_h=rng.randint(11, 24), grid_w=rng.randint(11, 24),
                prefix=_log_int(rng, 8, 256), suffix=_log_int(rng, 16, 256))
    if op == "score":
        case.update(layers=rng.choice([1, 1, 2, 4]), emb_dim=rng.choice([0, 0, 0, 768]))
    elif op == "select":
        case.update(keep_pct=rng.choice([5, 10, 25]))
    elif op == "round":
        case.update(gamma=rng.randint(1, 12), layers=_log_int(rng, 1, 28), draft_pct=rng.choice([0, 5, 10, 25]),
                    cache=rng.choice(["plain", "append", "paged"]), graph=rng.choice([True, True, False]))
    else:
        case.update(gamma=rng.randint(1, 12))
    return case


def _cost(case):
    """A pass's rough time in seconds: its bytes, and its arithmetic at the rate of its type's unit."""
    w = work(case)
    return w["bytes"] / 5e12 + w["flops"] / (6e12 if case["dtype"] == "fp32" else 3.5e14)


def draw(rng):
    most, most_bytes = max(_cost(c) for c in listed()), max(work(c)["bytes"] for c in listed())
    while True:
        case = _draw_once(rng)
        if _cost(case) <= most and work(case)["bytes"] <= most_bytes:
            return case


# ---------------------------------------------------------------------------------------------------------------
# inputs: the recipe of synth_inputs.py, drawn on the GPU
# ---------------------------------------------------------------------------------------------------------------

def _shape(case):
    H, Hkv, d = HEADS[case["heads"]]
    n_vis = case["frames"] * case["grid_h"] * case["grid_w"]
    return H, Hkv, d, n_vis, case["prefix"] + n_vis + case["suffix"]


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _normal(g, *shape):
    return torch.randn(shape, generator=g, device="cuda")


def _uniform(g, lo, hi, *shape):
    return torch.rand(shape, generator=g, device="cuda") * (hi - lo) + lo


def _text_queries(case, g):
    H, Hkv, d, _, _ = _shape(case)
    shared = torch.nn.functional.normalize(_normal(g, case["batch"], 1, Hkv, 1, d), dim=-1)
    q = _normal(g, case["batch"], case["suffix"], Hkv, H // Hkv, d) + 0.6 * math.sqrt(d) * shared
    return q.reshape(case["batch"], case["suffix"], H, d), shared[:, 0, :, 0]


def _cache(case, g, bias, n_rows):
    """K and V [B, Hkv, n_rows, d]: normal text rows and V; visual keys a smooth field over every frame whose phase
    drifts from frame to frame, plus noise, plus a bias of the frame's outer ring along `bias` [B, Hkv, d]."""
    _, Hkv, d, n_vis, _ = _shape(case)
    B, F, gh, gw = case["batch"], case["frames"], case["grid_h"], case["grid_w"]
    tdt, inv = TORCH_DTYPE[case["dtype"]], 1.0 / math.sqrt(d)
    k = torch.empty((B, Hkv, n_rows, d), dtype=tdt, device="cuda")
    v = torch.empty_like(k)
    xs = (torch.arange(gw, device="cuda") / gw).view(1, 1, 1, gw, 1)
    ys = (torch.arange(gh, device="cuda") / gh).view(1, 1, gh, 1, 1)
    ring = torch.zeros((gh, gw), device="cuda")
    ring[0] = ring[-1] = 1.0
    ring[:, 0] = ring[:, -1] = 1.0
    for b in range(B):
        k[b] = _normal(g, Hkv, n_rows, d).mul_(inv)
        v[b] = _normal(g, Hkv, n_rows, d).mul_(inv)
        field = _normal(g, Hkv, F, gh, gw, d).mul_(0.3)
        for _ in range(4):
            a, u, w = (_uniform(g, lo, hi, Hkv, 1, 1, 1, d) for lo, hi in ((0.5, 1.0), (0.0, 2.0), (0.0, 2.0)))
            phi = _uniform(g, 0.0, 2 * math.pi, Hkv, 1, d) + _uniform(g, -0.5, 0.5, Hkv, F, d).cumsum(1)
            wave = (2 * math.pi * (u * xs + w * ys)) + phi.view(Hkv, F, 1, 1, d)
            field.add_(wave.sin_().mul_(a))
        field.mul_(inv).add_(ring.view(1, 1, gh, gw, 1) * (1.5 * bias[b]).view(Hkv, 1, 1, 1, d))
        k[b, :, case["prefix"]:case["prefix"] + n_vis] = field.view(Hkv, n_vis, d)
    return k, v


def _to_pages(x, table):
    """[B, Hkv, N, d] -> pool [pages, PAGE, Hkv, d] in which page i of sequence b is number table[b, i]"""
    B, Hkv, N, d = x.shape
    n = table.shape[1]
    rows = torch.zeros((B, n * PAGE, Hkv, d), dtype=x.dtype, device=x.device)
    rows[:, :N] = x.transpose(1, 2)
    pool = torch.empty((B * n, PAGE, Hkv, d), dtype=x.dtype, device=x.device)
    pool[table.view(-1).long()] = rows.view(B * n, PAGE, Hkv, d)
    return pool


def prepare(case, seed):
    g = _gen(seed)
    tdt = TORCH_DTYPE[case["dtype"]]
    s = dict(case=case)
    if case["op"] == "verdict":
        # an LM-head-like row (a few likely words above a long tail); the draft's is the target's plus noise
        B, gamma, V = case["batch"], case["gamma"], case["vocab"]
        p = _normal(g, B, gamma + 1, V).mul_(2.0)
        hot = torch.randint(0, V, (B, gamma + 1, 4), generator=g, device="cuda")
        p.scatter_(2, hot, p.max() + _uniform(g, 0.0, 4.0, B, gamma + 1, 4))
        q = p[:, :gamma] + 0.6 * _normal(g, B, gamma, V)
        likely = torch.softmax(q / max(case["temperature"], 0.1), -1).view(B * gamma, V)
        s["tokens"] = torch.multinomial(likely, 1, generator=g).view(B, gamma).to(torch.int32)
        s["p"], s["q"] = p.to(tdt), q.to(tdt)
        s["u_accept"], s["u_sample"] = _uniform(g, 0.0, 1.0, B, gamma), _uniform(g, 0.0, 1.0, B)
        return s

    H, Hkv, d, n_vis, n_ctx = _shape(case)
    B = case["batch"]
    s["vid"] = h.video_desc(case["frames"], case["grid_h"], case["grid_w"], case["prefix"], CROP, CROP)
    if case["op"] == "score":
        s["q_txt"], s["k"] = [], []
        for _ in range(case["layers"]):
            q, shared = _text_queries(case, g)
            s["q_txt"].append(q.to(tdt))
            s["k"].append(_cache(case, g, shared, n_ctx)[0])
        s["emb"] = None
        if case["emb_dim"]:      # the vision encoder's tokens: neighbours resemble each other
            e = _normal(g, B, case["frames"], case["grid_h"], case["grid_w"], case["emb_dim"])
            e = e + 1.5 * e.roll(1, 1) + 1.5 * e.roll(1, 2) + 1.5 * e.roll(1, 3)
            s["emb"] = e.view(B, n_vis, case["emb_dim"]).to(tdt)
        return s
    _, shared = _text_queries(case, g)
    if case["op"] == "select":   # fused scores: sums of three per-frame z-scores
        s["scores"] = _normal(g, B, n_vis, 3).sum(-1).contiguous()
        s["k"], s["v"] = _cache(case, g, shared, n_ctx)
        s["keep"] = (n_vis * case["keep_pct"] + 99) // 100
        return s

    q_len = case["gamma"] + 1
    n_tot = n_ctx + q_len
    if case["op"] == "fp8":
        s["k"], s["v"] = _cache(case, g, shared, n_tot)
        s["q"] = _normal(g, B, q_len, H, d).to(tdt)
        return s

    # decoding rounds: every layer's cache, queries and outputs; workspaces are shared along a stream
    paged = case["cache"] == "paged"
    s["layers"] = []
    for _ in range(case["layers"]):
        k, v = _cache(case, g, shared, n_tot)
        layer = dict(q=_normal(g, B, q_len, H, d).to(tdt))
        layer["out"] = torch.empty_like(layer["q"])
        if case["draft_pct"]:
            keep = (n_vis * case["draft_pct"] + 99) // 100
            kept = torch.rand((n_vis,), generator=g, device="cuda").topk(keep).indices.sort().values + case["prefix"]
            whole = torch.arange(n_ctx, device="cuda")
            rows = torch.cat([whole[:case["prefix"]], kept, whole[case["prefix"] + n_vis:], whole[-1:]])
            layer.update(kd=k[:, :, rows].contiguous(), vd=v[:, :, rows].contiguous(),
                         qd=_normal(g, B, 1, H, d).to(tdt))
            layer["out_d"] = torch.empty_like(layer["qd"])
        if case["cache"] == "append":
            layer.update(k_new=k[:, :, n_ctx:].transpose(1, 2).contiguous(),
                         v_new=v[:, :, n_ctx:].transpose(1, 2).contiguous())
        if paged:
            n_pages = (n_tot + PAGE - 1) // PAGE
            layer["table"] = torch.randperm(B * n_pages, generator=g, device="cuda").view(B, n_pages).to(torch.int32)
            k, v = _to_pages(k, layer["table"]), _to_pages(v, layer["table"])
        layer.update(k=k, v=v)
        s["layers"].append(layer)
    kv = h.kv_desc(torch.empty((B, Hkv, 1, d), dtype=tdt, device="cuda"), H)

    def workspace(call, rows, n):
        return torch.empty(h.workspace_bytes(call, kv, None, rows, n), dtype=torch.uint8, device="cuda")

    s["n_ctx"], s["ws"] = n_ctx, workspace(h.CALL_VERIFY_ATTENTION, q_len, n_tot)
    if case["draft_pct"]:
        s["n_dctx"] = s["layers"][0]["kd"].shape[2] - 1
        s["ws_d"] = workspace(h.CALL_DRAFT_ATTENTION, 1, s["n_dctx"] + 1)
        s["side"] = torch.cuda.Stream()
    if case["graph"]:
        _round(s)
        torch.cuda.synchronize()
        s["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(s["graph"]):
            _round(s)
    return s


# ---------------------------------------------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------------------------------------------

def _round(s):
    """Every layer's verification on the current stream, the draft model's decode beside it on another."""
    case, n = s["case"], s["n_ctx"]
    cur = torch.cuda.current_stream()
    if case["draft_pct"]:
        s["side"].wait_stream(cur)
    for t in s["layers"]:
        if case["cache"] == "paged":
            h.hippo_verify_attention_paged(t["q"], t["k"], t["v"], t["table"], n, out=t["out"], workspace=s["ws"])
        elif case["cache"] == "append":
            h.hippo_verify_attention(t["q"], t["k"], t["v"], n, out=t["out"], workspace=s["ws"], k_new=t["k_new"],
                                     v_new=t["v_new"])
        else:
            h.hippo_verify_attention(t["q"], t["k"], t["v"], n, out=t["out"], workspace=s["ws"])
        if case["draft_pct"]:
            h.hippo_draft_attention(t["qd"], t["kd"], t["vd"], s["n_dctx"], out=t["out_d"], workspace=s["ws_d"],
                                    stream=s["side"])
    if case["draft_pct"]:
        cur.wait_stream(s["side"])


def run(s):
    case = s["case"]
    if case["op"] == "score":
        if case["layers"] == 1:
            return h.hippo_score_tokens(s["q_txt"][0], s["k"][0], s["vid"], emb=s["emb"])
        return h.hippo_score_tokens_layers(s["q_txt"], s["k"], s["vid"], emb=s["emb"])
    if case["op"] == "select":
        return h.hippo_select_gather_kv(s["scores"], s["keep"], s["k"], s["v"], s["vid"], HEADS[case["heads"]][0])
    if case["op"] == "fp8":
        kc, vc, ks, vs = h.hippo_quantize_kv_e4m3(s["k"], s["v"])
        out = h.hippo_verify_attention_fp8kv(s["q"], kc, vc, ks, vs, s["k"].shape[2] - s["q"].shape[1])
        return [kc, vc, ks, vs, out]
    if case["op"] == "verdict":
        if case["temperature"] == 0.0:
            return h.hippo_spec_verify(s["p"], None, s["tokens"], None, None, 0.0, want_alpha=True)
        return h.hippo_spec_verify(s["p"], s["q"], s["tokens"], s["u_accept"], s["u_sample"], case["temperature"],
                                   want_alpha=True)
    if case["graph"]:
        s["graph"].replay()
    else:
        _round(s)
    return [t[o] for t in s["layers"] for o in ("out", "out_d") if o in t]


# ---------------------------------------------------------------------------------------------------------------
# what a pass cannot do without, and how far a correct result may be off
# ---------------------------------------------------------------------------------------------------------------

def work(case):
    B, es = case["batch"], ELEM_BYTES[case["dtype"]]
    if case["op"] == "verdict":
        greedy = case["temperature"] == 0.0
        rows = case["gamma"] + 1 + (0 if greedy else case["gamma"])
        return {"bytes": B * rows * case["vocab"] * es, "flops": 4 * B * rows * case["vocab"]}
    H, Hkv, d, n_vis, n_ctx = _shape(case)
    if case["op"] == "score":
        L, layers = case["suffix"], case["layers"]
        de = case["emb_dim"] or Hkv * d
        emb = B * n_vis * de
        keys = layers * B * Hkv * n_vis * d
        # one product of queries and keys per layer; per token its row of the crop's Gram matrix, and one
        # dot product with the next frame
        return {"bytes": es * (keys + layers * B * L * H * d + (emb if case["emb_dim"] else 0)) + 4 * B * n_vis,
                "flops": 2 * layers * B * L * H * n_vis * d + 2 * emb * (CROP * CROP + 1)}
    if case["op"] == "select":
        keep = (n_vis * case["keep_pct"] + 99) // 100
        rows = n_ctx - n_vis + keep
        return {"bytes": 4 * B * (n_vis + keep) + 2 * 2 * B * Hkv * rows * d * es, "flops": B * n_vis}
    q_len = case["gamma"] + 1
    entries = B * Hkv * (n_ctx + q_len) * d
    qo = 2 * B * q_len * H * d
    per_query = 4 * B * H * d
    if case["op"] == "fp8":
        return {"bytes": 2 * entries * (2 + 1) + 2 * qo,
                "flops": per_query * q_len * (n_ctx + q_len) + 4 * entries}
    out = {"bytes": es * (2 * entries + qo), "flops": per_query * q_len * (n_ctx + q_len)}
    if case["draft_pct"]:
        n = n_ctx - n_vis + (n_vis * case["draft_pct"] + 99) // 100 + 1
        out["bytes"] += es * (2 * B * Hkv * n * d + 2 * B * H * d)
        out["flops"] += per_query * n
    return {k: v * case["layers"] for k, v in out.items()}


def tolerance(case):
    """About four times the distance from the same path in 64 bits, at the worst of the listed and some hundred drawn
    cases: fused scores 3.3e-6 (1.6e-5 at an element; Eq. 7 divides by a frame's deviation), attention 3.8e-7 (1.4e-6)
    in fp32 and 3.0e-3 (1.5e-2) in bf16, where probabilities and outputs are rounded, acceptance ratios 1.8e-7
    (6.0e-7).  Selected indices, gathered rows, cache codes and verdicts are whole."""
    if case["op"] == "score":
        return {"rel": 1.5e-5, "max": 7e-5}
    if case["op"] == "select":
        return "exact"
    if case["op"] == "verdict":
        return {"rel": 8e-7, "max": 2.4e-6, "differ": 0.0}
    if case["dtype"] == "fp32":
        return {"rel": 1.5e-6, "max": 6e-6}
    return {"rel": 1e-2, "max": 6e-2, "differ": 0.0}


# ---------------------------------------------------------------------------------------------------------------
# the same results in 64 bits, by plain torch
# ---------------------------------------------------------------------------------------------------------------

def _z_scores(x):
    """x [F, P]: every frame's tokens centred and divided by their population deviation (0 where that is 0)."""
    c = x - x.mean(1, keepdim=True)
    sigma = c.square().mean(1, keepdim=True).sqrt()
    return torch.where(sigma > 0, c / torch.where(sigma > 0, sigma, torch.ones_like(sigma)), torch.zeros_like(c))


def _exact_scores(case, s):
    H, Hkv, d, n_vis, _ = _shape(case)
    B, F, gh, gw, P0, G = case["batch"], case["frames"], case["grid_h"], case["grid_w"], case["prefix"], H // Hkv
    out = torch.empty((B, n_vis), dtype=torch.float64, device="cuda")
    for b in range(B):
        attn = torch.zeros(n_vis, dtype=torch.float64, device="cuda")
        for q, k in zip(s["q_txt"], s["k"]):
            for hk in range(Hkv):
                keys = k[b, hk, P0:P0 + n_vis].double().t().contiguous()
                for hq in range(hk * G, hk * G + G):
                    attn += torch.softmax(q[b, :, hq].double() @ keys / math.sqrt(d), -1).sum(0)
        emb = s["emb"][b].double() if s["emb"] is not None else \
            s["k"][0][b, :, P0:P0 + n_vis].double().transpose(0, 1).reshape(n_vis, Hkv * d)
        norm = emb.norm(dim=1, keepdim=True)
        unit = (emb / torch.where(norm > 0, norm, torch.ones_like(norm))).view(F, gh, gw, -1)
        near, count = torch.zeros((F, gh, gw), dtype=torch.float64, device="cuda"), torch.zeros(F, device="cuda")
        if F > 1:
            cos = (unit[1:] * unit[:-1]).sum(-1)
            near[1:] += cos
            near[:-1] += cos
            count[1:] += 1
            count[:-1] += 1
        temp = 1.0 - near / count.clamp(min=1).view(F, 1, 1)
        spa = torch.empty((F, gh, gw), dtype=torch.float64, device="cuda")
        for y in range(0, gh, CROP):
            for x in range(0, gw, CROP):
                crop = unit[:, y:y + CROP, x:x + CROP]
                rows = crop.reshape(F, -1, crop.shape[-1])
                cos = torch.bmm(rows, rows.transpose(1, 2).contiguous())
                spa[:, y:y + CROP, x:x + CROP] = cos.var(-1, unbiased=False).view(crop.shape[:3])
        out[b] = sum(_z_scores(t.reshape(F, gh * gw)) for t in (attn / (H * case["suffix"]), temp, spa)).view(-1)
    return out


def _exact_attention(q, k, v, n_ctx):
    """q [B, q_len, H, d] over k, v [B, Hkv, n_ctx + q_len, d]; row i sees the first n_ctx + 1 + i rows."""
    B, q_len, H, d = q.shape
    Hkv, n = k.shape[1], k.shape[2]
    hidden = torch.arange(n, device="cuda") > n_ctx + torch.arange(q_len, device="cuda").view(1, q_len, 1)
    out = torch.empty(q.shape, dtype=torch.float64, device="cuda")
    for b in range(B):
        for hk in range(Hkv):
            heads = slice(hk * (H // Hkv), (hk + 1) * (H // Hkv))
            rows = q[b, :, heads].double().transpose(0, 1)
            z = (rows.reshape(-1, d) @ k[b, hk].double().t().contiguous()).view(-1, q_len, n) / math.sqrt(d)
            p = torch.softmax(z.masked_fill(hidden, -math.inf), -1)
            out[b, :, heads] = (p.view(-1, n) @ v[b, hk].double()).view(-1, q_len, d).transpose(0, 1)
    return out


def _e4m3(x):
    """A cache [B, Hkv, N, d] -> (its values once coded in 8 bits, in 64 bits, and the heads' multipliers)."""
    mult = (x.abs().amax((2, 3)).float() / 448).view(*x.shape[:2], 1, 1)
    mult = torch.where(mult > 0, mult, torch.ones_like(mult))
    codes = (x.float() / mult).to(torch.float8_e4m3fn)
    return codes.double() * mult.double(), mult.view(x.shape[:2]).double()


def _from_pages(pool, table, n):
    B, d = table.shape[0], pool.shape[-1]
    rows = pool[table.view(-1).long()].view(B, -1, pool.shape[2], d)
    return rows[:, :n].transpose(1, 2)


def exact(case, seed):
    s = prepare(dict(case, graph=False), seed)
    if case["op"] == "select":
        return None
    if case["op"] == "verdict":
        alpha = None
        if case["temperature"] > 0.0:
            at = s["tokens"].long().unsqueeze(-1)
            log_p, log_q = (torch.log_softmax(x.double() / case["temperature"], -1).gather(2, at).squeeze(-1)
                            for x in (s["p"][:, :case["gamma"]], s["q"]))
            alpha = torch.exp(log_p - log_q).clamp(max=1.0)
        return None, None, alpha
    if case["op"] == "score":
        return _exact_scores(case, s)
    if case["op"] == "fp8":
        (k, ks), (v, vs) = _e4m3(s["k"]), _e4m3(s["v"])
        return [None, None, ks, vs, _exact_attention(s["q"], k, v, k.shape[2] - s["q"].shape[1])]
    out = []
    for t in s["layers"]:
        k, v = t["k"], t["v"]
        if case["cache"] == "paged":
            k, v = (_from_pages(x, t["table"], s["n_ctx"] + t["q"].shape[1]) for x in (k, v))
        out.append(_exact_attention(t["q"], k, v, s["n_ctx"]))
        if "qd" in t:
            out.append(_exact_attention(t["qd"], t["kd"], t["vd"], s["n_dctx"]))
    return out
