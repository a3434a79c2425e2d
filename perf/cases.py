"""The work a serving program has this library do, as cases that can be timed and compared.

Five kinds, each through the entry points of `paper_2509_09754_amd.lava`:

  layer    prefill end of one layer of one sequence: scores (which prepare the selection and form the
           layer's budget), layer-wide top-B, packed K/V.  Every buffer is one the program keeps.
  batch    the same for a ragged batch of sequences, one call per step for the whole batch
  stack    all layers of one sequence at once: plain scores, budgets shared among the layers, one table
           of selections and one of compactions into one pool
  cascade  the layer-by-layer driver: a step per arriving layer, which evicts earlier layers again
  decode   one new token per sequence over the packed caches (and the rows appended since)

Inputs are drawn on the device from the seed: standard normal queries and keys with a sink key and a
few keys turned towards a window query, values with log-normal row norms.  The head counts, window
sizes and budgets are those of the benchmark's configurations and of the tests; lengths run from one
thousand to 131072 tokens.
"""
import math

import torch

from paper_2509_09754_amd import lava

DEV = "cuda"
SINK = 4.0
KINDS = {"lava": lava.LAVA_SCORE_LAVA, "attention": lava.LAVA_SCORE_ATTENTION, "token_norm": lava.LAVA_SCORE_TOKEN_NORM}


def _heads(hq, hkv, d, w, dtype):
    return dict(hq=hq, hkv=hkv, d=d, w=w, dtype=dtype)


GQA4 = _heads(32, 8, 128, 32, "bf16")     # the benchmark's layer: 32 query heads on 8 KV heads
GQA7 = _heads(28, 4, 128, 32, "bf16")     # a group that is not a power of two and is swept in two parts
TINY = _heads(8, 2, 64, 8, "f32")         # the smallest configuration
FULL = _heads(32, 8, 128, 32, "f32")      # the same layer kept in 32 bits


def _layer(name, heads, n, budget, lse=False, score="lava", heavy=0.01):
    return dict(name=name, kind="layer", n=n, budget=budget, lse=lse, score=score, heavy=heavy, **heads)


def listed():
    return [
        # a short prompt on the smallest configuration: latency and launches
        _layer("layer_1k_f32_d64", TINY, 1024, 256),
        # an ordinary chat prompt, ragged length, 64 entries per head kept
        _layer("layer_4k", GQA4, 4115, 8 * 64),
        # a long document; budget 512 per head
        _layer("layer_32k", GQA4, 32768, 8 * 512),
        # the longest context the benchmark quotes; budget 1024 per head
        _layer("layer_131k", GQA4, 131072, 8 * 1024),
        # the prefill attention kept its log-sum-exp, so no statistics pass; odd length
        _layer("layer_100k_lse", GQA4, 100003, 8 * 1024, lse=True),
        # 28 query heads on 4 KV heads, odd length
        _layer("layer_21k_g7", GQA7, 21013, 4 * 512),
        # 32-bit cache with the per-token value-norm score, odd length
        _layer("layer_9k_f32_token_norm", FULL, 9001, 8 * 128, score="token_norm"),
        # a serving batch: 16 sequences of 4096 to 65536 tokens, 4096 entries each
        dict(name="batch16_ragged", kind="batch", batch=16, lo=4096, hi=65536, mix=1, budget=4096, **GQA4),
        # a 32-layer model, 32K tokens a layer, one budget of 131072 entries shared among the layers
        dict(name="stack32_32k", kind="stack", layers=32, n=32768, total=131072, **GQA4),
        # eight layers arriving one after the other, each step evicting the earlier ones again
        dict(name="cascade8_32k", kind="cascade", layers=8, n=32768, total=8 * 4096, mix=3, **GQA4),
        # a single user's next token: one compressed layer and a few appended rows
        dict(name="decode1", kind="decode", batch=1, rows=8192, tail=37, **GQA4),
        # next token of 64 users
        dict(name="decode64", kind="decode", batch=64, rows=8192, tail=0, **GQA4),
    ]


def _log_int(rng, lo, hi):
    """An integer of [lo, hi], spread over its logarithm."""
    return min(hi, max(lo, round(math.exp(rng.uniform(math.log(lo), math.log(hi))))))


def draw(rng):
    kind = rng.choice(["layer", "layer", "layer", "batch", "stack", "cascade", "decode", "decode"])
    if kind == "layer":
        heads = rng.choice([GQA4, GQA4, GQA4, GQA7, TINY, FULL])
        n = _log_int(rng, 1000, 32768 if heads in (TINY, FULL) else 131072)
        per_head = min(_log_int(rng, 64, 1024), n // 4)
        return dict(kind="layer", n=n, budget=heads["hkv"] * max(per_head, heads["w"]), lse=rng.random() < 0.25,
                    score=rng.choice(["lava", "lava", "lava", "lava", "attention", "token_norm"]),
                    heavy=round(rng.uniform(0.002, 0.03), 4), **heads)
    if kind == "batch":
        lo = _log_int(rng, 1000, 8192)
        return dict(kind="batch", batch=rng.randint(2, 16), lo=lo, hi=_log_int(rng, lo, 65536), mix=rng.randrange(1 << 20),
                    budget=8 * rng.randint(32, 512 if lo >= 2048 else 200), **GQA4)
    if kind == "stack":
        layers = rng.choice([8, 16, 28, 32])
        n = _log_int(rng, 1000, 32768)
        return dict(kind="stack", layers=layers, n=n, total=layers * 8 * min(_log_int(rng, 64, 512), n // 4), **GQA4)
    if kind == "cascade":
        n = _log_int(rng, 4096, 65536)
        layers = rng.randint(4, 12)
        return dict(kind="cascade", layers=layers, n=n, total=layers * 8 * min(rng.randint(64, 512), n // (2 * layers)),
                    mix=rng.randrange(1 << 20), **GQA4)
    return dict(kind="decode", batch=_log_int(rng, 1, 64), rows=_log_int(rng, 512, 8192), tail=rng.choice([0, 1, 130]),
                **rng.choice([GQA4, GQA4, GQA7]))


# ------------------------------------------------------------------------------------------- inputs
def _lengths(c):
    """The batch's sequence lengths, uniform in [lo, hi]: a property of the case, so that its work is known."""
    x, out = c["mix"] * 2654435761 + 12345, []
    for _ in range(c["batch"]):
        x = (x * 6364136223846793005 + 1442695040888963407) % (1 << 64)
        out.append(c["lo"] + (x >> 33) % (c["hi"] - c["lo"] + 1))
    return out


def _dtype(c):
    return torch.bfloat16 if c["dtype"] == "bf16" else torch.float32


def _generator(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _towards(k, q, rows, heads, gen):
    """k[rows] keep their norms and get cosine 0.8 to the queries q[...] of `heads`."""
    qhat = torch.nn.functional.normalize(q[heads], dim=-1)
    u = torch.randn(qhat.shape, generator=gen, device=DEV)
    u = torch.nn.functional.normalize(u - (u * qhat).sum(-1, keepdim=True) * qhat, dim=-1)
    k[rows] = k[rows].norm(dim=-1, keepdim=True) * (0.8 * qhat + 0.6 * u)


def _draw_layer(c, n, heavy, gen):
    """q [H, w, d], k and v [H_kv, n, d] of one layer, rounded once to the storage type."""
    hq, hkv, d, w, dt = c["hq"], c["hkv"], c["d"], c["w"], _dtype(c)
    q = torch.randn(hq, w, d, generator=gen, device=DEV)
    k = torch.randn(hkv, n, d, generator=gen, device=DEV)
    k[:, 0] *= SINK
    count = max(1, int(heavy * hkv * (n - w)))
    flat = torch.randint(0, hkv * (n - w - 1), (count,), generator=gen, device=DEV).unique()
    g, i = flat // (n - w - 1), 1 + flat % (n - w - 1)
    head = g * (hq // hkv) + torch.randint(0, hq // hkv, g.shape, generator=gen, device=DEV)
    row = torch.randint(0, w, g.shape, generator=gen, device=DEV)
    _towards(k.view(hkv * n, d), q.view(hq * w, d), g * n + i, head * w + row, gen)
    q, k = q.to(dt), k.to(dt)
    v = torch.randn(hkv, n, d, generator=gen, device=DEV)
    v *= torch.exp(0.5 * torch.randn(hkv, n, 1, generator=gen, device=DEV))
    return q, k, v.to(dt)


def _logits(c, q, k, g, wide):
    """Scaled logits of KV head g's query rows, [G, w, n], with the keys a row may not see at -inf."""
    G, w, d, n = c["hq"] // c["hkv"], c["w"], c["d"], k.shape[1]
    x = q[g * G: (g + 1) * G].to(wide).reshape(G * w, d) @ k[g].to(wide).t().contiguous()
    x = x.view(G, w, n) / math.sqrt(d)
    r = torch.arange(w, device=DEV).view(1, w, 1)
    j = torch.arange(w, device=DEV).view(1, 1, w)
    x[:, :, n - w:].masked_fill_(j > r, -math.inf)
    return x


def _lse(c, q, k):
    """What the prefill attention keeps: the window rows' log-sum-exp, [H, w]."""
    return torch.cat([_logits(c, q, k, g, torch.float32).logsumexp(-1) for g in range(c["hkv"])])


def _desc(c):
    return lava.LayerDesc.make(c["hq"], c["hkv"], c["d"], c["w"], c["dtype"], score_kind=KINDS[c.get("score", "lava")])


def _i64(x):
    return torch.tensor(x, dtype=torch.int64, device=DEV)


def _bytes(n):
    return torch.empty(max(int(n), 256), dtype=torch.uint8, device=DEV)


def _prepare_layer(c, seed):
    q, k, v = _draw_layer(c, c["n"], c["heavy"], _generator(seed))
    hkv, n, B, desc = c["hkv"], c["n"], c["budget"], _desc(c)
    s = dict(c=c, desc=desc, q=q, k=k, v=v, lse=_lse(c, q, k) if c["lse"] else None)
    s.update(scores=torch.empty(hkv * n, device=DEV), vbar=torch.empty(1, hkv, device=DEV), stat=torch.empty(1, device=DEV),
             ws=_bytes(lava.lava_window_scores_workspace_bytes(desc, 1, n)), ws_sel=_bytes(lava.lava_select_workspace_bytes(hkv * n)),
             e=torch.zeros(1, 1, device=DEV), total=_i64([B]), lo=_i64([[hkv * c["w"]]]), hi=_i64([[hkv * n]]), budgets=_i64([[0]]),
             counts=torch.empty(hkv, dtype=torch.int32, device=DEV), offs=torch.empty(hkv + 1, dtype=torch.int64, device=DEV),
             idx=torch.empty(B, dtype=torch.int32, device=DEV), kept=torch.empty(B, device=DEV),
             k_hat=torch.empty(B, c["d"], dtype=_dtype(c), device=DEV), v_hat=torch.empty(B, c["d"], dtype=_dtype(c), device=DEV))
    s["plan"] = lava.make_budget_plan(s["e"], 0, s["total"], s["lo"], s["hi"], s["budgets"])
    return s


def _prepare_batch(c, seed):
    gen, lens, hkv, d, B, desc, dt = _generator(seed), _lengths(c), c["hkv"], c["d"], c["budget"], _desc(c), _dtype(c)
    S, T = len(lens), sum(lens)
    q = torch.empty(S, c["hq"], c["w"], d, dtype=dt, device=DEV)
    k, v = (torch.empty(T * hkv, d, dtype=dt, device=DEV) for _ in range(2))
    start = [hkv * sum(lens[:b]) for b in range(S + 1)]
    for b, n in enumerate(lens):
        q[b], kb, vb = _draw_layer(c, n, 0.01, gen)
        k[start[b]: start[b + 1]], v[start[b]: start[b + 1]] = kb.view(-1, d), vb.view(-1, d)
    s = dict(c=c, desc=desc, lens=lens, q=q, k=k, v=v, start=start, widest=hkv * max(lens))
    s.update(scores=torch.empty(hkv * T, device=DEV), vbar=torch.empty(S, hkv, device=DEV), stat=torch.empty(S, device=DEV),
             ws=_bytes(lava.lava_window_scores_workspace_bytes(desc, S, T)),
             ws_sel=_bytes(lava.lava_select_batch_workspace_bytes(S, s["widest"])),
             e=torch.zeros(S, 1, device=DEV), total=_i64([B] * S), lo=_i64([[hkv * c["w"]]] * S), hi=_i64([[hkv * n] for n in lens]),
             budgets=_i64([[0]] * S), counts=torch.empty(S, hkv, dtype=torch.int32, device=DEV),
             offs=torch.empty(S, hkv + 1, dtype=torch.int64, device=DEV), idx=torch.empty(S, B, dtype=torch.int32, device=DEV),
             kept=torch.empty(S, B, device=DEV), k_hat=torch.empty(S, B, d, dtype=dt, device=DEV), v_hat=torch.empty(S, B, d, dtype=dt, device=DEV))
    s["plan"] = lava.make_budget_plan(s["e"], 0, s["total"], s["lo"], s["hi"], s["budgets"])
    part = lambda t, b: t[start[b]: start[b + 1]]  # noqa: E731
    s["select"] = (lava.SelectProblem * S)(*[
        lava.select_problem(part(s["scores"], b), B, s["counts"][b], s["offs"][b], s["idx"][b], s["kept"][b],
                            budget_dev=s["budgets"][b], primed=True) for b in range(S)])
    s["compact"] = (lava.CompactProblem * S)(*[
        lava.compact_problem(desc, lens[b], part(k, b), part(v, b), s["offs"][b], s["idx"][b], B, s["k_hat"][b], s["v_hat"][b])
        for b in range(S)])
    return s


def _stack_heavy(t, layers):
    """Layers attend more or less sharply: the share of strongly attended keys runs over 0.2 to 3 percent."""
    return 0.002 + 0.028 * ((t * 7) % layers) / layers


def _prepare_stack(c, seed):
    gen, L, n, hkv, d, total, desc, dt = _generator(seed), c["layers"], c["n"], c["hkv"], c["d"], c["total"], _desc(c), _dtype(c)
    dense = hkv * n
    q = torch.empty(L, c["hq"], c["w"], d, dtype=dt, device=DEV)
    k, v = (torch.empty(L, hkv, n, d, dtype=dt, device=DEV) for _ in range(2))
    for t in range(L):
        q[t], k[t], v[t] = _draw_layer(c, n, _stack_heavy(t, L), gen)
    s = dict(c=c, desc=desc, q=q, k=k, v=v)
    s.update(scores=torch.empty(L * dense, device=DEV), vbar=torch.empty(L, hkv, device=DEV), e=torch.empty(L, device=DEV),
             ws=_bytes(lava.lava_window_scores_workspace_bytes(desc, L, L * n)),
             ws_sel=_bytes(lava.lava_select_batch_workspace_bytes(L, dense)),
             total=_i64([total]), lo=_i64([[hkv * c["w"]] * L]), hi=_i64([[dense] * L]), budgets=_i64([[0] * L]),
             first=torch.zeros(L + 1, dtype=torch.int64, device=DEV), counts=torch.empty(L, hkv, dtype=torch.int32, device=DEV),
             offs=torch.empty(L, hkv + 1, dtype=torch.int64, device=DEV), idx=torch.empty(total, dtype=torch.int32, device=DEV),
             kept=torch.empty(total, device=DEV), k_hat=torch.empty(total, d, dtype=dt, device=DEV), v_hat=torch.empty(total, d, dtype=dt, device=DEV))
    s["select"] = (lava.SelectProblem * L)(*[
        lava.select_problem(s["scores"][t * dense: (t + 1) * dense], min(total, dense), s["counts"][t], s["offs"][t], s["idx"],
                            s["kept"], budget_dev=s["budgets"][0, t: t + 1], out_offset_dev=s["first"][t: t + 1]) for t in range(L)])
    s["compact"] = (lava.CompactProblem * L)(*[
        lava.compact_problem(desc, n, k[t], v[t], s["offs"][t], s["idx"], total, s["k_hat"], s["v_hat"],
                             out_offset_dev=s["first"][t: t + 1]) for t in range(L)])
    return s


def _prepare_cascade(c, seed):
    gen, L, n, hkv, d, w, desc, dt = _generator(seed), c["layers"], c["n"], c["hkv"], c["d"], c["w"], _desc(c), _dtype(c)
    layers = []
    for _ in range(L):
        # scores as the scoring step leaves them: plateaus of the pooling width, a heavy tail, the window at +inf
        base = torch.exp(2.0 * torch.randn(hkv, (n + 6) // 7, generator=gen, device=DEV)) * 1e-6
        scores = base.repeat_interleave(7, dim=1)[:, :n].contiguous()
        scores[:, n - w:] = math.inf
        layers.append(dict(scores=scores, k=torch.randn(hkv, n, d, generator=gen, device=DEV).to(dt),
                           v=torch.randn(hkv, n, d, generator=gen, device=DEV).to(dt)))
    state = lava.CascadeState(desc, L, c["total"], device=DEV)
    for t in state.k + state.v + state.pos + state.scores:
        t.zero_()
    state.e.copy_(1e-6 * (0.5 + torch.rand(L, generator=gen, device=DEV)))
    return dict(c=c, desc=desc, layers=layers, state=state, ws=_bytes(lava.lava_cascade_workspace_bytes(desc, n, L, c["total"])))


def _prepare_decode(c, seed):
    gen, S, R, tail, hq, hkv, d, desc, dt = _generator(seed), c["batch"], c["rows"], c["tail"], c["hq"], c["hkv"], c["d"], _desc(c), _dtype(c)
    # dynamic head budgets: uneven shares, now and then a head with nothing
    share = torch.exp(torch.randn(S, hkv, generator=gen, device=DEV)) * (torch.rand(S, hkv, generator=gen, device=DEV) > 0.05)
    share[:, 0] += 0.01
    ends = torch.floor(share.double().cumsum(1) / share.double().sum(1, keepdim=True) * R).to(torch.int64)
    offs = torch.cat([torch.zeros(S, 1, dtype=torch.int64, device=DEV), ends], 1)
    offs[:, -1] = R
    q = torch.randn(S, hq, d, generator=gen, device=DEV)
    k = torch.randn(S * R, d, generator=gen, device=DEV)
    rows = torch.randint(0, S * R, (max(1, S * R // 100),), generator=gen, device=DEV).unique()
    seq = rows // R
    g = torch.searchsorted(offs[seq, 1:].contiguous(), (rows % R).view(-1, 1), right=True).view(-1)
    head = g * (hq // hkv) + torch.randint(0, hq // hkv, rows.shape, generator=gen, device=DEV)
    _towards(k, q.view(S * hq, d), rows, seq * hq + head, gen)
    v = torch.randn(S * R, d, generator=gen, device=DEV) * torch.exp(0.5 * torch.randn(S * R, 1, generator=gen, device=DEV))
    s = dict(c=c, desc=desc, q=q.to(dt), k=k.to(dt), v=v.to(dt), offs=offs.contiguous(), k_tail=None, v_tail=None)
    if tail:
        s["k_tail"], s["v_tail"] = (torch.randn(S, hkv, 256, d, generator=gen, device=DEV).to(dt) for _ in range(2))
    s.update(out=torch.empty(S, hq, d, device=DEV), lse=torch.empty(S, hq, device=DEV),
             ws=_bytes(lava.lava_decode_workspace_bytes(desc, S, R, tail)))
    return s


def prepare(case, seed):
    return {"layer": _prepare_layer, "batch": _prepare_batch, "stack": _prepare_stack, "cascade": _prepare_cascade,
            "decode": _prepare_decode}[case["kind"]](case, seed)


# --------------------------------------------------------------------------------------------- passes
def _evicted(s, e):
    return {"scores": s["scores"], "vbar": s["vbar"], "stat": e, "budgets": s["budgets"], "counts": s["counts"], "offsets": s["offs"],
            "index": s["idx"], "kept_scores": s["kept"], "k": s["k_hat"], "v": s["v_hat"]}


def run(s):
    c, desc = s["c"], s["desc"]
    if c["kind"] == "layer":
        lava.lava_window_scores(desc, [c["n"]], s["q"], s["k"], s["v"], lse=s["lse"], scores=s["scores"], vbar=s["vbar"],
                                layer_stat=s["stat"], workspace=s["ws"], select_workspace=s["ws_sel"], budget_plan=s["plan"])
        lava.lava_select_topk(c["hkv"], s["scores"], c["budget"], budget_dev=s["budgets"], head_counts=s["counts"],
                              head_offsets=s["offs"], kept_idx=s["idx"], kept_scores=s["kept"], workspace=s["ws_sel"], primed=True)
        lava.lava_compact_kv(desc, c["n"], s["k"], s["v"], s["offs"], s["idx"], c["budget"], k_out=s["k_hat"], v_out=s["v_hat"])
        return _evicted(s, s["stat"])
    if c["kind"] == "batch":
        lava.lava_window_scores(desc, s["lens"], s["q"], s["k"], s["v"], scores=s["scores"], vbar=s["vbar"], layer_stat=s["stat"],
                                workspace=s["ws"], select_workspace=s["ws_sel"], budget_plan=s["plan"])
        lava.lava_select_topk_batch(c["hkv"], s["select"], s["widest"], workspace=s["ws_sel"])
        lava.lava_compact_batch(desc, s["compact"])
        return _evicted(s, s["stat"])
    if c["kind"] == "stack":
        L, dense = c["layers"], c["hkv"] * c["n"]
        lava.lava_window_scores(desc, [c["n"]] * L, s["q"], s["k"], s["v"], scores=s["scores"], vbar=s["vbar"], layer_stat=s["e"],
                                workspace=s["ws"])
        lava.lava_layer_budgets(s["e"].view(1, L), s["total"], s["lo"], s["hi"], budgets=s["budgets"])
        torch.cumsum(s["budgets"][0], 0, out=s["first"][1:])
        lava.lava_select_topk_batch(c["hkv"], s["select"], dense, workspace=s["ws_sel"])
        lava.lava_compact_batch(desc, s["compact"])
        return _evicted(s, s["e"])
    if c["kind"] == "cascade":
        st = s["state"]
        st.reset()
        for t, x in enumerate(s["layers"]):
            lava.lava_cascade_step(desc, t, c["n"], x["k"], x["v"], x["scores"], st, c["total"], workspace=s["ws"])
        i = st.cur
        return {"k": st.k[i], "v": st.v[i], "pos": st.pos[i], "scores": st.scores[i], "offsets": st.head_offsets[i],
                "start": st.layer_start[i], "counts": st.head_counts, "budgets": st.budgets}
    out, lse = lava.lava_decode_attention(desc, c["batch"], s["q"], s["k"], s["v"], s["offs"], c["rows"], k_tail=s["k_tail"],
                                          v_tail=s["v_tail"], tail_len=c["tail"], tail_capacity=256 if c["tail"] else 0,
                                          out=s["out"], lse=s["lse"], workspace=s["ws"])
    return {"out": out, "lse": lse}


# ------------------------------------------------------------------------------- work and correctness
def _evict_work(c, n, budget):
    """One layer of one sequence: Q, K and V in, the scores, the packed rows, their index and scores out."""
    e = 2 if c["dtype"] == "bf16" else 4
    row, score = c["d"] * e, c.get("score", "lava")
    v_rows = budget if score == "attention" else c["hkv"] * n
    return {"bytes": c["hq"] * c["w"] * (row + (4 if c.get("lse") else 0)) + (c["hkv"] * n + v_rows) * row + 4 * c["hkv"] * n
            + budget * (2 * row + 8),
            "flops": 2.0 * c["hq"] * c["w"] * n * c["d"] + v_rows * c["d"]}


def work(case):
    c = case
    if c["kind"] == "layer":
        return _evict_work(c, c["n"], c["budget"])
    if c["kind"] == "batch":
        parts = [_evict_work(c, n, c["budget"]) for n in _lengths(c)]
        return {k: sum(p[k] for p in parts) for k in ("bytes", "flops")}
    if c["kind"] == "stack":
        one = _evict_work(c, c["n"], c["total"] // c["layers"])
        return {k: c["layers"] * one[k] for k in one}
    row = c["d"] * (2 if c["dtype"] == "bf16" else 4)
    if c["kind"] == "cascade":
        # a step reads the arriving layer's scores and moves the retained rows (K, V, position, score)
        return {"bytes": c["layers"] * (4 * c["hkv"] * c["n"] + c["total"] * 2 * (2 * row + 8)), "flops": c["layers"] * c["hkv"] * c["n"]}
    rows = c["batch"] * (c["rows"] + c["hkv"] * c["tail"])
    return {"bytes": 2 * rows * row + c["batch"] * c["hq"] * (row + 4 * c["d"] + 4), "flops": 4.0 * rows * c["d"] * c["hq"] / c["hkv"]}


def tolerance(case):
    if case["kind"] == "cascade":   # selections on given scores, and copies
        return "exact"
    # 32-bit sums of exact products (bf16) or 32-bit products; integers differ only where two entries at the
    # threshold are a rounding apart.  Errors against 64 bits: 2e-7 to 1e-6 over the listed and drawn cases
    return {"rel": 4e-6, "max": 4e-5, "differ": 0.002}


def _exact_scores(c, n, q, k, v, lse):
    """scores [H_kv, n], vbar [H_kv], statistic of one layer in 64 bits."""
    hkv, w, kind = c["hkv"], c["w"], c.get("score", "lava")
    G, scores, vbar = c["hq"] // hkv, torch.full((hkv, n), math.inf, dtype=torch.float64, device=DEV), []
    for g in range(hkv):
        x = _logits(c, q, k, g, torch.float64)
        z = x.logsumexp(-1, keepdim=True) if lse is None else lse.view(hkv, G, w, 1)[g].double()
        raw = torch.exp(x - z).mean(1).amax(0)[: n - w]
        pooled = torch.nn.functional.max_pool1d(raw.view(1, 1, -1), 7, 1, 3).view(-1)
        norm = v[g].double().abs().sum(-1)
        vbar.append(torch.ones_like(norm[0]) if kind == "attention" else norm.max())
        scores[g, : n - w] = pooled * (norm[: n - w] if kind == "token_norm" else vbar[-1])
    s = scores[:, : n - w]
    S, T = s.sum(), torch.xlogy(s, s).sum()
    return scores, torch.stack(vbar), (S.log() - T / S) / (hkv * (n - w))


def _exact_evicted(parts):
    out = dict.fromkeys(("budgets", "counts", "offsets", "index", "kept_scores", "k", "v"))
    out.update(scores=torch.cat([p[0].view(-1) for p in parts]), vbar=torch.stack([p[1] for p in parts]),
               stat=torch.stack([p[2] for p in parts]))
    return out


def exact(case, seed):
    c = case
    if c["kind"] == "layer":
        s = _prepare_layer(c, seed)
        return _exact_evicted([_exact_scores(c, c["n"], s["q"], s["k"], s["v"], s["lse"])])
    if c["kind"] == "batch":
        s = _prepare_batch(c, seed)
        part = lambda t, b: t[s["start"][b]: s["start"][b + 1]].view(c["hkv"], -1, c["d"])  # noqa: E731
        return _exact_evicted([_exact_scores(c, n, s["q"][b], part(s["k"], b), part(s["v"], b), None) for b, n in enumerate(s["lens"])])
    if c["kind"] == "stack":
        s = _prepare_stack(c, seed)
        return _exact_evicted([_exact_scores(c, c["n"], s["q"][t], s["k"][t], s["v"][t], None) for t in range(c["layers"])])
    if c["kind"] == "cascade":
        return None
    s = _prepare_decode(c, seed)
    S, R, hq, hkv, d = c["batch"], c["rows"], c["hq"], c["hkv"], c["d"]
    G, offs = hq // hkv, s["offs"].tolist()
    q = s["q"].double().view(S, hkv, G, d)
    out, lse = torch.zeros(S, hkv, G, d, dtype=torch.float64, device=DEV), torch.full((S, hkv, G), -math.inf, dtype=torch.float64, device=DEV)
    for b in range(S):
        for g in range(hkv):
            lo, hi = b * R + offs[b][g], b * R + offs[b][g + 1]
            k, v = s["k"][lo:hi].double(), s["v"][lo:hi].double()
            if c["tail"]:
                k = torch.cat([k, s["k_tail"][b, g, : c["tail"]].double()])
                v = torch.cat([v, s["v_tail"][b, g, : c["tail"]].double()])
            if k.shape[0]:
                x = q[b, g] @ k.t().contiguous() / math.sqrt(d)
                lse[b, g] = x.logsumexp(-1)
                out[b, g] = torch.softmax(x, -1) @ v
    return {"out": out.view(S, hq, d), "lse": lse.view(S, hq)}
