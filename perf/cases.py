"""The calls whose speed this repository is measured by: token compression of video inputs in its three stages.

A case is one call of `paper_2506_02850_amd.binding` as a serving program makes it, with its inputs resident on the GPU:

  frames   metok_segment_compress / metok_segment_compress_batched (segmentation, key events / frames, adaptive pooling)
  prune    metok_prefill_prune / metok_prefill_prune_batched (attention scores, selection, compaction of the hidden states)
  cache    metok_kv_compact / metok_kv_compact_paged / metok_kv_relink_paged (compaction of the KV cache)

The program keeps the workspace between calls, and the output buffers wherever an output is longer than what one call
writes (their tails stay zero then).  Inputs are random tensors with the structure the method works on: events of frames
around a common centre, and visual tokens of which as many as the quota allows draw clearly more attention than the
others.  That gap at the quota keeps the selections the same whatever order a sum is taken in, so that whole outputs
can be compared; within the two groups scores spread as attention scores do.
"""
import math
import random

import torch

from paper_2506_02850_amd import binding as B

DEV = "cuda"


# ---------------------------------------------------------------------------------------------------------------------
# cases
# ---------------------------------------------------------------------------------------------------------------------
def _frames(**kw):
    c = dict(kind="frames", dtype="bf16", batch=1, T=32, gh=24, gw=24, d=1024, k=8, alpha=0.5, beta=0.4, s1=2, s2=3,
             sim=B.SIM_FLAT, reduce=B.EVENT_MEAN, edge=B.POOL_FLOOR)
    c.update(kw)
    return c


def _prune(**kw):
    c = dict(kind="prune", dtype="bf16", batch=1, n_vis=4096, vis_start=0, n_text=64, Tq=64, Hq=28, Hkv=4, dh=128, D=3584,
             events=8, classes="key", keep_key=0.5, keep_non=0.25, mode=B.SCORE_CAUSAL_ALL, attention=True, in_place=False)
    c.update(kw)
    return c


def _cache(**kw):
    c = dict(kind="cache", form="dense", dtype="bf16", batch=1, layers=28, Hkv=4, dh=128, n_vis=4096, n_text=64, page=16,
             l1=3, l2=10, l3=19, keep1=0.5, keep2=0.25, keep3=0.125, block=1)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: a handful of frames, where launches and host work are everything (the Tiny configuration)
        _frames(name="frames_tiny_f32", dtype="f32", T=8, gh=4, gw=4, d=64, k=4),
        # one video of 32 SigLIP frames at its appendix setting: the ordinary request of a LLaVA-OneVision service
        _frames(name="frames_32x27x27", T=32, gh=27, gw=27, d=1152, k=5, alpha=0.5, beta=0.4),
        # one video of 128 frames at the LongVA setting
        _frames(name="frames_128x24x24", T=128, k=13, alpha=0.5, beta=0.45),
        # a batch of videos of 64 frames on the odd grid (the frame count of the VILA-shaped workload)
        _frames(name="frames_8x64x27x27", batch=8, T=64, gh=27, gw=27, d=1152, k=3, alpha=0.5, beta=0.4),
        # throughput: eight videos of 256 frames, every frame pooled with stride 2
        _frames(name="frames_8x256_uniform", batch=8, T=256, k=16, alpha=1.0, beta=1.0, s1=2, s2=2),
        # one pruning level of one video after adaptive pooling of 32 frames: a few thousand tokens, a request's latency
        _prune(name="prune_2243", n_vis=2243, events=5, keep_key=0.76, keep_non=0.38),
        # the same for a decoder with as many kv heads as query heads
        _prune(name="prune_4507_mha", n_vis=4507, Hq=40, Hkv=40, D=5120, events=3, keep_key=0.65, keep_non=0.325),
        # float32 activations, small heads
        _prune(name="prune_5000_f32", dtype="f32", n_vis=5000, Hq=14, Hkv=2, dh=64, D=896, Tq=32, events=8),
        # one video of 128 frames with quotas per event (the retention class is the event)
        _prune(name="prune_18432_events", n_vis=18432, events=13, classes="event", keep_key=0.25, keep_non=0.25),
        # throughput: level 1 of eight LongVA-shaped videos
        _prune(name="prune_8x36864", batch=8, n_vis=36864, n_text=128, events=16, keep_key=0.5, keep_non=0.5),
        # the decoder's cache after three levels: dense, four videos of 36864 visual tokens
        _cache(name="cache_4x36992", batch=4, n_vis=36864, n_text=128),
        # one request's cache in pages of 16 rows, moved through the page table
        _cache(name="cache_paged_18496", form="paged", n_vis=18432, n_text=64),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_any(rng):
    kind = rng.choice(("frames", "frames", "prune", "prune", "cache"))
    if kind == "frames":
        dtype = rng.choice(("bf16", "bf16", "f32"))
        gh = rng.choice((rng.randint(4, 28), 16, 24, 27))
        gw = rng.choice((gh, gh, rng.randint(4, 28)))
        T = _log(rng, 4, 512)
        s1, s2 = rng.choice(((2, 3), (2, 3), (2, 2), (1, 2), (2, 4), (3, 4)))
        alpha = rng.choice((0.3, 0.5, 0.5, 0.7, 1.0))
        return _frames(dtype=dtype, batch=rng.choice((1, 1, 2, 4, 8)), T=T, gh=gh, gw=gw,
                       d=rng.choice((1024, 1152, 768, 8 * _log(rng, 8, 256))), k=max(1, min(T // 3, rng.randint(2, 16))),
                       alpha=alpha, beta=rng.choice((0.3, 0.4, 0.45, 1.0)), s1=s1, s2=s2,
                       sim=rng.choice((B.SIM_FLAT, B.SIM_FLAT, B.SIM_FLAT, B.SIM_TOKEN_MEAN)),
                       reduce=rng.choice((B.EVENT_MEAN, B.EVENT_MEAN, B.EVENT_MAX)),
                       edge=rng.choice((B.POOL_FLOOR, B.POOL_FLOOR, B.POOL_CEIL)))
    if kind == "prune":
        Hq, Hkv, dh, D = rng.choice(((28, 4, 128, 3584), (28, 4, 128, 3584), (40, 40, 128, 5120), (14, 2, 64, 896),
                                     (32, 8, 128, 4096), (16, 16, 64, 1024), (8, 2, 256, 2048), (4, 4, 32, 256)))
        dtype = "f32" if dh <= 128 and rng.random() < 0.25 else "bf16"
        Tq = rng.choice((64, 64, 32, 16, 1, rng.randint(2, 100)))
        batch = rng.choice((1, 1, 1, 2, 4, 8))
        return _prune(dtype=dtype, batch=batch, n_vis=_log(rng, 200, 40000), vis_start=rng.choice((0, 0, 14, rng.randint(1, 60))),
                      n_text=Tq + rng.choice((0, 0, rng.randint(1, 64))), Tq=Tq, Hq=Hq, Hkv=Hkv, dh=dh, D=D,
                      events=rng.randint(2, 16), classes=rng.choice(("key", "key", "event", "all")),
                      keep_key=rng.choice((0.5, 0.55, 0.76)), keep_non=rng.choice((0.25, 0.275, 0.38, 0.0)),
                      mode=rng.choice((B.SCORE_CAUSAL_ALL, B.SCORE_CAUSAL_ALL, B.SCORE_VISUAL_ONLY)),
                      attention=rng.random() < 0.85, in_place=D * (2 if dtype == "bf16" else 4) <= 16384 and rng.random() < 0.15)
    layers = rng.choice((2, 24, 28, 28, 40))
    return _cache(form=rng.choice(("dense", "dense", "paged", "relink")), dtype=rng.choice(("bf16", "bf16", "bf16", "f32")),
                  batch=rng.choice((1, 1, 2, 4)), layers=layers, Hkv=rng.choice((2, 4, 4, 8, 40)), dh=rng.choice((64, 128, 128)),
                  n_vis=_log(rng, 300, 37000), n_text=rng.choice((64, 128, rng.randint(1, 200))), page=rng.choice((16, 16, 64)),
                  l1=layers // 9, l2=layers // 3, l3=2 * layers // 3, block=rng.choice((1, 1, 16)))


def draw(rng):
    most = max(_cost(c) for c in listed())
    memory = max(_memory(c) for c in listed())
    while True:
        c = _draw_any(rng)
        if _cost(c) <= most and _memory(c) <= memory:
            return c


def _cost(c):
    """A rough time of one pass, for the bound on drawn cases only."""
    w = work(c)
    return w["bytes"] / 5e12 + 2 * w["flops"] / (0.8e15 if c["dtype"] == "bf16" else 8e13)


def _memory(c):
    e = _esize(c)
    if c["kind"] == "frames":
        return 4 * c["batch"] * c["T"] * c["gh"] * c["gw"] * c["d"] * e / 3
    if c["kind"] == "prune":
        return c["batch"] * (c["n_vis"] + c["n_text"]) * (c["Hkv"] * c["dh"] + 2 * c["D"]) * e
    return 2 * c["batch"] * c["layers"] * c["Hkv"] * (c["n_vis"] + c["n_text"]) * c["dh"] * e


# ---------------------------------------------------------------------------------------------------------------------
# what one pass cannot do without
# ---------------------------------------------------------------------------------------------------------------------
def _esize(c):
    return 2 if c["dtype"] == "bf16" else 4


def _side(g, s, edge):
    return max(1, g // s) if edge == B.POOL_FLOOR else -(-g // s)


def _stride(c, s):
    return max(1, min(math.ceil(s - 1e-9), max(c["gh"], c["gw"])))


def _strides(c):
    """(key event, key frame) -> stride"""
    return {(True, True): _stride(c, c["s1"]), (True, False): _stride(c, c["s2"]),
            (False, True): _stride(c, c["s1"] / c["alpha"]), (False, False): _stride(c, c["s2"] / c["alpha"])}


def work(case):
    c, e = case, _esize(case)
    if c["kind"] == "frames":
        rows = {key: _side(c["gh"], s, c["edge"]) * _side(c["gw"], s, c["edge"]) for key, s in _strides(c).items()}
        share = math.ceil(c["alpha"] * c["k"] - 1e-9) / c["k"]
        per_frame = sum((share if ke else 1 - share) * (c["beta"] if kf else 1 - c["beta"]) * rows[ke, kf] for ke, kf in rows)
        n = c["batch"] * c["T"] * c["gh"] * c["gw"] * c["d"]
        return {"bytes": n * e + c["batch"] * c["T"] * per_frame * (c["d"] * e + 4), "flops": 7 * n}
    if c["kind"] == "prune":
        S = c["vis_start"] + c["n_vis"] + c["n_text"]
        keep = sum(_quotas(c, [c["n_vis"] // _n_classes(c)] * _n_classes(c)))
        moved = (S - c["n_vis"] + keep) * c["D"] * e * 2
        meta = c["n_vis"] * 12 + keep * 16
        att = (c["Hkv"] * S + c["Hq"] * c["Tq"]) * c["dh"] * e if c["attention"] else 0
        return {"bytes": c["batch"] * (moved + meta + att),
                "flops": c["batch"] * 2 * c["Hq"] * c["Tq"] * S * c["dh"] if c["attention"] else 0}
    row = c["Hkv"] * c["dh"] * e * 2                       # K and V of one token in one layer
    total = 0
    for layer in range(c["layers"]):
        n = _kept_of_layer(c, layer)
        if n is not None:
            # with whole pages kept together a table entry replaces the copy
            total += n * 4 + (0 if c["form"] == "relink" and c["block"] % c["page"] == 0 else 2 * n * row)
    return {"bytes": c["batch"] * max(total, 4), "flops": 0}


# ---------------------------------------------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------------------------------------------
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _torch_dtype(c):
    return torch.bfloat16 if c["dtype"] == "bf16" else torch.float32


def _lengths(r, total, parts):
    cuts = sorted(r.sample(range(1, total), parts - 1)) if parts > 1 else []
    return [b - a for a, b in zip([0] + cuts, cuts + [total])]


def _i32(x):
    return torch.tensor(x, dtype=torch.int32, device=DEV)


def _prepare_frames(c, seed):
    r, g, dt = random.Random(seed), _gen(seed), _torch_dtype(c)
    Bn, T, N, d, k = c["batch"], c["T"], c["gh"] * c["gw"], c["d"], c["k"]
    feats = torch.empty((Bn, T, N, d), dtype=dt, device=DEV)
    text = torch.empty((Bn, d), dtype=dt, device=DEV)
    sigma = 2.0 / math.sqrt(d)                                # the noise of a token is twice as long as its centre
    for b in range(Bn):
        centres = torch.randn((k, d), generator=g, device=DEV)
        centres /= centres.norm(dim=1, keepdim=True)
        weights = [1.0 - 0.8 * i / max(1, k - 1) for i in range(k)]
        r.shuffle(weights)
        t = (torch.tensor(weights, device=DEV)[:, None] * centres).sum(0)
        t /= t.norm()
        text[b] = t.to(dt)
        event, lean = [], []
        for e, n in enumerate(_lengths(r, T, k)):
            event += [e] * n
            steps = [0.1 * (i + 1) / n for i in range(n)]     # frames of an event differ in how much they say about the text
            r.shuffle(steps)
            lean += steps
        base = centres[torch.tensor(event, device=DEV)] + torch.tensor(lean, device=DEV)[:, None] * t
        x = torch.randn((T, N, d), generator=g, device=DEV)
        feats[b] = x.mul_(sigma).add_(base[:, None, :]).to(dt)
        del x
    cap = B.metok_compress_encoder_tokens_capacity_rows(T, c["gh"], c["gw"], c["s1"], c["s2"], c["edge"])
    lead = (Bn,) if Bn > 1 else ()
    out = dict(out_tokens=torch.zeros(lead + (cap, d), dtype=dt, device=DEV),
               token_event=torch.zeros(lead + (cap,), dtype=torch.int32, device=DEV))
    code = B.BF16 if c["dtype"] == "bf16" else B.F32
    need = B.lib().metok_segment_compress_batched_workspace_bytes(Bn, T, c["gh"], c["gw"], d, code) if Bn > 1 else \
        B.lib().metok_segment_compress_workspace_bytes(T, c["gh"], c["gw"], d, code)
    return dict(case=c, feats=feats if Bn > 1 else feats[0], text=text if Bn > 1 else text[0], out=out,
                workspace=torch.empty(max(int(need), 256), dtype=torch.uint8, device=DEV))


def _n_classes(c):
    return {"key": 2, "event": c["events"], "all": 1}[c["classes"]]


def _quotas(c, population):
    if c["classes"] == "key":
        ratio = [c["keep_key"], c["keep_non"]]
    else:
        ratio = [c["keep_key"]] * len(population)
    return [min(n, math.ceil(f * n - 1e-9)) for f, n in zip(ratio, population)]


def _prepare_prune(c, seed):
    # the events' lengths belong to the case, so that the shapes of the outputs do not depend on the seed
    r, g, dt = random.Random(c["n_vis"] + c["events"]), _gen(seed), _torch_dtype(c)
    Bn, n_vis, dh, Hq, Hkv, Tq, E = c["batch"], c["n_vis"], c["dh"], c["Hq"], c["Hkv"], c["Tq"], c["events"]
    v0, S = c["vis_start"], c["vis_start"] + c["n_vis"] + c["n_text"]
    n_cls = _n_classes(c)
    hidden = torch.empty((Bn, S, c["D"]), dtype=dt, device=DEV)
    q = torch.empty((Bn, Hq, Tq, dh), dtype=dt, device=DEV)
    keys = torch.empty((Bn, Hkv, S, dh), dtype=dt, device=DEV)
    token_event = torch.empty((Bn, n_vis), dtype=torch.int32, device=DEV)
    token_seg = torch.empty((Bn, n_vis), dtype=torch.int32, device=DEV)
    orig = torch.empty((Bn, n_vis), dtype=torch.int32, device=DEV)
    scores = torch.empty((Bn, n_vis), dtype=torch.float32, device=DEV)
    weight = 0.7 + 0.6 * torch.rand((Bn, E), generator=g, device=DEV)
    # few query rows average little: their random part is smaller then, so that the gap at the quota stays
    noise = min(1.0, math.sqrt(Hq * Tq / 256.0))
    pull = math.sqrt(math.log(10.0) * math.sqrt(dh))          # a salient token's logits are higher by log 10
    quotas = []
    for b in range(Bn):
        ev = torch.repeat_interleave(torch.arange(E, device=DEV), torch.tensor(_lengths(r, n_vis, E), device=DEV))
        is_key = [1 if i < (E + 1) // 2 else 0 for i in range(E)]
        r.shuffle(is_key)
        if c["classes"] == "key":
            seg = 1 - torch.tensor(is_key, device=DEV)[ev]
        else:
            seg = ev if c["classes"] == "event" else torch.zeros_like(ev)
        population = torch.bincount(seg, minlength=n_cls).tolist()
        quota = _quotas(c, population)
        quotas.append(quota)
        salient = torch.zeros(n_vis, dtype=torch.bool, device=DEV)
        for s in range(n_cls):
            members = torch.nonzero(seg == s).flatten()
            salient[members[torch.randperm(members.numel(), generator=g, device=DEV)[:quota[s]]]] = True
        token_event[b], token_seg[b] = ev.int(), seg.int()
        orig[b] = (2 * torch.arange(n_vis, device=DEV) + torch.randint(0, 2, (n_vis,), generator=g, device=DEV)).int()
        if c["attention"]:
            u = torch.randn((Hkv, dh), generator=g, device=DEV)
            u /= u.norm(dim=1, keepdim=True)
            mu = torch.randn((E, dh), generator=g, device=DEV)
            kb = torch.randn((Hkv, S, dh), generator=g, device=DEV)
            kb[:, v0:v0 + n_vis] += 0.15 * mu[ev]
            kb -= (kb * u[:, None]).sum(-1, keepdim=True) * u[:, None]
            kb[:, v0:v0 + n_vis] += pull * salient.float()[None, :, None] * u[:, None]
            keys[b] = kb.to(dt)
            ug = u.repeat_interleave(Hq // Hkv, 0)[:, None]
            qb = noise * torch.randn((Hq, Tq, dh), generator=g, device=DEV)
            qb += (pull - (qb * ug).sum(-1, keepdim=True)) * ug
            q[b] = qb.to(dt)
            del kb, qb
        else:
            scores[b] = (torch.randperm(n_vis, generator=g, device=DEV) + 1).float() / n_vis
        shift = torch.randn(E, generator=g, device=DEV)
        hb = torch.randn((S, c["D"]), generator=g, device=DEV)
        hb[v0:v0 + n_vis] += shift[ev][:, None]
        hidden[b] = hb.to(dt)
        del hb
    code = B.BF16 if c["dtype"] == "bf16" else B.F32
    heads = (Hq, Hkv, dh, Tq) if c["attention"] else (0, 0, 0, 0)
    need = B.lib().metok_prefill_prune_batched_workspace_bytes(Bn, S, *heads, n_vis, code) if Bn > 1 else \
        B.lib().metok_prefill_prune_workspace_bytes(S, *heads, n_vis, code)
    state = dict(case=c, hidden=hidden, q=q, keys=keys, token_event=token_event, token_seg=token_seg, orig=orig, weight=weight,
                 scores=scores, quotas=quotas, workspace=torch.empty(max(int(need), 256), dtype=torch.uint8, device=DEV))
    if Bn == 1:
        for name in ("hidden", "q", "keys", "token_event", "token_seg", "orig", "weight", "scores"):
            state[name] = state[name][0]
    else:
        keep = [sum(x) for x in quotas]
        i32 = dict(dtype=torch.int32, device=DEV)
        state["out"] = {name: torch.zeros((Bn, max(keep)), **i32) for name in ("kept_idx", "token_seg_out", "token_event_out", "orig_idx_out")}
        if not c["in_place"]:
            state["out"]["hidden_out"] = torch.zeros((Bn, S - n_vis + max(keep), c["D"]), dtype=dt, device=DEV)
    return state


def _kept_of_layer(c, layer):
    """Rows that a layer keeps, or None for a layer that is left alone."""
    if layer < c["l1"]:
        return None
    share = c["keep1"] if layer < c["l2"] else c["keep2"] if layer < c["l3"] else c["keep3"]
    blocks = -(-c["n_vis"] // c["block"])
    whole = max(1, int(share * blocks))
    return min(c["n_vis"], whole * c["block"]) + c["n_text"]


def _prepare_cache(c, seed):
    g, dt = _gen(seed), _torch_dtype(c)
    Bn, L, n_vis = c["batch"], c["layers"], c["n_vis"]
    S = n_vis + c["n_text"]
    if c["form"] == "dense":
        shape = (Bn, c["Hkv"], S, c["dh"])
        table = None
    else:
        per_seq = -(-S // c["page"])
        shape = (Bn * per_seq, c["Hkv"], c["page"], c["dh"])
        table = torch.randperm(Bn * per_seq, generator=g, device=DEV).int().view(Bn, per_seq)
    kv = torch.empty((L, 2) + shape, dtype=dt, device=DEV)
    for layer in range(L):
        kv[layer].normal_(generator=g)
    # nested retained sets, one per level: whole blocks of visual tokens (of one token, or of a page), then the text rows
    full = n_vis // c["block"]                                 # blocks that are whole: the ragged one at the end is not kept
    order = [torch.randperm(full, generator=g, device=DEV) for _ in range(Bn)]
    sets, idx = {}, []
    for layer in range(L):
        n = _kept_of_layer(c, layer)
        if n is None:
            idx.append(None)
            continue
        if n not in sets:
            whole = min(full, max(1, int((n - c["n_text"]) // c["block"])))
            rows = torch.stack([torch.sort(o[:whole]).values for o in order])
            rows = (rows[:, :, None] * c["block"] + torch.arange(c["block"], device=DEV)).reshape(Bn, -1)
            text = torch.arange(n_vis, S, device=DEV).expand(Bn, -1)
            sets[n] = torch.cat([rows, text], 1).int().contiguous()
        idx.append(sets[n])
    code = B.BF16 if c["dtype"] == "bf16" else B.F32
    if c["form"] == "relink":
        need = B.lib().metok_kv_relink_paged_workspace_bytes(L, Bn, c["Hkv"], c["page"], table.shape[1], c["dh"], code)
    else:
        need = B.metok_kv_compact_workspace_bytes(L, Bn, c["Hkv"], S if table is None else table.shape[1] * c["page"], c["dh"], code)
    return dict(case=c, kv=kv, k=[kv[i, 0] for i in range(L)], v=[kv[i, 1] for i in range(L)], idx=idx, table=table, len_in=[S] * L,
                new_len=torch.zeros(L, dtype=torch.int32, device=DEV),
                workspace=torch.empty(max(int(need), 256), dtype=torch.uint8, device=DEV))


def prepare(case, seed):
    return {"frames": _prepare_frames, "prune": _prepare_prune, "cache": _prepare_cache}[case["kind"]](case, seed)


# ---------------------------------------------------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------------------------------------------------
def run(state):
    c = state["case"]
    if c["kind"] == "frames":
        call = B.metok_segment_compress_batched if c["batch"] > 1 else B.metok_segment_compress
        return call(state["feats"], c["gh"], c["gw"], c["k"], state["text"], c["alpha"], c["beta"], c["s1"], c["s2"],
                    sim_mode=c["sim"], event_reduce=c["reduce"], pool_edge=c["edge"], workspace=state["workspace"], out=state["out"])
    if c["kind"] == "prune":
        kw = dict(token_event=state["token_event"], event_weight=state["weight"], orig_idx=state["orig"],
                  workspace=state["workspace"], score_mode=c["mode"])
        if c["attention"]:
            kw.update(q_text=state["q"], k_all=state["keys"])
        else:
            kw.update(scores=state["scores"])
        hidden = state["hidden"]
        if c["batch"] > 1:
            if c["in_place"]:
                kw["hidden_out"] = hidden
            res = B.metok_prefill_prune_batched(hidden, c["vis_start"], c["n_vis"], state["token_seg"], state["quotas"], out=state["out"], **kw)
            if c["in_place"]:                                  # the rows behind the compacted sequence are unspecified
                rows = hidden.shape[1] - c["n_vis"]
                res["hidden_out"] = [hidden[b, :rows + n] for b, n in enumerate(res["n_keep"])]
            return res
        if c["in_place"]:
            kw["hidden_out"] = hidden[:hidden.shape[0] - c["n_vis"] + sum(state["quotas"][0])]
        return B.metok_prefill_prune(hidden, c["vis_start"], c["n_vis"], state["token_seg"], state["quotas"][0], **kw)
    if c["form"] == "relink":
        res = B.metok_kv_relink_paged(state["k"], state["v"], state["table"], state["idx"], len_in=state["len_in"], workspace=state["workspace"])
        return {"kv": state["kv"], **{name: x for name, x in res.items() if name != "workspace"}}
    if c["form"] == "paged":
        new_len = B.metok_kv_compact_paged(state["k"], state["v"], state["table"], state["idx"], state["new_len"], state["workspace"])
    else:
        new_len = B.metok_kv_compact(state["k"], state["v"], state["idx"], state["new_len"], state["workspace"])
    return {"kv": state["kv"], "new_len": new_len}


def tolerance(case):
    if case["kind"] == "cache" or (case["kind"] == "prune" and not case["attention"]):
        return "exact"                                         # rows are copied, nothing is computed
    if case["kind"] == "prune":
        # the float32 mean of thousands of softmax probabilities, summed in any order, exponentials of one instruction
        # (measured against 64 bits: 2e-7 to 6e-7 for both types of input)
        return {"rel": 3e-6, "max": 3e-5}
    if case["dtype"] == "f32":
        return {"rel": 4e-6, "max": 4e-5}                      # float32 sums over a frame
    return {"rel": 2e-3, "max": 1e-2}                          # pooled tokens are rounded once to bf16: one unit in the last place


# ---------------------------------------------------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------------------------------------------------
def _cos(a, den):
    return torch.where(den < 1e-12, torch.zeros_like(a), a / den.clamp_min(1e-300))


def _top(values, n):
    """The n highest values, the lower index first among equals, as a set of positions."""
    return set(sorted(range(len(values)), key=lambda i: (-values[i], i))[:n])


def _exact_video(c, feats, text):
    T, N, d, k = c["T"], c["gh"] * c["gw"], c["d"], c["k"]
    t = text.double()
    norm2, frame_score, pair = [], [], []
    before = None
    for f in range(T):
        x = feats[f].double()
        n = x.square().sum(1).sqrt()
        frame_score.append(_cos(x @ t, n * t.norm()).mean())
        norm2.append(n.square().sum())
        if before is not None:
            if c["sim"] == B.SIM_TOKEN_MEAN:
                pair.append(_cos((x * before[0]).sum(1), n * before[1]).mean())
            else:
                pair.append(_cos((x * before[0]).sum(), (norm2[-1] * norm2[-2]).sqrt()))
        before = (x, n)
    sim = torch.stack(pair) if pair else torch.zeros(0, dtype=torch.float64, device=feats.device)
    score = torch.stack(frame_score)
    S = sim.tolist()
    starts = [0] + [i + 1 for i in sorted(sorted(range(T - 1), key=lambda i: (S[i], i))[:k - 1])] + [T]
    fs = score.tolist()
    spans = list(zip(starts, starts[1:]))
    event_score = [max(fs[a:b]) if c["reduce"] == B.EVENT_MAX else sum(fs[a:b]) / (b - a) for a, b in spans]
    key_events = _top(event_score, math.ceil(c["alpha"] * k - 1e-9))
    strides = _strides(c)
    tokens = []
    for e, (a, b) in enumerate(spans):
        key_frames = _top(fs[a:b], min(b - a, math.ceil(c["beta"] * (b - a) - 1e-9)))
        for f in range(a, b):
            s = strides[e in key_events, (f - a) in key_frames]
            x = feats[f].double().view(c["gh"], c["gw"], d).permute(2, 0, 1)[None]
            if c["edge"] == B.POOL_CEIL:
                p = torch.nn.functional.avg_pool2d(x, s, ceil_mode=True)
            else:
                p = torch.nn.functional.avg_pool2d(x, (min(s, c["gh"]), min(s, c["gw"])), stride=s)
            tokens.append(p[0].permute(1, 2, 0).reshape(-1, d))
    return sim, score, torch.tensor(event_score, dtype=torch.float64, device=feats.device), torch.cat(tokens)


def _exact_scores(c, q, keys, weight, event):
    Hq, Tq, dh = q.shape
    v0, n_vis, S = c["vis_start"], c["n_vis"], keys.shape[1]
    total = torch.zeros(n_vis, dtype=torch.float64, device=q.device)
    pos = torch.arange(S, device=q.device)
    for h in range(Hq):
        kh = keys[h // (Hq // keys.shape[0])].double()
        logits = (q[h].double() @ kh.t().contiguous()) / math.sqrt(dh)
        if c["mode"] == B.SCORE_VISUAL_ONLY:
            p = torch.softmax(logits[:, v0:v0 + n_vis], 1)
        else:
            limit = torch.arange(S - Tq, S, device=q.device)[:, None]
            p = torch.softmax(logits.masked_fill(pos[None] > limit, -math.inf), 1)[:, v0:v0 + n_vis]
        total += p.sum(0)
    return weight.double()[event.long()] * total / (Hq * Tq)


def exact(case, seed):
    c = case
    if c["kind"] == "cache" or (c["kind"] == "prune" and not c["attention"]):
        return None
    s = prepare(c, seed)
    one = c["batch"] == 1
    if c["kind"] == "frames":
        if c["batch"] * c["T"] > 4000:
            return None
        got = [_exact_video(c, f, t) for f, t in ([(s["feats"], s["text"])] if one else zip(s["feats"], s["text"]))]
        pooled = torch.zeros(s["out"]["out_tokens"].shape, dtype=torch.float64, device=DEV).view(c["batch"], -1, c["d"])
        for b, v in enumerate(got):
            pooled[b, :v[3].shape[0]] = v[3]
        res = dict(sim=[v[0] for v in got], frame_score=[v[1] for v in got], event_score=[v[2] for v in got])
        res = {name: x[0] if one else torch.stack(x) for name, x in res.items()}
        res["out_tokens"] = pooled[0] if one else pooled
        none = ("event_start", "frame_event", "frame_offsets", "token_event", "event_is_key", "frame_is_key", "frame_stride")
        return {**res, **{name: None for name in none}}
    names = ("q", "keys", "weight", "token_event")
    per_video = [tuple(s[n] for n in names)] if one else list(zip(*(s[n] for n in names)))
    scores = [_exact_scores(c, *v) for v in per_video]
    return {"scores": scores[0] if one else torch.stack(scores)}
