"""The workloads this library's speed is judged on, each run through the public
entry points as a user's program calls them.

Inputs are synthetic, made on the GPU from a seed, in the shapes of the paper's
workloads: 25 audio tokens and two 144-token frames per second, the 3B thinker's
heads (16 query / 2 key, hidden 2048) and the 7B thinker's (28 / 4, hidden 3584),
head dim 128.  Planted structure keeps the method's discrete decisions away from
their boundaries, as in real scenes: top sets with lifted keys for the prune, and
scenes with shared or offset audio and visual drift for the scorer.
"""

import math

import torch

import paper_2608_08794_amd as A

AUDIO, VISUAL = A.APACK_AUDIO, A.APACK_VISUAL
LAYERS = 28            # decoder layers whose K/V the long-clip workloads compact
PROGRESSIVE = ((14, 0.7), (18, 0.5), (22, 0.3))   # prune layer, cumulative keep
FIRST_LAYER, DROP = 14, 0.10                      # the paper's every-layer schedule


# ---------------------------------------------------------------------------
# The cases
# ---------------------------------------------------------------------------

def _prune(name, dtype, hq, hkv, d, hidden, audio, visual, text, q_len, keep_a, keep_v, joint=False, layers=1):
    return dict(name=name, kind="prune", dtype=dtype, hq=hq, hkv=hkv, d=d, hidden=hidden, audio=audio, visual=visual,
                text=text, q_len=q_len, keep_a=keep_a, keep_v=keep_v, joint=joint, layers=layers)


def _scorer(name, dtype, dim, frames, per_frame, audio, query, window, alignment, structure):
    return dict(name=name, kind="scorer", dtype=dtype, dim=dim, frames=frames, per_frame=per_frame, audio=audio,
                query=query, window=window, alignment=alignment, structure=structure)


def listed():
    return [
        # A very short fp32 context (a test model, a few seconds of audio): the call's latency.
        _prune("prune_tiny_f32", "f32", 8, 2, 64, 512, 256, 1024, 32, 32, 0.5, 0.5),
        # One prune of a 30 s clip at the 3B shape, one layer compacted.
        _prune("prune_3b_30s", "bf16", 16, 2, 128, 2048, 750, 60 * 144, 64, 64, 0.6, 0.4),
        # One prune of a 60 s clip at the 7B shape after the pre-LLM stage, one layer compacted.
        _prune("prune_7b_60s", "bf16", 28, 4, 128, 3584, 1500, 7890, 64, 64, 0.5, 0.3),
        # The 3B layer with fp32 tensors: evaluation and parity runs in full precision.
        _prune("prune_3b_30s_f32", "f32", 16, 2, 128, 2048, 750, 60 * 144, 64, 64, 0.6, 0.4),
        # A 5-minute clip at the 7B shape: three progressive prunes, each compacting all layers (bench.py's step).
        dict(name="progressive_7b_5min", kind="progressive", hq=28, hkv=4, d=128, hidden=3584, audio=7500,
             visual=600 * 144, text=128, q_len=128),
        # The paper's schedule on the same clip: last query row, joint ranking, 10% dropped at each of 14 layers.
        dict(name="schedule_7b_5min", kind="schedule", hq=28, hkv=4, d=128, hidden=3584, audio=7500,
             visual=600 * 144, text=128, steps=14),
        # Compaction in place of a 28-layer cache, for callers that cannot hold it twice.
        dict(name="inplace_7b_5min", kind="inplace", hkv=4, d=128, hidden=3584, rows=94028, layers=28, keep=0.5),
        # Pre-LLM scorer of a 20 s clip at the 3B width, gate off: the shortest clips.
        _scorer("scorer_3b_20s", "bf16", 2048, 40, 144, 500, 32, 3, "gated_cka", "shared"),
        # Pre-LLM scorer of a 60 s clip at the 7B width, gate fired (the direct distance runs).
        _scorer("scorer_7b_60s_gated", "bf16", 3584, 120, 144, 1500, 64, 4, "gated_cka", "offset"),
        # The spatial-CKA alignment scorer on the same clip.
        _scorer("scorer_7b_60s_spatial", "bf16", 3584, 120, 144, 1500, 64, 4, "spatial_cka", "shared"),
        # fp32 embeddings, gate fired.
        _scorer("scorer_3b_60s_f32", "f32", 2048, 120, 144, 1500, 64, 3, "gated_cka", "offset"),
        # A ragged batch of eight clips: scorer, embedding gather, prune and compaction in one sequence.
        dict(name="ragged_7b_8clips", kind="ragged", hq=28, hkv=4, d=128, hidden=3584,
             seconds="224,284,267,163,284,294,292,42", queries="52,79,89,36,117,64,98,127"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["prune", "prune", "prune", "scorer", "scorer", "scorer", "ragged", "inplace", "schedule",
                       "progressive"])
    hq, hkv, hidden = rng.choice([(16, 2, 2048), (28, 4, 3584)])
    if kind == "prune":
        dtype = rng.choice(["bf16", "bf16", "f32"])
        d = rng.choice([128, 128, 64])
        sec = _log(rng, 3, 300 if dtype == "bf16" else 60)
        joint = rng.random() < 0.3
        case = _prune("", dtype, hq, hkv, d, hidden, 25 * sec + rng.randrange(25), 144 * sec + rng.randrange(288),
                      rng.randint(1, 160), 1 if joint else _log(rng, 1, 128), round(rng.uniform(0.2, 0.9), 2),
                      0.0 if joint else round(rng.uniform(0.2, 0.9), 2), joint,
                      rng.choice([1, 1, 28]) if dtype == "bf16" else 1)
    elif kind == "scorer":
        dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
        sec = _log(rng, 4, 150 if dtype == "bf16" else 60)
        case = _scorer("", dtype, rng.choice([2048, 3584, 3584, 1288]), 2 * sec + rng.randrange(2),
                       rng.choice([144, 144, 100, 64, 196]), 25 * sec + rng.randrange(25), rng.randint(1, 128),
                       rng.choice([3, 3, 4, 8]), rng.choice(["gated_cka", "gated_cka", "cka", "av_cosine",
                                                            "spatial_cka"]), rng.choice(["shared", "offset"]))
    elif kind == "ragged":
        n = rng.randint(2, 8)
        case = dict(name="", kind="ragged", hq=hq, hkv=hkv, d=128, hidden=hidden,
                    seconds=",".join(str(rng.randint(10, 160)) for _ in range(n)),
                    queries=",".join(str(rng.randint(8, 128)) for _ in range(n)))
    elif kind == "inplace":
        case = dict(name="", kind="inplace", hkv=hkv, d=128, hidden=hidden, rows=_log(rng, 3000, 94028),
                    layers=rng.choice([1, 28, 36]), keep=round(rng.uniform(0.3, 0.95), 2))
    else:
        sec = _log(rng, 20, 280)
        case = dict(name="", kind=kind, hq=hq, hkv=hkv, d=128, hidden=hidden, audio=25 * sec + rng.randrange(25),
                    visual=288 * sec + rng.randrange(144), text=rng.randint(1, 160))
        if kind == "schedule":
            case["steps"] = rng.randint(2, 14)
        else:
            case["q_len"] = _log(rng, 8, 128)
    del case["name"]
    return case


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _normal(g, *shape):
    return torch.randn(*shape, generator=g, device="cuda")


def _unit(g, *shape):
    x = _normal(g, *shape)
    return x.div_(x.norm(dim=-1, keepdim=True))


def _payload(g, dtype, *shape):
    """Values that are only moved: random finite bits."""
    if dtype == "f32":
        return _normal(g, *shape)
    t = torch.randint(-32768, 32768, shape, generator=g, device="cuda", dtype=torch.int16)
    return t.bitwise_and_(~0x4000).view(torch.bfloat16)


def _dt(dtype):
    return torch.bfloat16 if dtype == "bf16" else torch.float32


def _choose(g, rows, k):
    """k of `rows`, ascending."""
    return rows[torch.randperm(rows.numel(), generator=g, device="cuda")[:k]].sort().values


def _query(g, dtype, hq, hkv, q_len, d):
    """Q of one prune and the direction each key group's planted keys are lifted along."""
    if dtype == "f32":
        dirs = _unit(g, hkv, d)
        q = _normal(g, hq, q_len, d) + 3.0 * dirs.repeat_interleave(hq // hkv, 0)[:, None]
        return q, dirs
    q = (_normal(g, hq, q_len, d) / math.sqrt(d)).to(torch.bfloat16)
    m = q.float().view(hkv, -1, d).mean(1)
    return q, m / m.norm(dim=-1, keepdim=True)


def _keys(g, dtype, hkv, n, d, dirs, top, high=None):
    """K of one prune layer: noise, the planted top set lifted, a few rows lifted far more."""
    k = _normal(g, hkv, n, d)
    if dtype == "f32":
        k[:, top] += math.sqrt(d) * dirs[:, None]
        return k
    k /= math.sqrt(d)
    k[:, top] += 12.0 * dirs[:, None]
    if high is not None:
        k[:, high] += 60.0 * dirs[:, None]
    return k.to(torch.bfloat16)


def _positions(n):
    t = torch.arange(n, dtype=torch.int32, device="cuda")
    return torch.stack([t, (t * 7) % 1013, (t * 13) % 2039])


def _keep_count(keep, n):
    return A.apack_keep_count(keep, n)


def _cache_of(kv, hidden, pos):
    """A cache as a decoder holds it: a K and a V tensor per layer (views of kv, [layers][2][hkv][rows][d]), the hidden
    states and the position ids."""
    return dict(kv=kv, k=list(kv[:, 0]), v=list(kv[:, 1]), hidden=hidden, pos=pos, rows=hidden.shape[0])


def _cache(g, dtype, layers, hkv, n, d, hidden):
    return _cache_of(_payload(g, dtype, layers, 2, hkv, n, d), _payload(g, dtype, n, hidden), _positions(n))


def _cache_like(c, n):
    kv, hid = c["kv"], c["hidden"]
    return _cache_of(torch.zeros((*kv.shape[:3], n, kv.shape[4]), dtype=kv.dtype, device="cuda"),
                     torch.zeros((n, hid.shape[1]), dtype=hid.dtype, device="cuda"),
                     torch.zeros((3, n), dtype=torch.int32, device="cuda"))


def _first_rows(c, n):
    return _cache_of(c["kv"][:, :, :, :n], c["hidden"][:n], c["pos"][:, :n])


def _step_buffers(seq, hq, hkv, d, rows):
    n_kept, ws = A.apack_prune_layer_query([seq] if isinstance(seq, dict) else seq, hq, hkv, d)
    return dict(n_out=sum(n_kept), ws=torch.empty(ws, dtype=torch.uint8, device="cuda"),
                scores=torch.zeros(rows, dtype=torch.float32, device="cuda"),
                kept=torch.zeros(sum(n_kept), dtype=torch.int32, device="cuda"))


def _seq(n, spans, q_len, keep, basis=(0, 0), joint=False, tok_off=0, q_off=0):
    return dict(tok_off=tok_off, n_tokens=n, spans=spans, q_off=q_off, q_len=q_len, keep=keep, keep_basis=basis,
                joint=joint)


def _top_sets(g, spans, keep, joint):
    """The planted top set of one prune: ceil(keep * n) rows of each modality, or of both together."""
    rows = {m: torch.cat([torch.arange(b, b + n, device="cuda") for b, n, t in spans if t == m]) for m in (AUDIO, VISUAL)}
    if joint:
        every = torch.cat([rows[AUDIO], rows[VISUAL]]).sort().values
        return every, _choose(g, every, _keep_count(keep[0], every.numel()))
    return torch.cat([rows[AUDIO], rows[VISUAL]]), torch.cat(
        [_choose(g, rows[m], _keep_count(keep[i], rows[m].numel())) for i, m in enumerate((AUDIO, VISUAL))])


def _prepare_prune(c, g):
    n = c["audio"] + c["visual"] + c["text"]
    spans = [(0, c["audio"], AUDIO), (c["audio"], c["visual"], VISUAL)]
    keep = (c["keep_a"], c["keep_v"])
    seq = _seq(n, spans, c["q_len"], keep, joint=c["joint"])
    q, dirs = _query(g, c["dtype"], c["hq"], c["hkv"], c["q_len"], c["d"])
    every, top = _top_sets(g, spans, keep, c["joint"])
    cache = _cache(g, c["dtype"], c["layers"], c["hkv"], n, c["d"], c["hidden"])
    # Layer 0 is the prune layer.
    cache["k"][0][:] = _keys(g, c["dtype"], c["hkv"], n, c["d"], dirs, top, _choose(g, every, every.numel() // 20))
    b = _step_buffers(seq, c["hq"], c["hkv"], c["d"], n)
    return dict(kind="prune", seqs=[seq], q=q, cache=cache, out=_cache_like(cache, b["n_out"]), buf=b)


def _chain(c):
    """(prune layer, spans, keep, basis, joint, rows in) of every step of a progressive run."""
    a, v, text = c["audio"], c["visual"], c["text"]
    steps = []
    if c["kind"] == "progressive":
        ka, kv = a, v
        for layer, keep in PROGRESSIVE:
            steps.append((layer, _seq(ka + kv + text, [(0, ka, AUDIO), (ka, kv, VISUAL)], c["q_len"], (keep, keep),
                                      (a, v))))
            ka, kv = _keep_count(keep, a), _keep_count(keep, v)
    else:
        n = a + v
        for i in range(c["steps"]):
            steps.append((FIRST_LAYER + i, _seq(n + text, [(0, n, AUDIO)], 1, (1.0 - DROP, 0.0), joint=True)))
            n = _keep_count(1.0 - DROP, n)
    return steps


def _prepare_chain(c, g):
    steps = _chain(c)
    n = steps[0][1]["n_tokens"]
    hq, hkv, d = c["hq"], c["hkv"], c["d"]
    cache = _cache(g, "bf16", LAYERS, hkv, n, d, c["hidden"])
    # Nested planted sets, in the first step's rows: each prune layer's top set lies inside the one before it.
    parts = [torch.arange(b, b + m, device="cuda") for b, m, _ in steps[0][1]["spans"]]
    todo = []
    for layer, seq in steps:
        q, dirs = _query(g, "bf16", hq, hkv, seq["q_len"], d)
        parts = [_choose(g, p, _keep_count(seq["keep"][i], seq["keep_basis"][i] or p.numel()))
                 for i, p in enumerate(parts)]
        cache["k"][layer][:] = _keys(g, "bf16", hkv, n, d, dirs, torch.cat(parts))
        todo.append(dict(layer=layer, seq=seq, q=q, **_step_buffers(seq, hq, hkv, d, seq["n_tokens"])))
    # A progressive run keeps each step's cache; the every-layer schedule ping-pongs between two.
    if c["kind"] == "progressive":
        outs = [_cache_like(cache, s["n_out"]) for s in todo]
    else:
        pair = [_cache_like(cache, s["n_out"]) for s in todo[:2]]
        outs = [_first_rows(pair[i % 2], s["n_out"]) for i, s in enumerate(todo)]
    return dict(kind="chain", steps=todo, cache=cache, outs=outs)


def _prepare_inplace(c, g):
    cache = _cache(g, "bf16", c["layers"], c["hkv"], c["rows"], c["d"], c["hidden"])
    kept = _choose(g, torch.arange(c["rows"], device="cuda"), _keep_count(c["keep"], c["rows"])).int()
    ws = torch.empty(A.apack_compact_kv_inplace_workspace(kept.numel()), dtype=torch.uint8, device="cuda")
    return dict(kind="inplace", kept=kept, cache=cache, ws=ws)


def _clip(g, dtype, frames, per_frame, n_audio, n_query, dim, structure):
    """Embeddings of one clip of planted scenes of 8 to 24 frames.  Visual tokens cluster into eight objects a scene.
    shared: audio and visual drift together (the window CKA is high); offset: the audio swings while the visual drift
    is a trend (it is low, and the gate fires)."""
    lens, left = [], frames
    for x in torch.randint(8, 25, (frames // 8 + 1,), generator=g, device="cuda").tolist():
        x = left if left < 16 else min(x, left - 8)
        lens.append(x)
        left -= x
        if left <= 0:
            break
    s = len(lens)
    scene, objects, detail = _unit(g, s, dim), _unit(g, s, 8, dim), _unit(g, s, per_frame, dim)
    vdir, adir, sound = _unit(g, s, dim), _unit(g, s, dim), _unit(g, s, dim)
    cluster = torch.randint(0, 8, (s, per_frame), generator=g, device="cuda")
    lens_t = torch.tensor(lens, device="cuda")
    of = torch.arange(s, device="cuda").repeat_interleave(lens_t)
    at = torch.cat([torch.arange(x, device="cuda") for x in lens]).float()
    walk = _normal(g, frames) * 0.10
    if structure == "shared":
        parts = [w.cumsum(0) for w in walk.split(lens)]
        drift_v = torch.cat([w - w.mean() for w in parts])
        drift_a = drift_v
    else:
        drift_v = (at - (lens_t[of].float() - 1) / 2) * 0.10
        drift_a = torch.where(at % 2 == 0, -0.3, 0.3)
    xv = torch.empty((frames, per_frame, dim), dtype=_dt(dtype), device="cuda")
    for f0 in range(0, frames, 64):
        m = of[f0:f0 + 64]
        x = _unit(g, m.numel(), per_frame, dim) * 0.3
        x += 0.6 * scene[m][:, None] + 0.2 * detail[m] + (drift_v[f0:f0 + 64, None] * vdir[m])[:, None]
        x += objects[m[:, None], cluster[m]]
        xv[f0:f0 + 64] = x.to(xv.dtype)
    af = (torch.arange(n_audio, device="cuda") * frames) // n_audio
    xa = 0.5 * scene[of[af]] + sound[of[af]] + drift_a[af, None] * adir[of[af]] + 0.3 * _unit(g, n_audio, dim)
    picks = torch.randperm(s, generator=g, device="cuda")[:2]
    cue = scene[picks].sum(0) + objects[picks[0], 0]
    xq = cue[None] + 0.8 * _unit(g, n_query, dim)
    return xv.view(frames * per_frame, dim), xa.to(_dt(dtype)), xq.to(_dt(dtype))


def _scorer_state(clips, xv, xa, xq, params):
    n_kept, ws = A.apack_score_dynamics_query(clips, xv.shape[1], params)
    return dict(clips=clips, xv=xv, xa=xa, xq=xq, params=params,
                ws=torch.empty(ws, dtype=torch.uint8, device="cuda"),
                emb=torch.zeros((sum(n_kept), xv.shape[1]), dtype=xv.dtype, device="cuda"))


def _prepare_scorer(c, g):
    xv, xa, xq = _clip(g, c["dtype"], c["frames"], c["per_frame"], c["audio"], c["query"], c["dim"], c["structure"])
    clip = dict(n_frames=c["frames"], per_frame=c["per_frame"], n_audio=c["audio"], n_query=c["query"], vis_off=0,
                aud_off=0, qry_off=0)
    params = dict(window=c["window"], r_pre=0.5, alignment=c["alignment"])
    return dict(kind="scorer", scorer=_scorer_state([clip], xv, xa, xq, params))


def _ragged_layout(c):
    """Clips of the scorer and sequences of the prune: 2-second chunks of [visual | audio], then the text span."""
    secs, texts = [int(x) for x in c["seconds"].split(",")], [int(x) for x in c["queries"].split(",")]
    clips, seqs = [], []
    vo = ao = qo = tok = 0
    for t, nq in zip(secs, texts):
        f, na = 2 * t, 25 * t
        clips.append(dict(n_frames=f, per_frame=144, n_audio=na, n_query=nq, vis_off=vo, aud_off=ao, qry_off=qo))
        vis = A.apack_visual_budget(0.5, na, f * 144)
        chunks, spans, row = max(1, t // 2), [], 0
        for i in range(chunks):
            for total, m in ((vis, VISUAL), (na, AUDIO)):
                x = total // chunks + (1 if i < total % chunks else 0)
                spans.append((row, x, m))
                row += x
        seqs.append(_seq(row + nq, spans, nq, (0.5, 0.3), tok_off=tok, q_off=qo))
        vo, ao, qo, tok = vo + f * 144, ao + na, qo + nq, tok + row + nq
    return clips, seqs, tok, qo


def _prepare_ragged(c, g):
    clips, seqs, rows, q_rows = _ragged_layout(c)
    hq, hkv, d, hidden = c["hq"], c["hkv"], c["d"], c["hidden"]
    parts = [_clip(g, "bf16", x["n_frames"], 144, x["n_audio"], x["n_query"], hidden, ("shared", "offset")[i % 2])
             for i, x in enumerate(clips)]
    xv, xa, xq = (torch.cat([p[j] for p in parts]) for j in range(3))
    del parts
    q = torch.empty((hq, q_rows, d), dtype=torch.bfloat16, device="cuda")
    cache = _cache(g, "bf16", 1, hkv, rows, d, hidden)
    for s in seqs:
        qs, dirs = _query(g, "bf16", hq, hkv, s["q_len"], d)
        q[:, s["q_off"]:s["q_off"] + s["q_len"]] = qs
        _, top = _top_sets(g, s["spans"], s["keep"], False)
        cache["k"][0][:, s["tok_off"]:s["tok_off"] + s["n_tokens"]] = _keys(g, "bf16", hkv, s["n_tokens"], d, dirs, top)
    b = _step_buffers(seqs, hq, hkv, d, rows)
    return dict(kind="ragged", scorer=_scorer_state(clips, xv, xa, xq, dict(window=3, r_pre=0.5)),
                prune=dict(seqs=seqs, q=q, cache=cache, out=_cache_like(cache, b["n_out"]), buf=b))


def prepare(case, seed):
    g = _gen(seed)
    make = dict(prune=_prepare_prune, progressive=_prepare_chain, schedule=_prepare_chain, inplace=_prepare_inplace,
                scorer=_prepare_scorer, ragged=_prepare_ragged)
    return make[case["kind"]](case, g)


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------

def _compact(kept, a, b):
    A.apack_compact_kv(kept, a["rows"], a["k"], a["v"], b["k"], b["v"], a["hidden"], b["hidden"], a["pos"], b["pos"])


def _run_prune(s):
    a, out, b = s["cache"], s["out"], s["buf"]
    scores, kept, _ = A.apack_prune_layer(s["q"], a["k"][0], s["seqs"], scores=b["scores"], kept_rows=b["kept"],
                                          workspace=b["ws"])
    _compact(kept, a, out)
    return dict(scores=scores, kept=kept, kv=out["kv"], hidden=out["hidden"], pos=out["pos"])


def _run_chain(s):
    cache, got = s["cache"], {}
    for i, (st, out) in enumerate(zip(s["steps"], s["outs"])):
        scores, kept, _ = A.apack_prune_layer(st["q"], cache["k"][st["layer"]], [st["seq"]], scores=st["scores"],
                                              kept_rows=st["kept"], workspace=st["ws"])
        _compact(kept, cache, out)
        cache = out
        got["scores%d" % i], got["kept%d" % i] = scores, kept
    return dict(got, kv=cache["kv"], hidden=cache["hidden"], pos=cache["pos"])


def _run_scorer(s):
    out = A.apack_score_dynamics(s["xv"], s["xa"], s["xq"], s["clips"], s["params"], workspace=s["ws"])
    A.apack_compact_kv(out["kept"], s["xv"].shape[0], hidden_in=s["xv"], hidden_out=s["emb"])
    return dict(cka=out["cka"], score=out["score"], budget=out["budget"], segment=out["segment"], gate=out["gate"],
                kept=out["kept"], emb=s["emb"])


def run(s):
    if s["kind"] == "prune":
        return _run_prune(s)
    if s["kind"] == "chain":
        return _run_chain(s)
    if s["kind"] == "scorer":
        return _run_scorer(s["scorer"])
    if s["kind"] == "ragged":
        return dict(scorer=_run_scorer(s["scorer"]), prune=_run_prune(s["prune"]))
    c = s["cache"]
    A.apack_compact_kv_inplace(s["kept"], c["rows"], c["k"], c["v"], c["hidden"], c["pos"], workspace=s["ws"])
    return dict(kv=c["kv"], hidden=c["hidden"], pos=c["pos"])


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------

def _prune_work(seqs, hq, hkv, d, e, layers, hidden):
    """Logits of every query row against every candidate; K over the candidates, Q, the scores and the kept rows; one
    read and one write of every kept row of the planes."""
    nbytes = flops = 0
    row = layers * 2 * hkv * d * e + hidden * e + 3 * 4
    n_kept, _ = A.apack_prune_layer_query(seqs, hq, hkv, d)
    for s, k in zip(seqs, n_kept):
        cand = sum(n for _, n, _ in s["spans"])
        flops += 2.0 * cand * s["q_len"] * hq * d
        nbytes += cand * hkv * d * e + hq * s["q_len"] * d * e + 4 * s["n_tokens"] + k * (2 * row + 4)
    return nbytes, flops


def _scorer_work(clips, dim, e, gated):
    """X_V, X_A and X_Q once, the kept embeddings written; the audio-visual products of the clips whose gate fires."""
    nbytes = flops = 0
    for c, g in zip(clips, gated):
        nv = c["n_frames"] * c["per_frame"]
        b = A.apack_visual_budget(0.5, c["n_audio"], nv)
        nbytes += (nv + c["n_audio"] + c["n_query"] + b) * dim * e + 4 * b
        flops += 2.0 * nv * c["n_audio"] * dim if g else 4.0 * nv * dim
    return nbytes, flops


def work(c):
    if c["kind"] == "prune":
        spans = [(0, c["audio"], AUDIO), (c["audio"], c["visual"], VISUAL)]
        seq = _seq(c["audio"] + c["visual"] + c["text"], spans, c["q_len"], (c["keep_a"], c["keep_v"]),
                   joint=c["joint"])
        w = _prune_work([seq], c["hq"], c["hkv"], c["d"], 2 if c["dtype"] == "bf16" else 4, c["layers"], c["hidden"])
    elif c["kind"] in ("progressive", "schedule"):
        w = [sum(x) for x in zip(*(_prune_work([s], c["hq"], c["hkv"], c["d"], 2, LAYERS, c["hidden"])
                                   for _, s in _chain(c)))]
    elif c["kind"] == "inplace":
        row = c["layers"] * 2 * c["hkv"] * c["d"] * 2 + c["hidden"] * 2 + 12
        w = (_keep_count(c["keep"], c["rows"]) * (2 * row + 4), 0)
    elif c["kind"] == "scorer":
        clip = dict(n_frames=c["frames"], per_frame=c["per_frame"], n_audio=c["audio"], n_query=c["query"])
        # The covariances of a frame's unrelated patches and sounds match little, so the spatial scorer's gate fires.
        gated = c["alignment"] in ("av_cosine", "spatial_cka") or (c["alignment"] == "gated_cka" and
                                                                   c["structure"] == "offset")
        w = _scorer_work([clip], c["dim"], 2 if c["dtype"] == "bf16" else 4, [gated])
        if c["alignment"] == "spatial_cka":   # the frames' Grams, each entry once
            m = c["per_frame"] + c["audio"] / c["frames"]
            w = (w[0], w[1] + c["frames"] * m * (m + 1) * c["dim"])
    else:
        clips, seqs, _, _ = _ragged_layout(c)
        a = _scorer_work(clips, c["hidden"], 2, [i % 2 == 1 for i in range(len(clips))])
        b = _prune_work(seqs, c["hq"], c["hkv"], c["d"], 2, 1, c["hidden"])
        w = (a[0] + b[0], a[1] + b[1])
    return {"bytes": float(w[0]), "flops": float(w[1])}


def tolerance(c):
    if c["kind"] == "inplace":
        return "exact"
    # Scores and frame scores are 32-bit results of 32-bit sums (fp64 in the scorer but for the gate's products).  Kept
    # rows follow decisions that lie away from ties; a frame budget downstream of the gate's 32-bit products may move
    # by a unit between two frames.
    return {"rel": 1e-5, "max": 1e-4, "differ": 0.01}


# ---------------------------------------------------------------------------
# The same in 64 bits
# ---------------------------------------------------------------------------

def _exact_prune(q, k, seqs):
    """(scores, kept rows) of a packed batch in fp64."""
    hq, _, d = q.shape
    rep = hq // k.shape[0]
    scores = torch.zeros(k.shape[1], dtype=torch.float64, device="cuda")
    kept = []
    for s in seqs:
        lo, n = s["tok_off"], s["n_tokens"]
        tag = torch.zeros(n, dtype=torch.int32, device="cuda")
        for b, m, t in s["spans"]:
            tag[b:b + m] = 1 if s["joint"] else t
        cand = tag.nonzero().view(-1)
        acc = torch.zeros(cand.numel(), dtype=torch.float64, device="cuda")
        for h in range(hq):
            kh = k[h // rep, lo:lo + n][cand].double()
            x = q[h, s["q_off"]:s["q_off"] + s["q_len"]].double() @ kh.t() / math.sqrt(d)
            acc += torch.softmax(x, dim=1).sum(0)
        sc = torch.zeros(n, dtype=torch.float64, device="cuda")
        sc[cand] = acc / (hq * s["q_len"])
        scores[lo:lo + n] = sc
        keep = tag == 0
        for m in (1, 2):
            rows = (tag == m).nonzero().view(-1)
            kk = _keep_count(s["keep"][m - 1], s["keep_basis"][m - 1] or rows.numel())
            order = torch.sort(-sc[rows].float(), stable=True).indices
            keep[rows[order[:kk]]] = True
        kept.append(lo + keep.nonzero().view(-1))
    return scores, torch.cat(kept).int()


def _exact_scorer(s):
    """c_f and s_f of every frame in fp64, clip after clip."""
    cka, score = [], []
    p = dict(tau=0.78, beta=0.90, gamma=0.9, tau_sim=0.97, sigma=1.0, lam=0.5)
    align = s["params"].get("alignment", "gated_cka")
    for c in s["clips"]:
        F, P, na = c["n_frames"], c["per_frame"], c["n_audio"]
        xv = s["xv"][c["vis_off"]:c["vis_off"] + F * P].view(F, P, -1)
        xa = s["xa"][c["aud_off"]:c["aud_off"] + na].double()
        qbar = s["xq"][c["qry_off"]:c["qry_off"] + c["n_query"]].double().mean(0)
        v = torch.stack([x.double().mean(0) for x in xv])
        bins = [(f * na // F, -(-(f + 1) * na // F)) for f in range(F)]
        a = torch.stack([xa[l:h].mean(0) for l, h in bins])

        def centred(x):
            return x - x.mean(0)

        def degenerate(x, gram):
            return bool(gram.norm() <= 1e-8 * (x * x).sum())

        cf = torch.zeros(F, dtype=torch.float64, device="cuda")
        w = s["params"]["window"]
        for f in range(F):
            if align == "spatial_cka":
                x, y = xa[bins[f][0]:bins[f][1]], xv[f].double()
                cx, cy = centred(x), centred(y)
                ka, kv, num = cx @ cx.t(), cy @ cy.t(), (cx @ cy.t()).square().sum()
            else:
                lo, hi = (0, F) if F <= w else (min(max(f - w // 2, 0), F - w), min(max(f - w // 2, 0), F - w) + w)
                x, y = a[lo:hi], v[lo:hi]
                cx, cy = centred(x), centred(y)
                ka, kv = cx @ cx.t(), cy @ cy.t()
                num = (ka * kv).sum()
            if not degenerate(x, ka) and not degenerate(y, kv):
                cf[f] = num / (ka.norm() * kv.norm())
        fired = align == "av_cosine" or (align != "cka" and float(cf.mean()) < p["tau"])
        alpha = cf
        if fired:
            ua = xa / xa.norm(dim=1, keepdim=True)
            d = torch.empty(F, dtype=torch.float64, device="cuda")
            for f in range(F):
                x = xv[f].double()
                d[f] = 1 - ((x / x.norm(dim=1, keepdim=True)) @ ua.t()).max(1).values.mean()
            dh = (d - d.min()) / (d.max() - d.min()) if d.max() > d.min() else d * 0
            beta = 1.0 if align == "av_cosine" else p["beta"]
            alpha = (1 - beta) * cf + beta * (1 - dh)
        # Continuity, its smoothing, and one cut at the minimum of each run below the threshold.
        n2 = (v * v).sum(1)
        cs = ((v[:-1] * v[1:]).sum(1) / (n2[:-1] * n2[1:]).sqrt()).tolist()
        offs = range(-4, 5)
        wt = [math.exp(-0.5 * o * o / p["sigma"] ** 2) for o in offs]
        n = F - 1
        sm = []
        for i in range(n):
            acc = 0.0
            for o, x in zip(offs, wt):
                j = (i + o) % (2 * n)
                acc += x / sum(wt) * cs[j if j < n else 2 * n - 1 - j]
            sm.append(acc)
        starts, f = [0], 0
        while f < n:
            if sm[f] < p["tau_sim"]:
                e = f
                while e + 1 < n and sm[e + 1] < p["tau_sim"]:
                    e += 1
                starts.append(min(range(f, e + 1), key=lambda i: (sm[i], i)) + 1)
                f = e
            f += 1
        r = (1 + (v @ qbar) / (n2 * (qbar * qbar).sum()).sqrt()) / 2
        ends = starts[1:] + [F]
        gm = torch.stack([math.sqrt(e - b) * (p["lam"] * r[b:e].max() + (1 - p["lam"]) * r[b:e].mean())
                          for b, e in zip(starts, ends)])
        u = (gm / gm.max()).repeat_interleave(torch.tensor([e - b for b, e in zip(starts, ends)], device="cuda"))
        cka.append(cf)
        score.append(p["gamma"] * u + (1 - p["gamma"]) * alpha)
    return dict(cka=torch.cat(cka), score=torch.cat(score), budget=None, segment=None, gate=None, kept=None, emb=None)


def exact(case, seed):
    if case["kind"] == "inplace":
        return None
    s = prepare(case, seed)
    none = dict(kv=None, hidden=None, pos=None)
    if s["kind"] == "prune":
        scores, kept = _exact_prune(s["q"], s["cache"]["k"][0], s["seqs"])
        return dict(scores=scores, kept=kept, **none)
    if s["kind"] == "chain":
        got, rows = {}, torch.arange(s["cache"]["rows"], device="cuda")
        for i, st in enumerate(s["steps"]):
            scores, kept = _exact_prune(st["q"], s["cache"]["k"][st["layer"]][:, rows], [st["seq"]])
            rows = rows[kept.long()]
            got["scores%d" % i], got["kept%d" % i] = scores, kept
        return dict(got, **none)
    if s["kind"] == "scorer":
        return _exact_scorer(s["scorer"])
    pr = s["prune"]
    scores, kept = _exact_prune(pr["q"], pr["cache"]["k"][0], pr["seqs"])
    return dict(scorer=_exact_scorer(s["scorer"]), prune=dict(scores=scores, kept=kept, **none))
