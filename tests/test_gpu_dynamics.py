"""GPU parity of the pre-LLM scorer (Section 3.1, Eq. 1-4; Algorithm 1)
against the fp64 oracle, through the C ABI.

Discrete outputs (gate, segment ids, frame budgets, kept visual rows) must
be bit-exact; frame CKA and frame scores are fp32 casts of fp64 values and
must agree to fp32 resolution (1e-5 relative where the fp32 gate GEMM feeds
them).  Each case first certifies with the oracle that every decision sits
away from its boundary (1e-9 for fp64 decisions, 1e-4 downstream of the
fp32 gate GEMM).
"""

import numpy as np
import pytest

import workloads as W
from oracle import dynamics as OD, widen
from tests.gpu_util import THREE_PART_RMS, log, rms, three_part_rows, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2608_08794_amd as A
    A.library()


def _oracle(case, dtype="bf16"):
    out = []
    for s in case.seqs:
        xv = widen(case.xv, dtype)[s.vis_off:s.vis_off + s.n_frames * s.per_frame]
        xa = widen(case.xa, dtype)[s.aud_off:s.aud_off + s.n_audio]
        xq = widen(case.xq, dtype)[s.qry_off:s.qry_off + s.n_query]
        out.append(OD.score_sequence(xv, xa, xq, s.n_frames, s.per_frame, case.params))
    return out


def _certify(results):
    for r in results:
        m = r["margins"]
        assert m["cka_degenerate"] > 1.0, m
        assert m["gate"] > 1e-9 and m["segment"] > 1e-9 and m["segment_budget"] > 1e-9, m
        assert m["dafps"] > 1e-9 and m["dedup"] > 1e-9, m
        assert m["frame_budget"] > (1e-4 if r["gate"] else 1e-9), m


def _run(case, dtype="bf16"):
    import paper_2608_08794_amd as A
    xv, xa, xq = (to_dev(x, dtype) for x in (case.xv, case.xa, case.xq))
    out = A.apack_score_dynamics(xv, xa, xq, case.seqs, case.params)
    torch.cuda.synchronize()
    return {k: (v.cpu().numpy() if hasattr(v, "cpu") else v) for k, v in out.items()}


def _compare(case, got, want, dtype="bf16"):
    f0 = 0
    kept_all = []
    for i, (s, r) in enumerate(zip(case.seqs, want)):
        F = s.n_frames
        sl = slice(f0, f0 + F)
        assert bool(got["gate"][i]) == r["gate"], f"clip {i}: gate"
        np.testing.assert_array_equal(got["segment"][sl], r["segment"], err_msg=f"clip {i}: segments")
        np.testing.assert_array_equal(got["budget"][sl], r["frame_budget"], err_msg=f"clip {i}: budgets")
        np.testing.assert_allclose(got["cka"][sl], r["cka"].astype(np.float32), rtol=1e-6, atol=1e-7)
        tol = 1e-5 if r["gate"] else 1e-6
        np.testing.assert_allclose(got["score"][sl], r["score"].astype(np.float32), rtol=tol, atol=1e-7)
        assert got["n_kept"][i] == r["kept"].size
        kept_all.append(r["kept"] + s.vis_off)
        f0 += F
    want_kept = np.concatenate(kept_all) if kept_all else np.zeros(0, np.int64)
    np.testing.assert_array_equal(got["kept"].astype(np.int64), want_kept)


@pytest.mark.parametrize("structure", ["shared", "offset"])
def test_small_clip_parity(structure):
    case = W.dynamics_small(structure)
    log(f"[dynamics] small {structure}")
    want = _oracle(case)
    _certify(want)
    _compare(case, _run(case), want)


@pytest.mark.parametrize("structure", ["shared", "offset"])
def test_small_clip_parity_fp32_inputs(structure):
    case = W.dynamics_small(structure)
    f32 = W.DynamicsCase("f32", case.dim, W.bf16_bits_to_f32(case.xv), W.bf16_bits_to_f32(case.xa),
                         W.bf16_bits_to_f32(case.xq), case.seqs, case.params)
    want = _oracle(f32, "f32")
    _certify(want)
    _compare(f32, _run(f32, "f32"), want, "f32")


@pytest.mark.parametrize("structure", ["shared", "offset"])
def test_7b_shape_60s_clip_parity(structure):
    case = W.dynamics_cfg3(structure)
    log(f"[dynamics] 60 s clip, 3584-d, {structure}")
    want = _oracle(case)
    _certify(want)
    _compare(case, _run(case), want)


def _packed(parts, params, gaps=None):
    """Clips packed one after another; with gaps = (before, between, after),
    rows that belong to no clip (large random values) sit before the first
    clip, between clips and after the last one in all three buffers."""
    rng = np.random.default_rng(99)
    xv, xa, xq, seqs = [], [], [], []
    vo = ao = qo = 0
    dim = parts[0].dim

    def gap(n):
        nonlocal vo, ao, qo
        if n:
            for buf in (xv, xa, xq):
                buf.append(W.to_bf16_bits(rng.uniform(-40.0, 40.0, size=(n, dim)).astype(np.float32)))
            vo, ao, qo = vo + n, ao + n, qo + n

    for i, c in enumerate(parts):
        if gaps:
            gap(gaps[0] if i == 0 else gaps[1])
        s = c.seqs[0]
        seqs.append(W.AVSeq(s.n_frames, s.per_frame, s.n_audio, s.n_query, vo, ao, qo, s.seg_starts, s.structure))
        xv.append(c.xv)
        xa.append(c.xa)
        xq.append(c.xq)
        vo += c.xv.shape[0]
        ao += c.xa.shape[0]
        qo += c.xq.shape[0]
    if gaps:
        gap(gaps[2])
    return W.DynamicsCase("bf16", dim, np.concatenate(xv), np.concatenate(xa), np.concatenate(xq), seqs, params)


def test_ragged_batch_of_clips_with_edge_shapes():
    parts = [
        W.dynamics_small("offset", seed=21, frames=30, per_frame=16, audio=375),
        W.dynamics_small("shared", seed=22, frames=2, per_frame=7, audio=25),      # F < w
        W.dynamics_small("shared", seed=23, frames=1, per_frame=5, audio=9),       # one frame
        W.dynamics_small("offset", seed=24, frames=20, per_frame=70, audio=250),   # P not a multiple of 64
        W.dynamics_small("shared", seed=25, frames=12, per_frame=256, audio=150),  # largest P
        W.dynamics_small("offset", seed=27, frames=8, per_frame=160, audio=80),    # DA-FPS rows past LDS
        W.dynamics_small("shared", seed=28, frames=7, per_frame=151, audio=70),    # odd P * P, rows past LDS
    ]
    case = _packed(parts, {"window": 3, "r_pre": 0.5})
    want = _oracle(case)
    _certify(want)
    _compare(case, _run(case), want)


def test_batch_of_more_clips_than_lanes():
    """70 short clips (one without frames): each one's outputs are those of the
    clip alone, to the bit (the Grams of a batch share one list of items)."""
    import paper_2608_08794_amd as A
    rng = np.random.default_rng(70)
    frames = [int(f) for f in rng.integers(1, 14, 70)]
    frames[33] = 0
    P, dim = 20, 72
    xv, xa, xq = (to_dev(W.to_bf16_bits(rng.standard_normal((n, dim)).astype(np.float32)), "bf16")
                  for n in (sum(frames) * P, 70 * 9, 70 * 2))
    params = {"window": 3, "r_pre": 0.5}
    clips, vo = [], 0
    for i, f in enumerate(frames):
        clips.append(dict(n_frames=f, per_frame=P, n_audio=9, n_query=2, vis_off=vo, aud_off=9 * i, qry_off=2 * i))
        vo += f * P
    batch = A.apack_score_dynamics(xv, xa, xq, clips, params)
    f0 = k0 = 0
    for i, clip in enumerate(clips):
        one = A.apack_score_dynamics(xv, xa, xq, [clip], params)
        f1, k1 = f0 + frames[i], k0 + one["n_kept"][0]
        assert batch["n_kept"][i] == one["n_kept"][0]
        for key in ("cka", "score", "budget", "segment"):
            assert torch.equal(batch[key][f0:f1], one[key]), (i, key)
        assert torch.equal(batch["kept"][k0:k1], one["kept"]), i
        f0, k0 = f1, k1


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("row", ["anchor", "other", "many"])
def test_tokens_that_are_not_finite_keep_within_their_budgets(row, value, dtype):
    """Cosines with them are NaN: every frame still keeps as many different
    tokens of its own as its budget says, finite ones first where the frame is
    not an anchor."""
    import paper_2608_08794_amd as A
    case = W.dynamics_small("shared", frames=20, per_frame=24, audio=100)
    s = case.seqs[0]
    clean = W.bf16_bits_to_f32(case.xv).reshape(20, 24, case.dim)
    frame = 0 if row == "anchor" else 7
    tokens = [5] if row != "many" else list(range(0, 24, 2))
    x = clean.copy()
    x[frame, tokens, 3] = value
    conv = (lambda a: W.to_bf16_bits(a)) if dtype == "bf16" else (lambda a: a)
    xv, xa, xq = (to_dev(conv(np.ascontiguousarray(a, np.float32)), dtype) for a in
                  (x.reshape(-1, case.dim), W.bf16_bits_to_f32(case.xa), W.bf16_bits_to_f32(case.xq)))
    out = A.apack_score_dynamics(xv, xa, xq, case.seqs, case.params)
    kept, budget = out["kept"].cpu().numpy(), out["budget"].cpu().numpy()
    seg = out["segment"].cpu().numpy()
    assert budget.min() >= 0 and budget.max() <= 24 and budget.sum() == kept.size == out["n_kept"][0]
    at = 0
    for f in range(20):
        mine = kept[at:at + budget[f]] - f * 24 - s.vis_off
        at += budget[f]
        assert (np.diff(mine) > 0).all() and (mine >= 0).all() and (mine < 24).all(), f
        if f == frame and f and seg[f] == seg[f - 1] and budget[f] <= 24 - len(tokens):
            assert not set(mine) & set(tokens)


def test_rows_outside_every_clip_are_ignored():
    """Buffers longer than the clips need: rows before, between and after
    the clips (in X_V, X_A and X_Q alike) change nothing, and the norms and
    max-cosine slots are sized by the clips' rows, not by the buffers'."""
    parts = [
        W.dynamics_small("offset", seed=51, frames=16, per_frame=12, audio=60),
        W.dynamics_small("shared", seed=52, frames=9, per_frame=20, audio=40),
    ]
    case = _packed(parts, {"window": 3, "r_pre": 0.5}, gaps=(5, 37, 300))
    want = _oracle(case)
    _certify(want)
    _compare(case, _run(case), want)


def test_long_clips_on_both_plan_paths():
    """The per-clip plan keeps its per-frame arrays in LDS up to 1023 frames
    and in global memory past that: one clip at the LDS limit, one past it
    (112 segments, the gate fired)."""
    parts = [
        W.dynamics_small("shared", seed=42, frames=1023, per_frame=3, audio=2046),
        W.dynamics_small("offset", seed=43, frames=1500, per_frame=8, audio=3000),
    ]
    case = _packed(parts, {"window": 3, "r_pre": 0.5})
    want = _oracle(case)
    _certify(want)
    _compare(case, _run(case), want)


@pytest.mark.parametrize("window", [1, 2, 5, 9, 16])
def test_window_sizes(window):
    """Every window bucket of the band and CKA kernels (up to the largest
    window, 16), on a 20-frame clip."""
    case = W.dynamics_small("offset", seed=61, frames=20, per_frame=16, audio=100, window=window)
    want = _oracle(case)
    _certify(want)
    _compare(case, _run(case), want)


@pytest.mark.parametrize("dafps_k", [1, 2, 3, 4, 6, 7, 8, 12, 32])
def test_dafps_density_list_lengths(dafps_k):
    """Every length of the DA-FPS density list (its mean over the dafps_k
    largest cosines), on 40-token frames, so that 32 < P - 1."""
    case = W.dynamics_small("offset", seed=81, frames=24, per_frame=40, audio=150)
    case.params = {"window": 3, "r_pre": 0.5, "dafps_k": dafps_k}
    want = _oracle(case)
    _certify(want)
    _compare(case, _run(case), want)


def test_dafps_list_longer_than_the_frame():
    """dafps_k = 32 on 16-token frames: the mean runs over the P - 1 others."""
    case = W.dynamics_small("offset", seed=81, frames=24, per_frame=16, audio=150)
    case.params = {"window": 3, "r_pre": 0.5, "dafps_k": 32}
    want = _oracle(case)
    _certify(want)
    _compare(case, _run(case), want)


@pytest.mark.parametrize("cover,power", [(0.5, 1.0), (0.95, 0.0), (0.8, 2.0)])
def test_dafps_cover_and_power(cover, power):
    case = W.dynamics_small("shared", seed=84, frames=24, per_frame=24, audio=150)
    case.params = {"window": 3, "r_pre": 0.5, "cover_thresh": cover, "dafps_power": power}
    want = _oracle(case)
    _certify(want)
    _compare(case, _run(case), want)


@pytest.mark.parametrize("r_pre", [1.0, 0.05, 0.6])
def test_budget_extremes(r_pre):
    case = W.dynamics_small("offset", seed=31)
    case.params = {"window": 3, "r_pre": r_pre}
    want = _oracle(case)
    _certify(want)
    _compare(case, _run(case), want)


# -- alternative alignment scorers (the supplement's scorer comparison) -------

@pytest.mark.parametrize("alignment", ["gated_cka", "cka", "av_cosine", "spatial_cka"])
@pytest.mark.parametrize("structure", ["shared", "offset"])
def test_alignment_scorers_small_clips(structure, alignment):
    case = W.dynamics_small(structure, seed=8)
    case.params = dict(case.params, alignment=alignment)
    log(f"[dynamics] small {structure}, {alignment}")
    want = _oracle(case)
    _certify(want)
    _compare(case, _run(case), want)


@pytest.mark.parametrize("alignment", ["cka", "av_cosine", "spatial_cka"])
@pytest.mark.parametrize("structure", ["shared", "offset"])
def test_alignment_scorers_7b_shape_60s_clip(structure, alignment):
    case = W.dynamics_cfg3(structure)
    case.params = dict(case.params, alignment=alignment)
    log(f"[dynamics] 60 s clip, 3584-d, {structure}, {alignment}")
    want = _oracle(case)
    _certify(want)
    _compare(case, _run(case), want)


def test_spatial_cka_ragged_batch_with_edge_shapes():
    # Bins of one audio token (N_A = F), a frame with more audio rows than a
    # tile, P not a multiple of the 16-row tile, and the largest P.
    parts = [
        W.dynamics_small("offset", seed=21, frames=30, per_frame=16, audio=375),
        W.dynamics_small("shared", seed=26, frames=10, per_frame=9, audio=10),     # one audio row per bin
        W.dynamics_small("shared", seed=23, frames=1, per_frame=5, audio=40),      # 40 audio rows, one frame
        W.dynamics_small("offset", seed=24, frames=20, per_frame=70, audio=250),
        W.dynamics_small("shared", seed=25, frames=12, per_frame=256, audio=150),
    ]
    case = _packed(parts, {"window": 3, "r_pre": 0.5, "alignment": "spatial_cka"})
    want = _oracle(case)
    _certify(want)
    got = _run(case)
    _compare(case, got, want)
    f0 = sum(p.seqs[0].n_frames for p in parts[:1])
    assert np.all(got["cka"][f0:f0 + 10] == 0.0)   # one-token bins have no audio covariance


# -- degenerate inputs: zero frame, static scene, duplicate and zero tokens --

@pytest.mark.parametrize("alignment", ["gated_cka", "cka", "av_cosine", "spatial_cka"])
@pytest.mark.parametrize("structure", ["shared", "offset"])
def test_degenerate_inputs_parity(structure, alignment):
    """A zero frame, a static scene (repeated frames and audio), duplicate
    tokens in an anchor frame and zero tokens and audio rows: zero CKA on
    degenerate windows, cosine exactly 1 between repeated tokens and 0 for
    zero ones, so the ties these inputs create fall the same way (lower
    index) on both sides."""
    case = W.dynamics_edge(structure)
    case.params = dict(case.params, alignment=alignment)
    log(f"[dynamics] edge clip {structure}, {alignment}")
    want = _oracle(case)
    _certify(want)
    _compare(case, _run(case), want)


def test_degenerate_inputs_parity_fp32_and_wide_dim():
    """The same degenerate clip at the 7B embedding width (the 256-tile gate
    GEMM) and with fp32 inputs (the fp32 gate GEMM)."""
    case = W.dynamics_edge("offset", dim=3584, frames=40, per_frame=24, audio=500)
    log("[dynamics] edge clip, 3584-d, bf16")
    want = _oracle(case)
    _certify(want)
    _compare(case, _run(case), want)
    f32 = W.DynamicsCase("f32", case.dim, W.bf16_bits_to_f32(case.xv), W.bf16_bits_to_f32(case.xa),
                         W.bf16_bits_to_f32(case.xq), case.seqs, case.params)
    log("[dynamics] edge clip, 3584-d, fp32")
    want = _oracle(f32, "f32")
    _certify(want)
    _compare(f32, _run(f32, "f32"), want, "f32")


def test_scorer_is_deterministic():
    """Two runs of the 60 s 7B-shape clip with the gate fired (atomic
    maxima, split-K Grams, cross-workgroup sums) give the same bits."""
    case = W.dynamics_cfg3("offset")
    a, b = _run(case), _run(case)
    for key in ("cka", "score", "budget", "segment", "gate", "kept"):
        assert np.array_equal(a[key].view(np.uint8), b[key].view(np.uint8)), key
    assert a["n_kept"] == b["n_kept"]


@pytest.mark.parametrize("dim,per_frame,audio", [
    (8, 15, 40),      # one partial K step: most K slices of a Gram are empty
    (40, 16, 97),     # a partial last K step; a whole tile of tokens
    (264, 17, 200),   # one token past a tile
    (520, 32, 64),    # a whole 2 x 2 tile block
    (1032, 33, 400),  # one token past a block; audio bins of two tiles
])
@pytest.mark.parametrize("alignment", ["gated_cka", "spatial_cka"])
def test_gram_blocks_at_their_edges(dim, per_frame, audio, alignment):
    """Anchor and spatial Grams where the tile blocks, the padding between
    audio and visual tiles and the K slices have remainders."""
    case = W.dynamics_small("offset", seed=92, dim=dim, frames=18, per_frame=per_frame, audio=audio)
    case.params = dict(case.params, alignment=alignment)
    want = _oracle(case)
    _certify(want)
    _compare(case, _run(case), want)


@pytest.mark.parametrize("frames,per_frame", [
    (127, 16),   # 256 pooling blocks of two slices: sixteen waves, one row each
    (127, 3),    # more waves than rows
    (128, 9),    # 258 blocks: four waves
    (40, 200),   # sixteen waves, a second turn of loads for the last rows
])
def test_pooling_blocks_either_side_of_the_rule(frames, per_frame):
    """Frame means and token norms where the pooling changes its wave count."""
    case = W.dynamics_small("offset", seed=96, dim=520, frames=frames, per_frame=per_frame, audio=3 * frames)
    want = _oracle(case)
    _certify(want)
    _compare(case, _run(case), want)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("dim,frames,audio", [
    (8, 127, 255),     # one partial K step, one short tile
    (40, 128, 256),    # a whole tile
    (264, 129, 257),   # one row and one column past a tile
    (1288, 300, 600),  # several tiles, a partial last K step
])
def test_gate_gemm_of_any_dim_and_dtype(dim, frames, audio, dtype):
    """Largest cosines of single-token frames (the frame score is 1 - d_hat
    with gamma 0) where the products' tiles and K steps have remainders, for
    fp32 rows (three bf16 parts each) and for bf16 rows."""
    import paper_2608_08794_amd as A
    rng = np.random.default_rng(dim)
    wide = np.exp(2.0 * rng.standard_normal((frames + audio, dim)))   # values over many binades
    x = (rng.standard_normal((frames + audio, dim)) * wide).astype(np.float32)
    raw = W.to_bf16_bits(x) if dtype == "bf16" else x
    xv, xa = raw[:frames], raw[frames:]
    clip = dict(n_frames=frames, per_frame=1, n_audio=audio, n_query=1, vis_off=0, aud_off=0, qry_off=0)
    out = A.apack_score_dynamics(to_dev(xv, dtype), to_dev(xa, dtype), to_dev(xa[:1], dtype), [clip],
                                 {"alignment": "av_cosine", "gamma": 0.0, "r_pre": 1.0})
    got = out["score"].cpu().numpy().astype(np.float64)
    d, _ = OD.direct_distance(widen(xv, dtype), widen(xa, dtype), frames, 1)
    want = 1.0 - OD.minmax(d)
    # Each of the 6 K / 32 partial sums (and K / 32 in bf16), the parts left
    # out and the scaling round by at most 2^-24 of sum |x y| <= |x| |y|; the
    # score holds three such errors over the range of d, and its own rounding.
    n = (6 if dtype == "f32" else 1) * (dim // 32 + 1) + 4
    tol = 4.0 * n * 2.0 ** -24 / (d.max() - d.min()) + 2.0 ** -23
    np.testing.assert_allclose(got, want, rtol=0, atol=tol)


@pytest.mark.parametrize("audio,visual,dim", [
    (33, 200, 64),      # 64-row tiles, one K stage (of four in flight)
    (33, 200, 320),     # five K stages
    (470, 9000, 320),   # 96 rows
    (700, 9000, 128),   # 128 rows
    (470, 17281, 128),  # 160 rows
    (1125, 9000, 128),  # 192 rows
    (1500, 9000, 128),  # 224 rows
    (700, 17281, 192),  # 256 rows
])
def test_gate_gemm_tile_heights(audio, visual, dim):
    """Largest cosines with every height of the 256-column tiles (chosen by
    how the tiles fill the compute units), with short last tiles and with
    fewer, as many and more K stages than LDS holds; one token per frame, the
    frame score is 1 - d_hat with gamma 0."""
    import paper_2608_08794_amd as A
    rng = np.random.default_rng(audio + visual)
    xv, xa = (W.to_bf16_bits(rng.standard_normal((n, dim)).astype(np.float32)) for n in (visual, audio))
    clip = dict(n_frames=visual, per_frame=1, n_audio=audio, n_query=1, vis_off=0, aud_off=0, qry_off=0)
    out = A.apack_score_dynamics(to_dev(xv, "bf16"), to_dev(xa, "bf16"), to_dev(xa[:1], "bf16"), [clip],
                                 {"alignment": "av_cosine", "gamma": 0.0, "r_pre": 1.0})
    got = out["score"].cpu().numpy().astype(np.float64)
    d, _ = OD.direct_distance(widen(xv, "bf16"), widen(xa, "bf16"), visual, 1)
    want = 1.0 - OD.minmax(d)
    # As above: dim / 32 partial sums and the scaling, each rounded by at most
    # 2^-24 of |x| |y|, three times over the range of d.
    tol = 4.0 * (dim // 32 + 4) * 2.0 ** -24 / (d.max() - d.min()) + 2.0 ** -23
    np.testing.assert_allclose(got, want, rtol=0, atol=tol)


@pytest.mark.parametrize("audio,visual,dim", [(7612, 20, 64), (6150, 34, 512)])
def test_gate_gemm_in_the_least_workspace(audio, visual, dim):
    """A workspace without room for the list of low tiles takes higher ones:
    the same bits, within the bytes given."""
    import re
    import paper_2608_08794_amd as A
    rng = np.random.default_rng(audio)
    xv, xa = (to_dev(W.to_bf16_bits(rng.standard_normal((n, dim)).astype(np.float32)), "bf16")
              for n in (visual, audio))
    clip = dict(n_frames=visual, per_frame=1, n_audio=audio, n_query=1, vis_off=0, aud_off=0, qry_off=0)
    args = (xv, xa, xa[:1].contiguous(), [clip], {"alignment": "av_cosine", "gamma": 0.0, "r_pre": 1.0})
    with pytest.raises(A.ApackError) as e:
        A.apack_score_dynamics(*args, workspace=torch.empty(256, dtype=torch.uint8, device="cuda"))
    least = int(re.search(r"< (\d+) needed", str(e.value)).group(1))
    assert least < A.apack_score_dynamics_query([clip], dim, args[4])[1]
    buf = torch.full((least + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
    got, want = A.apack_score_dynamics(*args, workspace=buf[:least]), A.apack_score_dynamics(*args)
    torch.cuda.synchronize()
    assert bool((buf[least:] == 0xA5).all())
    for k in ("cka", "score", "budget", "segment", "gate", "kept"):
        assert torch.equal(got[k].cpu(), want[k].cpu()), k


def test_gate_gemm_past_2_to_the_31_elements():
    """A clip whose last gate GEMM tiles start past 2^31 elements of the
    visual rows (131072 rows of 16384): frame scores 1 - d_hat (gamma 0)
    against torch, tile by tile."""
    import paper_2608_08794_amd as A
    dim, per_frame, frames, audio = 16384, 256, 514, 40
    n = frames * per_frame
    gen = torch.Generator(device="cuda").manual_seed(7)
    xv = torch.empty((n, dim), dtype=torch.bfloat16, device="cuda")
    for r in range(0, n, 8192):
        xv[r:r + 8192] = torch.randn((min(8192, n - r), dim), generator=gen, device="cuda")
    xa = torch.randn((audio, dim), generator=gen, device="cuda").bfloat16()
    xv[-per_frame:] = xa[0]   # the last frame repeats an audio row: the smallest distance
    clip = dict(n_frames=frames, per_frame=per_frame, n_audio=audio, n_query=1, vis_off=0, aud_off=0, qry_off=0)
    out = A.apack_score_dynamics(xv, xa, xa[:1].clone(), [clip], {"alignment": "av_cosine", "gamma": 0.0, "r_pre": 0.01})
    got = out["score"].cpu().double()
    an = xa.double()
    an /= an.norm(dim=1, keepdim=True)
    cos = []
    for r in range(0, n, 4096):
        x = xv[r:r + 4096].double()
        cos.append((x @ an.T).amax(dim=1) / x.norm(dim=1))
    d = 1.0 - torch.cat(cos).view(frames, per_frame).mean(dim=1).cpu()
    want = 1.0 - (d - d.min()) / (d.max() - d.min())
    # dim / 32 partial sums and the scaling round by at most 2^-24 of |x| |y|,
    # three times over the range of d.
    tol = 4.0 * (dim // 32 + 4) * 2.0 ** -24 / float(d.max() - d.min()) + 2.0 ** -23
    np.testing.assert_allclose(got.numpy(), want.numpy(), rtol=0, atol=tol)


@pytest.mark.parametrize("up,down", [(0, 0), (0, -60), (-118, 0), (-122, -118), (60, 100), (112, -120), (125, 125)])
def test_fp32_gate_gemm_of_rows_of_any_magnitude(up, down):
    """The direct distance is a cosine: visual rows times 2^up and audio rows
    times 2^down (products past fp32's range at both ends, parts of values
    below bf16's smallest subnormal) give the same bits as unscaled ones."""
    import paper_2608_08794_amd as A
    rng = np.random.default_rng(17)
    frames, audio, dim = 130, 70, 264
    x = np.clip(rng.standard_normal((frames + audio, dim)), -4, 4)
    # The scaled rows are rounded once (some elements are subnormal there),
    # and the unscaled ones are their exact multiples.
    sv = np.ldexp(x[:frames], up).astype(np.float32)
    sa = np.ldexp(x[frames:], down).astype(np.float32)
    ov = np.ldexp(sv.astype(np.float64), -up).astype(np.float32)
    oa = np.ldexp(sa.astype(np.float64), -down).astype(np.float32)
    clip = dict(n_frames=frames, per_frame=1, n_audio=audio, n_query=1, vis_off=0, aud_off=0, qry_off=0)
    got = []
    for xv, xa in ((ov, oa), (sv, sa)):
        out = A.apack_score_dynamics(to_dev(xv, "f32"), to_dev(xa, "f32"), to_dev(oa[:1], "f32"), [clip],
                                     {"alignment": "av_cosine", "gamma": 0.0, "r_pre": 1.0})
        got.append(out["score"].cpu().numpy())
    np.testing.assert_array_equal(got[0].view(np.uint32), got[1].view(np.uint32))
    d, _ = OD.direct_distance(ov.astype(np.float64), oa.astype(np.float64), frames, 1)
    # Rounding as in test_gate_gemm_of_any_dim_and_dtype.
    tol = 4.0 * (6 * (dim // 32 + 1) + 4) * 2.0 ** -24 / (d.max() - d.min()) + 2.0 ** -23
    np.testing.assert_allclose(got[0].astype(np.float64), 1.0 - OD.minmax(d), rtol=0, atol=tol)


# rms errors that a kernel of v_mfma_f32_32x32x2_f32 measured on the rows below.
@pytest.mark.parametrize("dim,kind,fp32_unit", [
    (264, "normal", 4.09e-8), (264, "one_signed", 2.59e-7), (264, "wide", 8.69e-8),
    (2048, "normal", 3.73e-8), (2048, "one_signed", 4.46e-7), (2048, "wide", 2.49e-7),
    (3584, "normal", 4.63e-8), (3584, "one_signed", 6.17e-7), (3584, "wide", 2.38e-7),
])
def test_fp32_gate_gemm_error_is_no_larger_than_the_fp32_matrix_units(dim, kind, fp32_unit):
    """rms error of 1 - distance over random rows (d_hat divides by the
    distance's range, which is taken out again)."""
    import paper_2608_08794_amd as A
    rng = np.random.default_rng(dim)
    frames, audio = 200, 60
    x = rng.standard_normal((frames + audio, dim))
    if kind == "one_signed":
        x = np.abs(x)
    if kind == "wide":
        x *= np.exp(2.0 * rng.standard_normal(x.shape))
    x = x.astype(np.float32)
    x[0], x[1] = x[frames], -x[frames]   # cosines of 1 and about -1 or 0: a wide range of d
    xv, xa = x[:frames], x[frames:]
    clip = dict(n_frames=frames, per_frame=1, n_audio=audio, n_query=1, vis_off=0, aud_off=0, qry_off=0)
    out = A.apack_score_dynamics(to_dev(xv, "f32"), to_dev(xa, "f32"), to_dev(xa[:1], "f32"), [clip],
                                 {"alignment": "av_cosine", "gamma": 0.0, "r_pre": 1.0})
    d, _ = OD.direct_distance(xv.astype(np.float64), xa.astype(np.float64), frames, 1)
    err = rms(out["score"].cpu().numpy(), 1.0 - OD.minmax(d)) * (d.max() - d.min())
    print(f"[gate error] dim {dim} {kind}: rms {err:.2e}", flush=True)
    assert err <= fp32_unit


@pytest.mark.parametrize("dim,frames,audio", [(8, 127, 255), (40, 128, 256), (264, 129, 257), (1288, 300, 600),
                                              (3584, 260, 513)])
def test_fp32_gate_gemm_sums_all_six_products(dim, frames, audio):
    """Rows whose second and third bf16 parts count: a part or a product that
    is lost or stale in any K step or tile exceeds the bound (an emulation on
    the CPU checks that it does)."""
    import paper_2608_08794_amd as A
    xv, xa = three_part_rows(np.random.default_rng(dim), frames, audio, dim)
    clip = dict(n_frames=frames, per_frame=1, n_audio=audio, n_query=1, vis_off=0, aud_off=0, qry_off=0)
    out = A.apack_score_dynamics(to_dev(xv, "f32"), to_dev(xa, "f32"), to_dev(xa[:1], "f32"), [clip],
                                 {"alignment": "av_cosine", "gamma": 0.0, "r_pre": 1.0})
    d, _ = OD.direct_distance(xv.astype(np.float64), xa.astype(np.float64), frames, 1)
    assert rms(out["score"].cpu().numpy(), 1.0 - OD.minmax(d)) < THREE_PART_RMS
