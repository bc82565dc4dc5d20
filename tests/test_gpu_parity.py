"""Parity of the HIP library with the CPU oracle, through the C ABI, on an MI355X.

Bars: tree and recombination indices bit-exact when both sides read the same
injected log-probabilities; float32 end to end: identical token sequences and
hypothesis scores within 1e-3, except after a decision the oracle took by less
than 1e-4; bf16-joint variant: scores within 2e-2, near tie below 5e-3 (this library's own
choice: a bf16 rounding boundary crossed on one side only moves a logit by about 5e-4, and a
few hundred such events add up over a decode).  A tree that leaves the oracle's at a near tie
is walked step by step (tree_check.py) instead of being dropped.
"""
import math

import numpy as np
import pytest

import synth_inputs as S
from gpu_common import compare, gpu_decode, gpu_decode_injected, make_walk, to_gpu

pytestmark = pytest.mark.gpu

TOL, TIE = 1e-3, 1e-4
# bf16-joint variant (the workloads name the precision, the paper does not): operands rounded to bfloat16 on one side
# in float32, on the other in float64; a rounding boundary crossed on one side only moves a logit by ~5e-4 at H = 640.
# Near-tie bar 5e-3 (every divergence measured at full size sat below it).  Score tolerance 2e-2: the bf16 matrix
# instructions add 16 k per step in an order of their own, and one utterance of workload c2 then ended 1.13e-2 from the
# oracle after 680 steps (1e-2, the value before those instructions were used, failed on it).
TOL_BF16, TIE_BF16 = 2e-2, 5e-3


@pytest.fixture(scope="module")
def amd():
    import paper_2506_00185_amd as A
    A.load_library()
    return A


def _case(c, seed, perturb=True, zero_len=False):
    w = S.make_weights(c, seed)
    if perturb:
        w = S.perturb_biases(w, seed + 1)
    L = S.make_lengths(c, seed + 2)
    if zero_len and len(L) > 2:
        L[1] = 0
        L[2] = c["T"]
    enc = S.make_enc(c, L, seed + 3)
    return w, L, enc


# ---------------------------------------------------------------- single stages

@pytest.mark.parametrize("prec,B,T,T_min,D,H", [("f32", 3, 37, 32, 96, 64), ("bf16", 3, 37, 32, 96, 64),
                                                ("f32", 5, 77, 72, 160, 224), ("bf16", 40, 60, 55, 64, 160),
                                                ("f32", 7, 300, 3, 64, 96), ("bf16", 12, 300, 3, 64, 96)])
def test_encoder_projection_matches_oracle(amd, oracle, prec, B, T, T_min, D, H):
    """Every frame of every utterance up to its length (tiles of the product that hold nothing but frames behind
    the ends of their utterances are left out: the last two cases have many), ragged tiles along both axes; the bf16
    variant rounds both operands to nearest even (a truncating conversion would show at this tolerance) and takes
    the 128 x 128 tile from 2048 frames up."""
    c = S.custom_config(B=B, T=T, T_min=T_min, D=D, H=H, P=32, E=32, V=40, beam=2, s=1, prec=prec)
    w, L, enc = _case(c, 300, zero_len=T_min < 10)
    dec = amd.BeamDecoder(c, w)
    gpu_decode(dec, enc, L, want_tree=False)
    f = dec.debug_encproj(c["B"], c["T"])
    rng = np.random.default_rng(5)
    picks = [(0, 0), (B - 1, L[B - 1] - 1), (B // 2, L[B // 2] // 2)]
    picks += [(b, L[b] - 1) for b in range(B) if L[b] > 0]                   # the last frame in use of each utterance
    picks += [(b, int(rng.integers(max(L[b], 1)))) for b in rng.integers(B, size=12)]
    for b, t in picks:
        if t < 0:
            continue
        np.testing.assert_allclose(f[b * c["T"] + t], oracle.enc_proj(c, w, enc[b, t]), atol=2e-5, rtol=0)


@pytest.mark.parametrize("n_target,order,V", [(1000, 4, 12), (60000, 4, 300), (30000, 6, 64), (200, 1, 50),
                                              (80000, 3, 1500)])
def test_lm_rows_match_oracle_lm(amd, oracle, n_target, order, V):
    """(V = 1500: more tokens than a block holds in registers, and successor lists longer than a block.)"""
    lm = S.make_lm(V=V, order=order, n_target=n_target, zipf_s=1.1, seed=n_target + order)
    g, o = amd.NGramLM(lm), oracle.LM(lm)
    rng = np.random.default_rng(1)
    w = max(order - 1, 1)
    ctx = np.full((64, w), -1, np.int32)
    stored = lm["tokens"][lm["order"] == max(order - 1, 1)]
    for i in range(64):
        n = rng.integers(0, order)  # tokens of history available
        if order > 1 and i % 3 == 0 and len(stored):
            hist = stored[rng.integers(0, len(stored))][: order - 1][::-1]
            n = min(n, len(hist))
            ctx[i, :n] = hist[:n]
        else:
            ctx[i, :n] = rng.integers(0, V, n)
    if order > 1:
        ctx[1] = -1
        ctx[1, 0] = 0  # the most frequent token alone: the longest successor list of the model
    got = g.debug_query(ctx)
    for i in range(64):
        hist = [int(x) for x in ctx[i] if x >= 0][::-1]  # oldest first
        want = o.query(hist, V)
        np.testing.assert_allclose(got[i], want, rtol=0, atol=2e-5)


# ------------------------------------------------------- index parity (injected)

@pytest.mark.parametrize("algo", ["alsd", "aes"])
@pytest.mark.parametrize("beam,V,model", [(4, 37, "rnnt"), (2, 5, "rnnt"), (7, 130, "rnnt"), (16, 64, "rnnt"),
                                          (1, 37, "rnnt"), (4, 37, "tdt"), (6, 9, "tdt")])
def test_injected_tree_and_recombination_are_bit_exact(amd, oracle, algo, beam, V, model):
    durations = (0, 1, 2, 3, 4) if model == "tdt" else ()
    B, T, C = 5, 14, 6
    c = S.custom_config(B=B, T=T, T_min=3, D=32, H=32, P=32, E=32, V=V, beam=beam, s=2, algo=algo, model=model,
                        durations=durations, gamma=1.5 if (algo == "aes" and V == 37) else float("inf"))
    L = S.make_lengths(c, 17)
    L[1] = 0
    L[2] = T
    tok, dur = S.make_injected(B, T, C, V, len(durations), seed=beam * 100 + V, levels=96 if V < 10 else 400,
                               blank_boost=40)
    w = S.make_weights(c, 1)
    dec = amd.BeamDecoder(c, w)
    g = gpu_decode_injected(dec, tok, dur, L)
    o = oracle.decode(c, None, None, L, injected=(tok, dur), log=True)
    assert np.array_equal(g["n_steps"], o["n_steps"])
    full, exempt = compare(g, o, tol=1e-9, tie=0.0, exact_tree=True)
    assert full == B and exempt == 0
    assert o["collisions"].sum() == 0


@pytest.mark.parametrize("algo", ["alsd", "aes"])
@pytest.mark.parametrize("beam,V,model,levels,boost", [(8, 3, "rnnt", 32, 0), (16, 2, "rnnt", 16, 0),
                                                       (4, 2, "rnnt", 16, 4), (8, 4, "tdt", 32, 0),
                                                       (4, 3, "rnnt", 200, 100)])
def test_injected_merge_heavy_tables_are_bit_exact(amd, oracle, algo, beam, V, model, levels, boost):
    """Tiny vocabularies and closely spaced (often tied) log-probabilities: many hypotheses with equal
    transcripts meet in the beam, so recombination and the tie-break order carry the result."""
    durations = (0, 1, 2, 3, 4) if model == "tdt" else ()
    B, T, C = 5, 14, 6
    c = S.custom_config(B=B, T=T, T_min=3, D=32, H=32, P=32, E=32, V=V, beam=beam, s=2, algo=algo, model=model,
                        durations=durations)
    L = S.make_lengths(c, 17)
    L[1] = 0
    L[2] = T
    tok, dur = S.make_injected(B, T, C, V, len(durations), seed=beam * 100 + V, levels=levels, blank_boost=boost)
    dec = amd.BeamDecoder(c, S.make_weights(c, 1))
    g = gpu_decode_injected(dec, tok, dur, L)
    o = oracle.decode(c, None, None, L, injected=(tok, dur), log=True)
    assert np.array_equal(g["n_steps"], o["n_steps"])
    full, exempt = compare(g, o, tol=1e-9, tie=0.0, exact_tree=True)
    assert full == B and exempt == 0
    n = o["n_steps"].max()
    slots = np.arange(beam)[None, None, :]
    m = o["log_merged"][:, :n]
    assert np.sum((m >= 0) & (m != slots)) >= 3, "the table does not exercise recombination"


@pytest.mark.parametrize("algo", ["alsd", "aes"])
@pytest.mark.parametrize("beam", [8, 9, 12, 16])
@pytest.mark.parametrize("spacing", [0.0, 2.0 ** -12, 2.0 ** -6], ids=["equal", "close", "apart"])
def test_injected_many_candidates_near_the_last_one_kept(amd, oracle, algo, beam, spacing):
    """Candidates of much the same score: far more than the 64 that are ranked against each other reach a first bound of the Beam
    best (close), or every bound (equal)."""
    B, T, C, V = 3, 8, 5, 120
    c = S.custom_config(B=B, T=T, T_min=3, D=32, H=32, P=32, E=32, V=V, beam=beam, s=3, algo=algo)
    L = S.make_lengths(c, 17)
    tok = (-5.0 - spacing * np.random.default_rng(beam).permuted(np.tile(np.arange(V + 1), (B, T, C, 1)), axis=-1)).astype(np.float32)
    g = gpu_decode_injected(amd.BeamDecoder(c, S.make_weights(c, 1)), tok, None, L)
    o = oracle.decode(c, None, None, L, injected=(tok, None), log=True)
    assert np.array_equal(g["n_steps"], o["n_steps"])
    full, exempt = compare(g, o, tol=1e-9, tie=0.0, exact_tree=True)
    assert full == B and exempt == 0


@pytest.mark.parametrize("T,beam,tree_kib", [(130, 8, 64), (150, 16, 144)])
def test_injected_long_utterances_walk_the_tree_in_memory(amd, oracle, T, beam, tree_kib):
    """Trees of more than 64 KiB per utterance (steps x beam x 8 bytes), and of more than the back-trace can hold in
    LDS beside its tables (160 - 17 KiB), which is then walked back where it lies, not from an on-chip copy; a
    shorter utterance beside it in the same batch ends earlier."""
    B, C, V, s = 2, 3, 6, 7
    assert T * (s + 1) * beam * 8 > tree_kib * 1024
    c = S.custom_config(B=B, T=T, T_min=3, D=32, H=32, P=32, E=32, V=V, beam=beam, s=s, algo="alsd")
    L = np.array([T, 41], np.int32)
    tok, _ = S.make_injected(B, T, C, V, 0, seed=77, levels=200, blank_boost=10)
    dec = amd.BeamDecoder(c, S.make_weights(c, 1))
    g = gpu_decode_injected(dec, tok, None, L)
    o = oracle.decode(c, None, None, L, injected=(tok, None), log=True)
    assert np.array_equal(g["n_steps"], o["n_steps"]) and g["n_steps"].max() > 300
    full, exempt = compare(g, o, tol=1e-9, tie=0.0, exact_tree=True)
    assert full == B and exempt == 0


def test_injected_tree_walk_gives_the_transcripts(amd, oracle):
    """Back-trace through (parent, token) on the host reproduces what the library reports."""
    B, T, C, V, beam = 3, 10, 4, 20, 5
    c = S.custom_config(B=B, T=T, D=32, H=32, P=32, E=32, V=V, beam=beam, s=3)
    L = np.array([10, 7, 1], np.int32)
    tok, _ = S.make_injected(B, T, C, V, 0, seed=5, blank_boost=100)
    dec = amd.BeamDecoder(c, S.make_weights(c, 1))
    g = gpu_decode_injected(dec, tok, None, L)
    o = oracle.decode(c, None, None, L, injected=(tok, None), log=True, snap_every=1)
    for b in range(B):
        n = g["n_steps"][b]
        for step in range(1, n + 1):
            for k in range(beam):
                want_len = o["snap_lens"][b, step - 1, k]
                if want_len < 0:
                    continue
                toks, slot = [], k
                for st in range(step - 1, -1, -1):
                    tk = g["token"][st, b, slot]
                    if tk >= 0:
                        toks.append(tk)
                    slot = g["parent"][st, b, slot]
                toks.reverse()
                assert toks == list(o["snap_tokens"][b, step - 1, k, :want_len])


# ------------------------------------------------------------ float32 end to end

@pytest.mark.parametrize("algo", ["alsd", "aes"])
@pytest.mark.parametrize("beam", [1, 3, 4])
def test_config1_tiny(amd, oracle, algo, beam):
    c = S.config(1, algo=algo, beam=beam)
    w, L, enc = S.make_weights(c), S.make_lengths(c), None
    enc = S.make_enc(c, L)
    dec = amd.BeamDecoder(c, w)
    g = gpu_decode(dec, enc, L)
    o = oracle.decode(c, w, enc, L, log=True)
    full, exempt = compare(g, o, TOL, TIE, walk=make_walk(oracle, c, w, enc, L, g, TOL))
    assert full + exempt == 1


@pytest.mark.parametrize("name,kw", [
    ("rnnt_alsd_ragged", dict(B=6, T=24, T_min=5, beam=4, s=3, algo="alsd")),
    ("rnnt_alsd_two_row_tiles", dict(B=6, T=16, T_min=8, beam=7, s=2, algo="alsd")),
    ("rnnt_aes", dict(B=5, T=20, T_min=6, beam=4, s=2, algo="aes")),
    ("rnnt_aes_margin", dict(B=5, T=20, T_min=6, beam=4, s=2, algo="aes", gamma=2.3)),
    ("tdt_aes_margin", dict(B=7, T=40, T_min=10, beam=4, s=2, algo="aes", gamma=2.3, model="tdt",
                            durations=(0, 1, 2, 3, 4))),
    ("tdt_alsd", dict(B=4, T=30, T_min=10, beam=5, s=2, algo="alsd", model="tdt", durations=(0, 1, 2, 3, 4))),
    ("beam16", dict(B=3, T=12, T_min=6, beam=16, s=2, algo="alsd")),
    ("rnnt_alsd_beam2", dict(B=5, T=16, T_min=6, beam=2, s=3, algo="alsd")),
    ("rnnt_alsd_beam1", dict(B=4, T=16, T_min=6, beam=1, s=3, algo="alsd")),
])
def test_full_width_model_small_batch(amd, oracle, name, kw):
    """Real layer widths (V = 1024 + blank spans 33 column chunks with a ragged tail), small batch."""
    c = S.custom_config(D=1024, H=640, P=640, E=640, V=1024, blank_bias=3.0, **kw)
    w, L, enc = _case(c, 400 + len(name), zero_len=True)
    if c["model"] == "tdt":
        w["b_out"][c["V"] + 2] += 2.0
    dec = amd.BeamDecoder(c, w)
    g = gpu_decode(dec, enc, L)
    o = oracle.decode(c, w, enc, L, log=True)
    full, exempt = compare(g, o, TOL, TIE, walk=make_walk(oracle, c, w, enc, L, g, TOL))
    assert full + exempt == c["B"]
    assert full >= c["B"] // 2, (full, exempt)
    assert g["lens"][1, 0] == 0 and g["scores"][1, 0] == 0.0 and g["n_steps"][1] == 0  # the empty utterance


@pytest.mark.parametrize("name,kw,prec", [
    ("rnnt_alsd_256_slots", dict(B=32, T=6, T_min=2, beam=8, s=2, algo="alsd"), "f32"),
    ("tdt_aes_288_slots", dict(B=36, T=16, T_min=5, beam=8, s=2, algo="aes", model="tdt", durations=(0, 1, 2, 3, 4)), "f32"),
    ("tdt_alsd_256_slots_bf16", dict(B=64, T=14, T_min=4, beam=4, s=2, algo="alsd", model="tdt",
                                     durations=(0, 1, 2, 3, 4)), "bf16"),
])
def test_full_width_model_wide_batch(amd, oracle, name, kw, prec):
    """From 256 slots up at the real layer widths: more joint blocks than compute units, so the blank and duration
    columns (alone in the last column chunk, V % 32 == 0) are computed by the token chunks' blocks, and the blocks of
    the recurrent product take four slot tiles each (256 slots) or two (288: the last block of a gate tile has one).
    In the resident loop, and in the replayed graph that this describes."""
    c = S.custom_config(D=256, H=640, P=640, E=640, V=1024, blank_bias=3.0, prec=prec, **kw)
    w, L, enc = _case(c, 450 + len(name))
    if c["model"] == "tdt":
        w["b_out"][c["V"] + 2] += 2.0
    dec = amd.BeamDecoder(c, w)
    o = oracle.decode(c, w, enc, L, log=True)
    tol, tie = (TOL_BF16, TIE_BF16) if prec == "bf16" else (TOL, TIE)
    for loop in ("resident", "graph"):
        if loop == "graph":
            dec.debug_rebuild_resident(0)
        g = gpu_decode(dec, enc, L)
        assert dec.last_step_loop() == loop
        full, exempt = compare(g, o, tol, tie, walk=make_walk(oracle, c, w, enc, L, g, tol))
        assert full + exempt == c["B"]
        assert full >= c["B"] // 2, (full, exempt)


def test_odd_shapes(amd, oracle):
    """Vocabulary, batch and frame counts that are not multiples of any tile size."""
    c = S.custom_config(B=9, T=11, T_min=1, D=96, H=160, P=96, E=64, V=77, beam=5, s=2, algo="alsd")
    w, L, enc = _case(c, 500)
    dec = amd.BeamDecoder(c, w, max_B=12, max_T=15, max_beam=8)
    g = gpu_decode(dec, enc, L)
    o = oracle.decode(c, w, enc, L, log=True)
    full, exempt = compare(g, o, TOL, TIE, walk=make_walk(oracle, c, w, enc, L, g, TOL))
    assert full + exempt == 9 and full >= 5


def test_stateless_prediction_network(amd, oracle):
    c = S.custom_config(B=4, T=20, T_min=8, D=128, H=160, P=160, E=160, V=300, beam=10, s=2, algo="aes",
                        pred="stateless", ctx=2, blank_bias=3.0)
    w, L, enc = _case(c, 600)
    dec = amd.BeamDecoder(c, w)
    g = gpu_decode(dec, enc, L)
    o = oracle.decode(c, w, enc, L, log=True)
    full, exempt = compare(g, o, TOL, TIE, walk=make_walk(oracle, c, w, enc, L, g, TOL))
    assert full + exempt == 4 and full >= 2


@pytest.mark.parametrize("pred", ["lstm", "stateless"])
def test_bf16_joint_variant(amd, oracle, pred):
    c = S.custom_config(B=4, T=20, T_min=8, D=128, H=160, P=160, E=160, V=300, beam=4, s=2, algo="alsd",
                        pred=pred, ctx=2 if pred == "stateless" else 0, prec="bf16", blank_bias=3.0)
    w, L, enc = _case(c, 700)
    dec = amd.BeamDecoder(c, w)
    g = gpu_decode(dec, enc, L)
    o = oracle.decode(c, w, enc, L, log=True)
    full, exempt = compare(g, o, TOL_BF16, TIE_BF16, walk=make_walk(oracle, c, w, enc, L, g, TOL_BF16))
    assert full + exempt == 4
    # the variant must differ from the float32 run, or the rounding is not happening
    o32 = oracle.decode(dict(c, prec="f32"), w, enc, L)
    assert not np.allclose(o32["scores"], o["scores"], atol=1e-6)


def test_lm_fusion(amd, oracle):
    V = 300
    c = S.custom_config(B=4, T=16, T_min=8, D=128, H=160, P=160, E=160, V=V, beam=8, s=3, algo="alsd",
                        blank_bias=3.0)
    w, L, enc = _case(c, 800)
    lm = S.make_lm(V=V, order=4, n_target=40000, zipf_s=1.1, seed=3)
    glm, olm = amd.NGramLM(lm), oracle.LM(lm)
    dec = amd.BeamDecoder(c, w)
    g = gpu_decode(dec, enc, L, lm=glm, lm_weight=0.3)
    o = oracle.decode(c, w, enc, L, lm=olm, lm_weight=0.3, log=True)
    full, exempt = compare(g, o, TOL, TIE, walk=make_walk(oracle, c, w, enc, L, g, TOL, lm=olm, lm_weight=0.3))
    assert full + exempt == 4 and full >= 2
    # weight 0 gives the run without LM
    g0 = gpu_decode(dec, enc, L, lm=glm, lm_weight=0.0)
    g1 = gpu_decode(dec, enc, L)
    np.testing.assert_array_equal(g0["tokens"], g1["tokens"])
    np.testing.assert_allclose(g0["scores"], g1["scores"], atol=1e-9)
    assert not np.array_equal(g["scores"], g1["scores"])


def test_lm_fusion_with_a_row_too_large_for_the_projection_launch(amd, oracle):
    """LM rows of more than 16 KiB (V > 4096) are built beside the cell update, not beside the projection's tiles."""
    V = 4200
    c = S.custom_config(B=3, T=10, T_min=6, D=64, H=96, P=96, E=96, V=V, beam=3, s=2, algo="alsd", blank_bias=3.0)
    w, L, enc = _case(c, 830)
    lm = S.make_lm(V=V, order=3, n_target=30000, zipf_s=1.1, seed=9)
    glm, olm = amd.NGramLM(lm), oracle.LM(lm)
    dec = amd.BeamDecoder(c, w, joint_path="fused")
    g = gpu_decode(dec, enc, L, lm=glm, lm_weight=0.4)
    o = oracle.decode(c, w, enc, L, lm=olm, lm_weight=0.4, log=True)
    full, exempt = compare(g, o, TOL, TIE, walk=make_walk(oracle, c, w, enc, L, g, TOL, lm=olm, lm_weight=0.4))
    assert full + exempt == 3 and full >= 2
    assert not np.array_equal(g["scores"], gpu_decode(dec, enc, L)["scores"])


@pytest.mark.parametrize("rule,prune,beam,algo", [(3, "late", 4, "alsd"), (4, "early", 4, "alsd"), (3, "early", 8, "alsd"),
                                                  (4, "early", 10, "aes")])
def test_lm_fusion_rules_and_early_pruning(amd, oracle, rule, prune, beam, algo):
    """Eq. (3) and early pruning (Sec. 2.3) against the oracle's versions of them; beam 10 goes through
    the multi-pass selection of wide beams."""
    V = 300
    c = S.custom_config(B=4, T=16, T_min=8, D=128, H=160, P=160, E=160, V=V, beam=beam, s=3, algo=algo,
                        blank_bias=3.0)
    w, L, enc = _case(c, 810 + beam)
    lm = S.make_lm(V=V, order=4, n_target=40000, zipf_s=1.1, seed=3)
    glm, olm = amd.NGramLM(lm), oracle.LM(lm)
    dec = amd.BeamDecoder(c, w, lm_rule=rule, lm_prune=prune)
    g = gpu_decode(dec, enc, L, lm=glm, lm_weight=0.5)
    o = oracle.decode(c, w, enc, L, lm=olm, lm_weight=0.5, lm_rule=rule, lm_prune=prune, log=True)
    full, exempt = compare(g, o, TOL, TIE, walk=make_walk(oracle, c, w, enc, L, g, TOL, lm=olm, lm_weight=0.5,
                                                          lm_rule=rule, lm_prune=prune))
    assert full + exempt == 4 and full >= 2
    # the mode must matter on this input, or the test could not tell it from the default
    o_default = oracle.decode(c, w, enc, L, lm=olm, lm_weight=0.5)
    assert not np.allclose(o_default["scores"], o["scores"], atol=1e-6)


# ------------------------------------------- AES++ maximum-length prefix search

@pytest.mark.parametrize("beam,V,model,levels,boost", [(4, 37, "rnnt", 400, 40), (8, 3, "rnnt", 32, 0), (3, 5, "tdt", 96, 10),
                                                       (16, 4, "rnnt", 64, 0), (6, 2, "rnnt", 16, 0)])
def test_injected_prefix_search_tree_is_bit_exact(amd, oracle, beam, V, model, levels, boost):
    """Tiny vocabularies: the beam often holds a transcript together with its one-token extension in one frame,
    so the prefix credit decides many cuts."""
    durations = (0, 1, 2) if model == "tdt" else ()
    B, T, C = 5, 14, 6
    c = S.custom_config(B=B, T=T, T_min=3, D=32, H=32, P=32, E=32, V=V, beam=beam, s=3, algo="aes", model=model,
                        durations=durations, aes_prefix=True)
    L = S.make_lengths(c, 19)
    L[1] = 0
    L[2] = T
    tok, dur = S.make_injected(B, T, C, V, len(durations), seed=beam * 100 + V + 7, levels=levels, blank_boost=boost)
    dec = amd.BeamDecoder(c, S.make_weights(c, 1))
    g = gpu_decode_injected(dec, tok, dur, L)
    o = oracle.decode(c, None, None, L, injected=(tok, dur), log=True)
    assert np.array_equal(g["n_steps"], o["n_steps"])
    full, exempt = compare(g, o, tol=1e-9, tie=0.0, exact_tree=True)
    assert full == B and exempt == 0
    o_plain = oracle.decode(dict(c, aes_prefix=False), None, None, L, injected=(tok, dur), log=True)
    assert not (np.array_equal(o_plain["log_parent"], o["log_parent"]) and np.array_equal(o_plain["log_token"], o["log_token"])), \
        "the prefix search changes nothing on this table"


@pytest.mark.parametrize("kw", [dict(beam=4), dict(beam=8, gamma=2.3), dict(beam=4, model="tdt", durations=(0, 1, 2, 3, 4))])
def test_prefix_search_with_the_networks(amd, oracle, kw):
    c = S.custom_config(B=5, T=20, T_min=8, D=128, H=160, P=160, E=160, V=300, s=3, algo="aes", blank_bias=3.0,
                        aes_prefix=True, **kw)
    w, L, enc = _case(c, 1200 + kw["beam"])
    dec = amd.BeamDecoder(c, w)
    g = gpu_decode(dec, enc, L)
    o = oracle.decode(c, w, enc, L, log=True)
    full, exempt = compare(g, o, TOL, TIE)
    assert full + exempt == 5 and full >= 3
    with pytest.raises(RuntimeError, match="aes_prefix_search"):
        amd.BeamDecoder(dict(c, model="tdt", durations=(0, 1), tdt_pairs=True), S.make_weights(dict(c, model="tdt", durations=(0, 1)), 3))


# ------------------------------------------- TDT with every (symbol, duration) pair as a candidate

@pytest.mark.parametrize("algo", ["alsd", "aes"])
@pytest.mark.parametrize("beam,V", [(4, 37), (6, 9), (8, 3), (1, 20)])
def test_injected_tdt_pairs_tree_is_bit_exact(amd, oracle, algo, beam, V):
    durations = (0, 1, 2, 3, 4)
    B, T, C = 5, 14, 6
    c = S.custom_config(B=B, T=T, T_min=3, D=32, H=32, P=32, E=32, V=V, beam=beam, s=2, algo=algo, model="tdt",
                        durations=durations, tdt_pairs=True)
    L = S.make_lengths(c, 18)
    L[1] = 0
    L[2] = T
    tok, dur = S.make_injected(B, T, C, V, len(durations), seed=beam * 100 + V + 1, levels=96 if V < 10 else 400,
                               blank_boost=40)
    dec = amd.BeamDecoder(c, S.make_weights(c, 1))
    g = gpu_decode_injected(dec, tok, dur, L)
    o = oracle.decode(c, None, None, L, injected=(tok, dur), log=True)
    assert np.array_equal(g["n_steps"], o["n_steps"])
    full, exempt = compare(g, o, tol=1e-9, tie=0.0, exact_tree=True)
    assert full == B and exempt == 0
    # the rule matters on this input
    o1 = oracle.decode(dict(c, tdt_pairs=False), None, None, L, injected=(tok, dur))
    assert beam == 1 or not np.array_equal(o1["scores"], o["scores"])


@pytest.mark.parametrize("algo,beam", [("alsd", 4), ("aes", 8)])
def test_tdt_pairs_with_the_networks(amd, oracle, algo, beam):
    c = S.custom_config(B=4, T=20, T_min=8, D=128, H=160, P=160, E=160, V=300, beam=beam, s=2, algo=algo,
                        model="tdt", durations=(0, 1, 2, 3, 4), blank_bias=3.0, tdt_pairs=True)
    w, L, enc = _case(c, 1100 + beam)
    dec = amd.BeamDecoder(c, w)
    g = gpu_decode(dec, enc, L)
    o = oracle.decode(c, w, enc, L, log=True)
    full, exempt = compare(g, o, TOL, TIE)  # (the step-by-step walk knows the one-duration rule only)
    assert full + exempt == 4 and full >= 2
    with pytest.raises(RuntimeError, match="tdt_all_pairs"):
        amd.BeamDecoder(dict(c, model="rnnt", durations=()), S.make_weights(dict(c, model="rnnt", durations=()), 3))


# ------------------------------------------- vocabularies that fill their last chunk

@pytest.mark.parametrize("kw", [
    dict(V=64, H=96, beam=4, B=9, algo="alsd"),                                           # 2 token chunks, 32 rows a tile
    dict(V=128, H=192, beam=8, B=5, algo="aes", model="tdt", durations=(0, 1, 2, 3, 4), gamma=2.3),
    dict(V=96, H=160, beam=3, B=7, algo="alsd", prec="bf16", model="tdt", durations=(0, 1, 2)),
    dict(V=32, H=800, beam=2, B=3, algo="aes"),                                           # one token chunk, a wide joint
    dict(V=160, H=128, beam=12, B=4, algo="alsd"),                                        # selection in a launch of its own
])
def test_blank_and_durations_alone_in_the_last_chunk(amd, oracle, kw):
    """V % 32 == 0: blank and durations get no blocks of their own; the token-chunk blocks of a tile compute them for
    one hypothesis each (or several, when the tile has more hypotheses than the vocabulary has chunks)."""
    c = S.custom_config(T=16, T_min=5, D=64, P=96, E=64, s=3, blank_bias=3.0, **kw)
    w, L, enc = _case(c, 1400 + kw["V"], zero_len=True)
    dec = amd.BeamDecoder(c, w)
    g = gpu_decode(dec, enc, L)
    o = oracle.decode(c, w, enc, L, log=True)
    tol, tie = (TOL_BF16, TIE_BF16 * 2) if c["prec"] == "bf16" else (TOL, TIE)
    full, exempt = compare(g, o, tol, tie, walk=make_walk(oracle, c, w, enc, L, g, tol))
    assert full + exempt == c["B"] and full >= c["B"] // 2


# ------------------------------------------- logits through HBM (bf16 matrix-core joint)

@pytest.mark.parametrize("name,kw,lm_w", [
    ("rnnt_aes_k10", dict(model="rnnt", algo="aes", beam=10, V=2501, B=5), 0.0),
    ("rnnt_alsd_k4", dict(model="rnnt", algo="alsd", beam=4, V=1030, B=9), 0.0),
    ("tdt_alsd_k6", dict(model="tdt", algo="alsd", beam=6, V=777, B=3, durations=(0, 1, 2, 3, 4)), 0.0),
    ("rnnt_alsd_k16_lm", dict(model="rnnt", algo="alsd", beam=16, V=300, B=2), 0.3),
    ("rnnt_alsd_k5_lm_early", dict(model="rnnt", algo="alsd", beam=5, V=300, B=3), 0.4),
    # fewer 32-column chunks than the beam is wide: the chunk statistics give no bound, every key is collected
    ("rnnt_aes_k16_v200", dict(model="rnnt", algo="aes", beam=16, V=200, B=2), 0.0),
    # ... and more keys than the row kernel's list holds: its plain rounds over the row in memory
    ("rnnt_alsd_k12_v300", dict(model="rnnt", algo="alsd", beam=12, V=300, B=2), 0.0),
])
def test_materialized_logits_path(amd, oracle, name, kw, lm_w):
    """Same bars as the bf16 variant of the fused path; shapes that leave ragged tails in every
    tile of the contraction (V % 256, V % 4, rows % 160) and in the row scan."""
    c = S.custom_config(T=14, T_min=5, D=64, H=160, P=96, E=96, s=2, pred="stateless", ctx=2, prec="bf16",
                        blank_bias=3.0, **kw)
    w, L, enc = _case(c, 900 + kw["beam"])
    glm = olm = None
    if lm_w:
        lm = S.make_lm(V=c["V"], order=3, n_target=20000, zipf_s=1.1, seed=5)
        glm, olm = amd.NGramLM(lm), oracle.LM(lm)
    prune = "early" if name.endswith("early") else "late"
    dec = amd.BeamDecoder(c, w, joint_path="materialized", lm_prune=prune)
    g = gpu_decode(dec, enc, L, lm=glm, lm_weight=lm_w)
    o = oracle.decode(c, w, enc, L, lm=olm, lm_weight=lm_w, lm_prune=prune, log=True)
    full, exempt = compare(g, o, TOL_BF16, TIE_BF16, walk=make_walk(oracle, c, w, enc, L, g, TOL_BF16, lm=olm,
                                                                    lm_weight=lm_w, lm_prune=prune))
    assert full + exempt == c["B"] and full >= 1
    # and against the fused path of this library, to the same bar
    dec_f = amd.BeamDecoder(c, w, joint_path="fused", lm_prune=prune)
    gf = gpu_decode(dec_f, enc, L, lm=glm, lm_weight=lm_w)
    same = sum(int(np.array_equal(g["tokens"][b, 0], gf["tokens"][b, 0])) for b in range(c["B"]))
    assert same >= c["B"] - exempt - 1


@pytest.mark.parametrize("lm_w", [0.0, 0.3])
def test_materialized_logits_path_with_every_duration_pair(amd, oracle, lm_w):
    """The row kernel without a tail (chunk statistics, or the whole row when an LM term is in the keys), then the
    selection over (symbol, duration) pairs and the activations in launches of their own."""
    c = S.custom_config(B=4, T=14, T_min=5, D=64, H=160, P=96, E=96, V=700, beam=4, s=2, algo="alsd", model="tdt",
                        durations=(0, 1, 2, 3, 4), pred="stateless", ctx=2, prec="bf16", blank_bias=3.0, tdt_pairs=True)
    w, L, enc = _case(c, 1190)
    glm = olm = None
    if lm_w:
        lm = S.make_lm(V=c["V"], order=3, n_target=20000, zipf_s=1.1, seed=7)
        glm, olm = amd.NGramLM(lm), oracle.LM(lm)
    dec = amd.BeamDecoder(c, w, joint_path="materialized")
    g = gpu_decode(dec, enc, L, lm=glm, lm_weight=lm_w)
    o = oracle.decode(c, w, enc, L, lm=olm, lm_weight=lm_w, log=True)
    full, exempt = compare(g, o, TOL_BF16, TIE_BF16)  # (the step-by-step walk knows the one-duration rule only)
    assert full + exempt == 4 and full >= 2
    gf = gpu_decode(amd.BeamDecoder(c, w, joint_path="fused"), enc, L, lm=glm, lm_weight=lm_w)
    same = sum(int(np.array_equal(g["tokens"][b, 0], gf["tokens"][b, 0])) for b in range(4))
    assert same >= 4 - exempt - 1


def test_materialized_path_is_refused_where_it_cannot_run(amd):
    c = S.custom_config(B=2, T=8, T_min=4, D=64, H=64, P=64, E=64, V=50, beam=2, s=2, algo="alsd")
    w, L, enc = _case(c, 950)
    with pytest.raises(RuntimeError, match="MATERIALIZED"):
        amd.BeamDecoder(c, w, joint_path="materialized")


# ------------------------------------------------------------- behaviour of the ABI

def test_graph_replay_equals_plain_launches_and_repeats(amd):
    c = S.custom_config(B=5, T=20, T_min=6, D=128, H=160, P=160, E=160, V=300, beam=4, s=3, algo="alsd")
    w, L, enc = _case(c, 900)
    a = amd.BeamDecoder(c, w, use_graph=True)
    b = amd.BeamDecoder(c, w, use_graph=False)
    ra = [gpu_decode(a, enc, L) for _ in range(3)]
    rb = gpu_decode(b, enc, L)
    for r in ra:
        for key in ("tokens", "lens", "scores", "n_steps", "parent", "token", "merged"):
            np.testing.assert_array_equal(r[key], rb[key])
    # a different batch on the same handle, then the first one again
    L2 = L.copy()
    L2[0] = 3
    r2 = gpu_decode(a, enc, L2)
    assert r2["n_steps"][0] <= 3 * 4
    r3 = gpu_decode(a, enc, L)
    np.testing.assert_array_equal(r3["scores"], rb["scores"])


def test_async_enqueue_gives_the_same_result(amd):
    """async_enqueue = 1 enqueues the upper bound of steps without following the device; the result is the
    same as that of the default loop, bit for bit, with and without graph replay."""
    c = S.custom_config(B=5, T=20, T_min=6, D=128, H=160, P=160, E=160, V=300, beam=4, s=3, algo="alsd")
    w, L, enc = _case(c, 900)
    ref = gpu_decode(amd.BeamDecoder(c, w, use_graph=False), enc, L)
    for graph in (True, False):
        dec = amd.BeamDecoder(c, w, use_graph=graph, async_enqueue=True)
        for _ in range(2):
            r = gpu_decode(dec, enc, L)
            for key in ("tokens", "lens", "scores", "n_steps", "parent", "token", "merged"):
                np.testing.assert_array_equal(r[key], ref[key])


def test_enqueue_pacing_hears_from_every_kind_of_step(amd, capfd, monkeypatch):
    """The enqueueing thread follows the device through a pinned word that one launch per chunk of 16 steps writes.
    Every kind of step (full-width and generic LSTM models, stateless, materialised logits with and without an LM,
    injected log-probabilities) must write it: a decode of several chunks never has to fall back to waiting for the
    stream (the library reports a fall-back on stderr when RNNT_BEAM_TRACE_PACING is set at create), and decodes the
    same as with everything enqueued up front."""
    monkeypatch.setenv("RNNT_BEAM_TRACE_PACING", "1")
    cases = [
        (S.custom_config(B=3, T=30, T_min=20, D=64, H=640, P=640, E=640, V=300, beam=4, s=3, algo="alsd"), {}),
        (S.custom_config(B=3, T=30, T_min=20, D=64, H=640, P=640, E=640, V=300, beam=4, s=3, algo="alsd",
                         prec="bf16"), {}),
        (S.custom_config(B=3, T=30, T_min=20, D=64, H=160, P=96, E=96, V=300, beam=4, s=3, algo="aes"), {}),
        (S.custom_config(B=3, T=30, T_min=20, D=64, H=160, P=96, E=96, V=300, beam=4, s=3, pred="stateless",
                         ctx=2), {}),
        (S.custom_config(B=3, T=30, T_min=20, D=64, H=160, P=96, E=96, V=300, beam=4, s=3, pred="stateless", ctx=2,
                         prec="bf16"), dict(joint_path="materialized")),
        (S.custom_config(B=3, T=30, T_min=20, D=64, H=160, P=96, E=96, V=300, beam=12, s=3, pred="stateless", ctx=2,
                         prec="bf16"), dict(joint_path="materialized")),
    ]
    for i, (c, kw) in enumerate(cases):
        w, L, enc = _case(c, 1200 + i)
        dec = amd.BeamDecoder(c, w, **kw)
        dec.debug_rebuild_resident(0)  # (the resident loop has no chunks)
        r = gpu_decode(dec, enc, L)
        assert dec.last_step_loop() == "graph" and r["n_steps"].max() > 2 * 16
        ref = gpu_decode(amd.BeamDecoder(c, w, async_enqueue=True, **kw), enc, L)
        for key in ("tokens", "lens", "scores", "n_steps"):
            np.testing.assert_array_equal(r[key], ref[key])
    c = S.custom_config(B=3, T=30, T_min=20, D=64, H=160, P=96, E=96, V=300, beam=5, s=3, pred="stateless", ctx=2,
                        prec="bf16")
    w, L, enc = _case(c, 1210)
    lm = amd.NGramLM(S.make_lm(V=c["V"], order=3, n_target=5000, zipf_s=1.1, seed=5))
    r = gpu_decode(amd.BeamDecoder(c, w, joint_path="materialized"), enc, L, lm=lm, lm_weight=0.3)
    assert r["n_steps"].max() > 2 * 16
    B, T, C, V = 2, 40, 3, 6
    c = S.custom_config(B=B, T=T, T_min=30, D=32, H=32, P=32, E=32, V=V, beam=4, s=3, algo="alsd")
    tok, _ = S.make_injected(B, T, C, V, 0, seed=78, levels=200, blank_boost=10)
    r = gpu_decode_injected(amd.BeamDecoder(c, S.make_weights(c, 1)), tok, None, S.make_lengths(c, 3))
    assert r["n_steps"].max() > 2 * 16
    assert "pacing fell back" not in capfd.readouterr().err


def test_split_projection_at_a_generic_width(amd, oracle):
    """P = 128: the prediction projection is split in two along k across blocks with the generic (any P % 128 == 0)
    form of the kernel, and all gate tiles ride in the main launch."""
    c = S.custom_config(B=6, T=18, T_min=7, D=64, H=96, P=128, E=64, V=90, beam=4, s=2, algo="alsd", blank_bias=3.0)
    w, L, enc = _case(c, 970)
    dec = amd.BeamDecoder(c, w)
    g = gpu_decode(dec, enc, L)
    o = oracle.decode(c, w, enc, L, log=True)
    full, exempt = compare(g, o, TOL, TIE, walk=make_walk(oracle, c, w, enc, L, g, TOL))
    assert full + exempt == 6 and full >= 4


@pytest.mark.parametrize("kw", [dict(B=11, beam=4, algo="alsd"), dict(B=3, beam=8, algo="aes", gamma=2.3),
                                dict(B=19, beam=2, algo="aes", model="tdt", durations=(0, 1, 2, 3, 4)),
                                dict(B=32, beam=4, algo="alsd", prec="bf16"), dict(B=8, beam=1, algo="alsd")])
def test_single_launch_step_loop_equals_the_per_step_launches(amd, oracle, kw):
    """persistent_kernel = 1: the whole loop in one launch, the blocks of each XCD decoding their own utterances.
    At these widths (P = 192) both paths run the same tile routines on the same operands, so trees, transcripts
    and scores must be identical bit for bit; batches that leave some XCDs without an utterance included."""
    c = S.custom_config(T=22, T_min=6, D=64, H=192, P=192, E=64, V=150, s=3, blank_bias=3.0, **kw)
    w, L, enc = _case(c, 1300 + kw["B"], zero_len=True)
    ref = gpu_decode(amd.BeamDecoder(c, w, use_graph=False), enc, L)
    dec = amd.BeamDecoder(c, w, persistent=True)
    for _ in range(2):
        r = gpu_decode(dec, enc, L)
        assert r["rc"] == 0 and dec.last_step_loop() == "single launch"
        for key in ("tokens", "lens", "scores", "n_steps", "parent", "token", "merged"):
            np.testing.assert_array_equal(r[key], ref[key])
    o = oracle.decode(c, w, enc, L, log=True)
    tol, tie = (TOL_BF16, TIE_BF16) if c["prec"] == "bf16" else (TOL, TIE)
    full, exempt = compare(r, o, tol, tie, walk=make_walk(oracle, c, w, enc, L, r, tol))
    assert full + exempt == c["B"] and full >= c["B"] // 2


def test_single_launch_step_loop_gives_up_cleanly(amd):
    """A wait between blocks that runs into its limit ends the kernel (every block returns) and is reported."""
    c = S.custom_config(B=4, T=12, T_min=6, D=64, H=192, P=192, E=64, V=50, beam=4, s=2, algo="alsd")
    w, L, enc = _case(c, 1350)
    dec = amd.BeamDecoder(c, w, persistent=True)
    dec.debug_set_spin_limit(1)
    r = gpu_decode(dec, enc, L, want_tree=False, check=False)
    assert r["rc"] == -3
    dec.debug_set_spin_limit(1 << 22)
    r = gpu_decode(dec, enc, L, want_tree=False)
    assert r["rc"] == 0 and np.all(r["lens"][:, 0] >= 0)


def test_error_paths(amd):
    import torch
    from paper_2506_00185_amd import RnntBeamError
    c = S.custom_config(B=2, T=8, D=32, H=32, P=32, E=32, V=10, beam=2, s=2)
    w, L, enc = _case(c, 950)
    dec = amd.BeamDecoder(c, w)
    r = dec.__class__.results
    with pytest.raises(RnntBeamError, match="-5"):
        dec._shape = (2, 2)
        dec.results()
    with pytest.raises(RnntBeamError, match="-1"):
        dec.decode(to_gpu(enc, torch.float32), to_gpu(L, torch.int32), beam=3)  # beyond max_beam
    with pytest.raises(RnntBeamError):
        amd.BeamDecoder(dict(c, H=33), w)  # unsupported width
    ct = S.custom_config(B=2, T=8, D=32, H=32, P=32, E=32, V=10, beam=2, s=2, model="tdt", durations=(0, 1, 300))
    with pytest.raises(RnntBeamError, match="255"):
        amd.BeamDecoder(ct, S.make_weights(ct, 1))  # a duration that does not fit a byte
    bad = enc.copy()
    bad[1, 2, 3] = np.nan
    dec.decode(to_gpu(bad, torch.float32), to_gpu(L, torch.int32))
    assert dec.results(check=False)["rc"] == -4
    Lbad = L.copy()
    Lbad[0] = 99
    dec.decode(to_gpu(enc, torch.float32), to_gpu(Lbad, torch.int32))
    assert dec.results(check=False)["rc"] == -1
    g = gpu_decode(dec, enc, L, want_tree=False)  # the handle still works
    assert g["rc"] == 0 and np.all(g["lens"][:, 0] >= 0)
