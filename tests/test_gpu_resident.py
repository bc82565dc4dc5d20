"""The resident step loop (one launch that keeps the weights on chip, what a default decoder runs) against the per-step
launches (use_graph=False), bit for bit: both form every sum in the same order.  Shapes at the edges of its tiles: beams
of every selection form, one to three tiles of 16 slots per group, one to eight groups, widths of 64 to 640 with W_hh and
output-layer tiles that do not divide evenly, vocabularies of one column pair to the largest that fits, utterances
without frames."""
from __future__ import annotations

import numpy as np
import pytest

import synth_inputs as S
from gpu_common import compare, gpu_decode

pytestmark = pytest.mark.gpu

KEYS = ("tokens", "lens", "scores", "n_steps", "parent", "token", "merged")
W640 = dict(H=640, P=640, E=640, D=64)
ST = dict(pred="stateless")
TDT = dict(model="tdt", durations=(0, 1, 2, 3, 4))
CASES = [
    dict(B=1, beam=1, V=2, H=64, P=64, E=32, D=32),
    dict(B=1, beam=16, V=1024, s=2, **W640),
    dict(B=2, beam=5, V=1023, algo="aes", **W640),
    dict(B=3, beam=4, V=33, H=64, P=192, E=64, D=32, **TDT),
    dict(B=5, beam=8, V=700, H=576, P=128, E=64, D=32, algo="aes", gamma=2.3),
    dict(B=8, beam=2, V=513, H=320, P=320, E=64, D=32, algo="aes", aes_prefix=True),
    dict(B=13, beam=3, V=129, H=448, P=640, E=64, D=32, prec="bf16"),
    dict(B=19, beam=4, V=1024, prec="bf16", algo="aes", gamma=2.3, **W640, **TDT),
    dict(B=11, beam=9, V=512, prec="bf16", H=256, P=256, E=64, D=32),
    dict(B=20, beam=12, V=1000, s=1, **W640),
    dict(B=40, beam=1, V=1024, **W640),
    dict(B=50, beam=4, V=90, **W640),
    # lengths that let later slot tiles run empty well before the first
    dict(B=40, beam=8, V=300, T=40, T_min=1, **W640),
    dict(B=17, beam=13, V=300, T=40, T_min=1, prec="bf16", **W640),
    # stateless decoders: every context length, both precisions, up to a full tile of slots per group
    dict(B=1, beam=3, V=2, H=64, P=64, E=64, D=32, **ST, ctx=1),
    dict(B=8, beam=4, V=1024, prec="bf16", algo="aes", s=2, **W640, **ST, ctx=2),
    dict(B=8, beam=13, V=1000, prec="bf16", **W640, **ST, ctx=3),
    dict(B=1, beam=16, V=1024, **W640, **ST, ctx=3),
    dict(B=8, beam=10, V=700, algo="aes", **W640, **ST, ctx=1),
    dict(B=16, beam=8, V=257, H=448, P=64, E=64, D=32, **ST, ctx=4),
    dict(B=23, beam=5, V=1023, **W640, **ST, ctx=2),
    dict(B=30, beam=4, V=129, prec="bf16", H=192, P=192, E=192, D=32, algo="aes", gamma=2.3, **ST, ctx=4, **TDT),
    # the per-step launches fold the blank and duration columns into the token columns' blocks (V % 32 == 0, 640 wide, more than
    # 256 blocks): the same sums in the same order, one to three tiles of slots, every precision and network
    dict(B=15, beam=12, V=1024, **W640),
    dict(B=29, beam=8, V=1024, algo="aes", **W640, **TDT),
    dict(B=128, beam=2, V=512, s=2, **W640),
    dict(B=15, beam=12, V=1024, prec="bf16", **W640),
    dict(B=57, beam=4, V=1024, prec="bf16", **W640, **TDT),
    dict(B=64, beam=2, V=1024, **W640, **ST, ctx=2),
    dict(B=57, beam=1, V=1024, prec="bf16", **W640, **ST, ctx=1, **TDT),
    # split products of unequal widths, one of them 640
    dict(B=9, beam=4, V=90, H=384, P=640, E=64, D=32), dict(B=5, beam=8, V=700, H=640, P=320, E=64, D=32, **TDT),
    dict(B=17, beam=9, V=300, H=512, P=384, E=64, D=32), dict(B=8, beam=8, V=513, H=320, P=64, E=64, D=32, **ST, ctx=2),
]


@pytest.mark.parametrize("kw", CASES, ids=lambda kw: f"b{kw['B']}_k{kw['beam']}_v{kw['V']}_h{kw['H']}_p{kw['P']}_{kw.get('prec', 'f32')}_ctx{kw.get('ctx', 0)}")
def test_resident_loop_equals_the_per_step_launches(kw):
    import paper_2506_00185_amd as A
    c = S.custom_config(**dict(dict(T=17, T_min=3, s=3, blank_bias=3.0), **kw))
    w = S.perturb_biases(S.make_weights(c, 5), 6)
    L = S.make_lengths(c, 7)
    if c["B"] > 2:
        L[1] = 0
    enc = S.make_enc(c, L, 8)
    plain = A.BeamDecoder(c, w, use_graph=False)
    ref = gpu_decode(plain, enc, L)
    assert plain.last_step_loop() == "launches"
    dec = A.BeamDecoder(c, w)
    for _ in range(2):
        r = gpu_decode(dec, enc, L)
        assert dec.last_step_loop() == "resident"
        for key in KEYS:
            np.testing.assert_array_equal(r[key], ref[key])


W192 = dict(H=192, P=192, E=64, D=32)


@pytest.mark.parametrize("loop,kw", [
    ("graph", dict(B=32, beam=12, V=512, **W192)), ("graph", dict(B=33, beam=8, V=512, **W192)),      # three tiles, float32
    ("resident", dict(B=33, beam=8, V=513, **W192)), ("resident", dict(B=33, beam=8, V=90, prec="bf16", **W192)),
    ("graph", dict(B=9, beam=9, V=385, **W192)), ("resident", dict(B=9, beam=9, V=384, **W192)),      # two tiles, wide beams
    ("resident", dict(B=9, beam=8, V=385, **W192)), ("resident", dict(B=8, beam=9, V=385, **W192)),
    ("graph", dict(B=9, beam=9, V=513, prec="bf16", **W192)), ("resident", dict(B=9, beam=9, V=512, prec="bf16", **W192)),
    ("resident", dict(B=9, beam=9, V=600, **dict(W192, P=384))),
    ("graph", dict(B=8, beam=9, V=90, **dict(W192, H=128), **ST, ctx=1)), ("resident", dict(B=8, beam=8, V=90, **dict(W192, H=128), **ST, ctx=1)),
    ("graph", dict(B=1, beam=9, V=90, prec="bf16", **W192, **ST, ctx=1)), ("resident", dict(B=2, beam=9, V=90, prec="bf16", **W192, **ST, ctx=1)),
    ("resident", dict(B=1, beam=9, V=90, **W192, **ST, ctx=1)),
])
def test_loop_that_decodes_a_batch_on_either_side_of_a_rule(loop, kw):
    import paper_2506_00185_amd as A
    c = S.custom_config(**dict(dict(T=8, T_min=3, s=2, blank_bias=3.0), **kw))
    w = S.perturb_biases(S.make_weights(c, 5), 6)
    L = S.make_lengths(c, 7)
    enc = S.make_enc(c, L, 8)
    ref = gpu_decode(A.BeamDecoder(c, w, use_graph=False), enc, L)
    dec = A.BeamDecoder(c, w)
    r = gpu_decode(dec, enc, L)
    assert dec.last_step_loop() == loop
    if c["B"] * c["beam"] <= 256:
        for key in KEYS:
            np.testing.assert_array_equal(r[key], ref[key])


W256 = dict(H=256, P=256, E=64, D=32)


@pytest.mark.parametrize("loop,kw", [
    ("resident", dict(B=25, beam=9, V=512, **W256)), ("resident", dict(B=17, beam=12, V=29, **W256)),     # three tiles, float32
    ("resident", dict(B=33, beam=8, V=90, **dict(W256, H=512, P=512))), ("resident", dict(B=9, beam=9, V=600, **W256)),
    ("resident", dict(B=25, beam=10, V=1000, prec="bf16", **dict(W256, H=320, P=320))),
    ("resident", dict(B=9, beam=9, V=700, **dict(W256, P=192))), ("graph", dict(B=9, beam=9, V=700, **dict(W192, P=128))),
    ("graph", dict(B=1, beam=9, V=90, prec="bf16", **dict(W256, H=320), **ST, ctx=1)),
    ("resident", dict(B=1, beam=9, V=90, prec="bf16", **dict(W256, H=384), **ST, ctx=1)),
])
def test_loop_of_wide_and_narrow_decoders_with_several_tiles(loop, kw):
    test_loop_that_decodes_a_batch_on_either_side_of_a_rule(loop, kw)


@pytest.mark.parametrize("prune,rule,beam,B,more", [("late", 4, 8, 9, {}), ("early", 3, 4, 17, {}), ("late", 3, 11, 4, {}),
                                                    ("late", 4, 6, 10, dict(ST, ctx=2)),
                                                    # up to four hypotheses of more than 512 tokens: two waves per row
                                                    ("late", 4, 4, 1, dict(V=1024)), ("late", 3, 2, 9, dict(V=515)),
                                                    ("early", 4, 3, 2, dict(V=777))])
def test_resident_loop_with_an_lm(prune, rule, beam, B, more):
    import paper_2506_00185_amd as A
    c = S.custom_config(**dict(dict(B=B, T=15, T_min=4, s=3, beam=beam, V=300, blank_bias=3.0, **W640), **more))
    w = S.perturb_biases(S.make_weights(c, 15), 16)
    L = S.make_lengths(c, 17)
    enc = S.make_enc(c, L, 18)
    lm = A.NGramLM(S.make_lm(V=c["V"], order=4, n_target=20000, zipf_s=1.1, seed=19))
    kw = dict(lm_rule=rule, lm_prune=prune)
    ref = gpu_decode(A.BeamDecoder(c, w, use_graph=False, **kw), enc, L, lm=lm, lm_weight=0.3)
    dec = A.BeamDecoder(c, w, **kw)
    r = gpu_decode(dec, enc, L, lm=lm, lm_weight=0.3)
    assert dec.last_step_loop() == "resident"
    for key in KEYS:
        np.testing.assert_array_equal(r[key], ref[key])


def test_resident_loop_that_gives_up_is_replaced_by_the_per_step_launches():
    import paper_2506_00185_amd as A
    c = S.custom_config(B=9, T=12, T_min=4, s=3, beam=4, V=300, blank_bias=3.0, **W640)
    w = S.make_weights(c, 25)
    L = S.make_lengths(c, 27)
    enc = S.make_enc(c, L, 28)
    ref = gpu_decode(A.BeamDecoder(c, w, use_graph=False), enc, L)
    dec = A.BeamDecoder(c, w)
    dec.debug_set_spin_limit(1)  # (its blocks then wait in vain for one more)
    for _ in range(2):
        r = gpu_decode(dec, enc, L)
        assert dec.last_step_loop() == "graph"
        for key in KEYS:
            np.testing.assert_array_equal(r[key], ref[key])
    dec.debug_set_spin_limit(1 << 22)
    r = gpu_decode(dec, enc, L)
    np.testing.assert_array_equal(r["tokens"], ref["tokens"])


def test_resident_loop_is_tried_again_after_launches_that_gave_up():
    import paper_2506_00185_amd as A
    c = S.custom_config(B=2, T=5, D=32, H=64, P=64, E=64, V=30, beam=2, s=2)
    w = S.make_weights(c, 25)
    L = S.make_lengths(c, 27)
    enc = S.make_enc(c, L, 28)
    dec = A.BeamDecoder(c, w)

    def loops(n):
        out = []
        for _ in range(n):
            gpu_decode(dec, enc, L)
            out.append(dec.last_step_loop())
        return out

    assert loops(1) == ["resident"]
    dec.debug_set_spin_limit(1)
    assert loops(1 + 4 + 1 + 8 + 1) == ["graph"] * 15  # three launches give up
    dec.debug_set_spin_limit(1 << 22)
    assert loops(16 + 2) == ["graph"] * 16 + ["resident"] * 2
    dec.debug_set_spin_limit(1)
    assert loops(1) == ["graph"]
    dec.debug_set_spin_limit(1 << 22)
    assert loops(4 + 1) == ["graph"] * 4 + ["resident"]  # the count had started anew


@pytest.mark.parametrize("kw", [{}, dict(prec="bf16"), dict(ST, ctx=1)], ids=["lstm", "bf16", "stateless"])
def test_decoder_without_memory_for_the_resident_loop_uses_the_per_step_launches(kw):
    import paper_2506_00185_amd as A
    c = S.custom_config(B=3, T=9, D=32, H=64, P=64, E=64, V=30, beam=3, s=2, **kw)
    w = S.make_weights(c, 25)
    L = S.make_lengths(c, 27)
    enc = S.make_enc(c, L, 28)
    dec = A.BeamDecoder(c, w)
    ref = gpu_decode(dec, enc, L)
    for alloc, loop in [(i, "graph") for i in range(5)] + [(100, "resident"), (-1, "resident")]:
        dec.debug_rebuild_resident(alloc)
        r = gpu_decode(dec, enc, L)
        assert dec.last_step_loop() == loop
        for key in KEYS:
            np.testing.assert_array_equal(r[key], ref[key])


@pytest.mark.parametrize("kw", [dict(beam=12), dict(beam=12, prec="bf16", B=24), dict(beam=4, B=8), dict(beam=4, B=8, **ST, ctx=2)],
                         ids=["straddles_two_tiles", "bf16", "one_tile", "stateless"])
@pytest.mark.parametrize("step", [0, 1, 5])
def test_logits_that_do_not_come_end_the_resident_loop_as_a_whole(kw, step):
    """The hypotheses of an utterance lie in two tiles of slots and the logits of the second never come: the block that selects
    for it has some rows and not others.  Every wave of it ends, and what the per-step launches then decode is the result."""
    import paper_2506_00185_amd as A
    c = S.custom_config(**dict(dict(B=16, T=12, T_min=8, s=3, V=300, blank_bias=3.0, **W640), **kw))
    w = S.make_weights(c, 35)
    L = S.make_lengths(c, 37)
    enc = S.make_enc(c, L, 38)
    ref = gpu_decode(A.BeamDecoder(c, w, use_graph=False), enc, L)
    dec = A.BeamDecoder(c, w)
    dec.debug_stall_resident(step)
    r = gpu_decode(dec, enc, L)
    assert dec.last_step_loop() == "graph"
    for key in KEYS:
        np.testing.assert_array_equal(r[key], ref[key])
    dec.debug_stall_resident(-1)
    for _ in range(2):
        r = gpu_decode(dec, enc, L)
        for key in KEYS:
            np.testing.assert_array_equal(r[key], ref[key])


@pytest.mark.parametrize("h,B,beam", [(64, 3, 4), (320, 9, 5), (640, 5, 9), (640, 17, 4)])
def test_split_products_over_a_wide_range_of_scales(oracle, h, B, beam):
    """Outputs of the prediction and encoder projections times powers of two from 2^-6 to 2^6, columns of the output layer by their
    inverses: the same function (ReLU is homogeneous), but rows, columns and activations of sizes far apart, which the split into
    float16 has to scale.  The tolerance is that of float32 models: a value down to 2^-28 of the largest keeps 23 bits."""
    import paper_2506_00185_amd as A
    c = S.custom_config(B=B, T=12, T_min=6, s=3, V=90, beam=beam, blank_bias=3.0, H=h, P=h, E=64, D=64)
    w = {k: np.array(v) for k, v in S.make_weights(c, 75).items()}
    L = S.make_lengths(c, 77)
    enc = S.make_enc(c, L, 78)
    f = (2.0 ** np.random.default_rng(79).integers(-6, 7, h)).astype(np.float32)
    for k in ("W_enc", "W_pred"):
        w[k] = w[k] * f[:, None]
    for k in ("b_enc", "b_pred"):
        w[k] = w[k] * f
    w["W_out"] = w["W_out"] / f[None, :]
    w["W_hh"][5] = 0.0         # a row without weights
    w["W_hh"][7] *= 2.0 ** -30
    dec = A.BeamDecoder(c, w)
    g = gpu_decode(dec, enc, L)
    assert dec.last_step_loop() == "resident"
    o = oracle.decode(c, w, enc, L, log=True)
    full, exempt = compare(g, o, 1e-3, 1e-4)
    assert full >= (c["B"] + 1) // 2
    ref = gpu_decode(A.BeamDecoder(c, w, use_graph=False), enc, L)
    for key in KEYS:
        np.testing.assert_array_equal(g[key], ref[key])


@pytest.mark.parametrize("loop,kw", [
    ("resident", dict(B=3, beam=4, V=90, H=64, P=64, E=64)), ("resident", dict(B=9, beam=5, V=90, **dict(W640, H=320, P=448))),
    ("resident", dict(B=5, beam=4, V=90, **W640, **TDT)),
    # the per-step launches would fold the blank and duration columns
    ("resident", dict(B=57, beam=4, V=1024, T=6, **W640, **TDT)),
    ("launches", dict(B=57, beam=4, V=1024, T=6, **W640, **TDT)), ("launches", dict(B=3, beam=4, V=90, H=96, P=96, E=64)),
    ("launches", dict(B=9, beam=5, V=90, **dict(W640, H=320, P=448))),
    ("resident", dict(B=3, beam=4, V=90, **W640, **ST, ctx=2)),
])
def test_weights_that_are_not_finite(oracle, loop, kw):
    """A weight of -inf closes what it leads to (a token, a duration, a unit of the joint, a forget gate) and a token whose row holds a
    NaN is no candidate: the same as finite weights with biases of -inf or -1e30 there (the oracle's)."""
    import paper_2506_00185_amd as A
    c = S.custom_config(**dict(dict(T=12, T_min=3, s=3, blank_bias=3.0, D=64), **kw))
    w = {k: np.array(v) for k, v in S.make_weights(c, 91).items()}
    L = S.make_lengths(c, 92)
    enc = S.make_enc(c, L, 93)
    V, P, lstm = c["V"], c["P"], c["pred"] == "lstm"
    on, off, unit, gate = 5, 9, 7, 3   # joint: a unit that is always active, one to be closed; LSTM: a positive unit, a forget gate
    w["W_enc"][on] = w["W_pred"][on] = 0.0
    w["b_pred"][on] = 2.0
    w["W_out"][:, on] = 0.0
    closed = [V // 2, V - 1] + ([V + 2] if c["durations"] else [])  # two tokens, a duration
    w["b_out"][closed] = 6.0           # (they would win often)
    if lstm:
        w["b_ih"][2 * P + unit] = 20.0  # cell candidate and gates of the unit: its state stays positive
        w["b_ih"][3 * P + unit] = w["b_ih"][unit] = 5.0
    ref = {k: v.copy() for k, v in w.items()}
    w["W_out"][closed, on] = -np.inf
    if loop == "resident":             # (the per-step launches add NaN logits up)
        w["W_out"][V // 3, off] = np.nan
        ref["b_out"][V // 3] = -np.inf
    ref["b_out"][closed] = -np.inf
    if lstm:
        w["W_hh"][P + gate, unit] = w["W_pred"][off, unit] = -np.inf
        ref["b_ih"][P + gate] = ref["b_pred"][off] = -1e30
    dec = A.BeamDecoder(c, w, use_graph=loop == "resident")
    g = gpu_decode(dec, enc, L)
    assert dec.last_step_loop() == loop
    o = oracle.decode(c, ref, enc, L, log=True)
    full, exempt = compare(g, o, 1e-3, 1e-4)
    assert full >= (c["B"] + 1) // 2
    assert not np.isin(g["tokens"], closed[:2] + ([V // 3] if loop == "resident" else [])).any()


@pytest.mark.parametrize("h,B,beam,apart,huge", [(320, 9, 5, 0, 0), (640, 5, 9, 13, 0), (640, 17, 4, 0, 0), (576, 3, 4, 13, 0), (640, 3, 4, 0, 2.0 ** 90),
                                                 (320, 3, 4, 13, 2.0 ** -100)])
def test_split_products_of_rows_with_outliers(oracle, h, B, beam, apart, huge):
    """Units up to 2^26 apart, as above, or in every row of W_out a weight 2^26 times the others on a unit that is never active; in those of
    W_pred and W_hh too: the same function.  23 bits of every operand remain: the tolerance is that of float32 models.  huge: rows that
    are not split at all."""
    import paper_2506_00185_amd as A
    c = S.custom_config(B=B, T=12, T_min=6, s=3, V=90, beam=beam, blank_bias=3.0, H=h, P=h, E=64, D=64)
    w = {k: np.array(v) for k, v in S.make_weights(c, 81).items()}
    L = S.make_lengths(c, 82)
    enc = S.make_enc(c, L, 83)
    off, silent, P = 3, 5, h
    w["b_pred"][off] = -1e9                      # joint: ReLU gives 0
    w["b_ih"][3 * P + silent] = -1e9             # LSTM: the output gate is shut
    f = (2.0 ** np.random.default_rng(84).integers(-apart, apart + 1, h)).astype(np.float32)
    f[off] = 1.0
    for k in ("W_enc", "W_pred"):
        w[k] = w[k] * f[:, None]
    for k in ("b_enc", "b_pred"):
        w[k] = w[k] * f
    w["W_out"] = w["W_out"] / f[None, :]
    ref = {k: np.array(v) for k, v in w.items()}
    if not apart:
        w["W_out"][:, off] = np.float32(max(huge, 2.0 ** 26 * np.abs(w["W_out"]).mean()))
    w["W_pred"][:, silent] *= 2.0 ** 26
    w["W_hh"][:, silent] = np.float32(2.0 ** 26 * np.abs(w["W_hh"]).mean())
    if huge and huge < 1.0:
        w["W_hh"][P + 7] = ref["W_hh"][P + 7] = huge
    dec = A.BeamDecoder(c, w)
    g = gpu_decode(dec, enc, L)
    assert dec.last_step_loop() == "resident"
    o = oracle.decode(c, ref, enc, L, log=True)
    full, exempt = compare(g, o, 1e-3, 1e-4)
    assert full >= (c["B"] + 1) // 2
    ref = gpu_decode(A.BeamDecoder(c, w, use_graph=False), enc, L)
    for key in KEYS:
        np.testing.assert_array_equal(g[key], ref[key])


@pytest.mark.parametrize("h,p,more", [(320, 320, {}), (640, 640, {}), (448, 640, {}), (640, 640, dict(ST, ctx=2)),
                                      # per-step launches: four waves a block, halves of k
                                      (352, 352, {}), (384, 384, dict(use_graph=False))])
def test_error_of_split_products_against_64_bits(oracle, h, p, more):
    """Scores of decodes with logits of some hundreds, whose errors are those of the products, against the oracle's 64 bits: no larger
    than with float32 instructions, which the same decoder runs when a token that a bias has closed is closed by a weight without a
    split.  Bound: 4 standard errors of the ratio of the two (0.02 to 0.03 at 20 decodes of 16 utterances) above 1."""
    import paper_2506_00185_amd as A
    square, n = np.zeros(2), 0
    more = dict(more)
    use_graph = more.pop("use_graph", True)
    for seed in range(100, 120):
        c = S.custom_config(**dict(dict(B=16, T=3, T_min=3, s=2, V=300, beam=8, blank_bias=0.0, H=h, P=p, E=64, D=64), **more))
        w = {k: np.array(v) for k, v in S.make_weights(c, seed).items()}
        w["W_out"] = w["W_out"] * 100.0
        w["W_enc"][0] = w["W_pred"][0] = 0.0
        w["b_pred"][0] = 1.0                    # a unit that is always active
        w["b_out"][c["V"] - 1] = -1e30
        ref = {k: np.array(v) for k, v in w.items()}
        ref["W_out"][c["V"] - 1, 0] = -np.inf
        L = S.make_lengths(c, seed + 1)
        enc = S.make_enc(c, L, seed + 2)
        o = oracle.decode(c, w, enc, L)
        lists = [[{tuple(r["tokens"][b, j, :l]): r["scores"][b, j] for j, l in enumerate(r["lens"][b]) if l >= 0} for b in range(c["B"])]
                 for r in (o, *[gpu_decode(A.BeamDecoder(c, x, use_graph=use_graph), enc, L, want_tree=False) for x in (w, ref)])]
        for want, split, plain in zip(*lists):
            for k in want.keys() & split.keys() & plain.keys():
                square += (split[k] - want[k]) ** 2, (plain[k] - want[k]) ** 2
                n += 1
    ratio = float(np.sqrt(square[0] / square[1]))
    print("error, split over float32:", round(ratio, 3), "of", n, "scores")
    assert n > 1000 and ratio <= 1.1


@pytest.mark.parametrize("h,p,more", [(64, 64, {}), (256, 256, {}), (640, 128, dict(V=700)), (192, 640, dict(B=9)), (256, 64, ST),
                                      (96, 160, {}), (128, 128, dict(B=10, beam=10, V=500))])
def test_narrow_decoders_multiply_in_float32(h, p, more):
    """... as they do with a weight that has no split: a token that a bias has closed anyhow is closed by such a weight too."""
    import paper_2506_00185_amd as A
    c = S.custom_config(**dict(dict(B=5, T=12, T_min=6, s=3, V=90, beam=4, blank_bias=3.0, H=h, P=p, E=64, D=64, ctx=2 if more is ST else 0), **more))
    w = {k: np.array(v) for k, v in S.make_weights(c, 75).items()}
    w["W_enc"][0] = w["W_pred"][0] = 0.0
    w["b_pred"][0] = 1.0                        # a unit that is always active
    w["b_out"][c["V"] - 1] = -1e30
    ref = {k: np.array(v) for k, v in w.items()}
    ref["W_out"][c["V"] - 1, 0] = -np.inf
    L = S.make_lengths(c, 77)
    enc = S.make_enc(c, L, 78)
    got, want = [gpu_decode(A.BeamDecoder(c, x), enc, L) for x in (w, ref)]
    for key in KEYS:
        np.testing.assert_array_equal(got[key], want[key])


@pytest.mark.parametrize("kw", [dict(B=5, beam=4), dict(B=17, beam=9, prec="bf16"), dict(B=8, beam=4, **ST, ctx=2)], ids=["lstm", "bf16", "stateless"])
def test_groups_that_do_not_lie_on_one_xcd(kw):
    """Their hand-over stores are written through: the same words arrive."""
    import paper_2506_00185_amd as A
    c = S.custom_config(**dict(dict(T=17, T_min=3, s=3, V=300, blank_bias=3.0, **W640), **kw))
    w = S.make_weights(c, 45)
    L = S.make_lengths(c, 47)
    enc = S.make_enc(c, L, 48)
    dec = A.BeamDecoder(c, w)
    ref = gpu_decode(dec, enc, L)
    groups, local = dec.debug_resident_groups()
    assert groups == local == min(c["B"], 8)  # (the other decode hands over through the L2)
    dec.debug_stall_resident(-2)
    r = gpu_decode(dec, enc, L)
    assert dec.last_step_loop() == "resident"
    assert dec.debug_resident_groups() == (groups, 0)
    for key in KEYS:
        np.testing.assert_array_equal(r[key], ref[key])


def test_resident_loop_does_not_start_beside_a_single_launch_loop():
    """The single-launch loop's blocks wait for each other too.  One of another handle waits on its stream, behind 40 ms of other
    work, to begin."""
    import torch
    import paper_2506_00185_amd as A
    c = S.custom_config(B=4, T=9, D=64, H=64, P=64, E=64, V=40, beam=4, s=2)
    w = S.make_weights(c, 45)
    L = S.make_lengths(c, 47)
    enc = S.make_enc(c, L, 48)
    dec, single = A.BeamDecoder(c, w), A.BeamDecoder(c, w, persistent=True)
    ref = gpu_decode(dec, enc, L)
    assert dec.last_step_loop() == "resident"
    x, n = torch.as_tensor(enc).cuda(), torch.as_tensor(L).cuda()
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        torch.cuda._sleep(80_000_000)
        single.decode(x, n)
    dec.decode(x, n)
    r = dec.results()
    assert dec.last_step_loop() == "graph" and single.last_step_loop() == "single launch"
    r1 = single.results()
    for key in ("tokens", "lens", "scores", "n_steps"):
        np.testing.assert_array_equal(r[key], ref[key])
        np.testing.assert_array_equal(r1[key], ref[key])
    gpu_decode(dec, enc, L)
    assert dec.last_step_loop() == "resident"


def test_nan_of_all_ones_in_the_encoder_output():
    """The bit pattern that marks empty places of the hand-over arrays, as data: the decode ends and reports it, in this loop."""
    import torch
    import paper_2506_00185_amd as A
    c = S.custom_config(B=9, T=10, V=90, beam=4, s=2, **W640)
    w = S.make_weights(c, 65)
    L = S.make_lengths(c, 67)
    enc = S.make_enc(c, L, 68)
    dec = A.BeamDecoder(c, w)
    n = torch.as_tensor(L).cuda()
    x = torch.as_tensor(enc).cuda()
    x.view(torch.int32)[3, 2, 5] = -1
    dec.decode(x, n)
    assert dec.results(check=False)["rc"] == -4 and dec.last_step_loop() == "resident"
    gpu_decode(dec, enc, L)
    assert dec.last_step_loop() == "resident"


def test_threads_that_decode_on_streams_of_their_own():
    """Two handles for the resident loop, one for the single-launch loop and one with a launch per step, each in a thread and on a
    stream of its own: whatever loop a decode finds free, the results are those of the same decode alone."""
    import threading
    import torch
    import paper_2506_00185_amd as A
    c = S.custom_config(B=6, T=12, D=64, H=192, P=192, E=64, V=150, beam=4, s=2, blank_bias=3.0)
    w = S.make_weights(c, 55)
    L = S.make_lengths(c, 57)
    enc = S.make_enc(c, L, 58)
    ref = gpu_decode(A.BeamDecoder(c, w, use_graph=False), enc, L)
    x, n = torch.as_tensor(enc).cuda(), torch.as_tensor(L).cuda()
    handles = [A.BeamDecoder(c, w), A.BeamDecoder(c, w), A.BeamDecoder(c, w, persistent=True), A.BeamDecoder(c, w, use_graph=False)]
    torch.cuda.synchronize()
    out = [[] for _ in handles]

    def work(i):
        s = torch.cuda.Stream()
        for _ in range(12):
            handles[i].decode(x, n, stream=s)
            out[i].append((handles[i].results(), handles[i].last_step_loop()))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(handles))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for i, results in enumerate(out):
        assert len(results) == 12
        for r, loop in results:
            assert loop in (("resident", "graph"), ("resident", "graph"), ("single launch",), ("launches",))[i]
            for key in ("tokens", "lens", "scores", "n_steps"):
                np.testing.assert_array_equal(r[key], ref[key])


@pytest.mark.parametrize("B,beam", [(32, 12), (29, 8), (57, 1), (113, 2)])
def test_folded_columns_that_take_a_tile_more_than_there_is_room_for(B, beam):
    """Eight durations and the largest vocabulary: nine columns beside 64 tiles of tokens and 40 of the projection.  Fewer blocks of a
    group select then (three or two instead of four, for up to five utterances each), and the loop decodes the batch all the same."""
    import paper_2506_00185_amd as A
    c = S.custom_config(B=B, beam=beam, V=1024, T=17, T_min=3, s=2, model="tdt", durations=(0, 1, 2, 3, 4, 5, 6, 7), blank_bias=3.0, **W640)
    w = S.perturb_biases(S.make_weights(c, 5), 6)
    L = S.make_lengths(c, 7)
    L[1] = 0
    enc = S.make_enc(c, L, 8)
    ref = gpu_decode(A.BeamDecoder(c, w, use_graph=False), enc, L)
    dec = A.BeamDecoder(c, w)
    for _ in range(2):
        r = gpu_decode(dec, enc, L)
        assert dec.last_step_loop() == "resident"
        for key in KEYS:
            np.testing.assert_array_equal(r[key], ref[key])
