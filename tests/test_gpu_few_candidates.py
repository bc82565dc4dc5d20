"""The selection from a lower bound of the K-th best candidate (resident loop, and k_utt_few behind materialised logits) where the bound is
no help: equal logits, of all tokens or of all but a few, whose candidates all reach it.  Then the first of equal ones count, in the
order of (hypothesis, token).  And the edges of the row kernel's beams and vocabularies."""
from __future__ import annotations

import numpy as np
import pytest

import synth_inputs as S
from gpu_common import compare, gpu_decode, make_walk
from test_gpu_resident import KEYS, ST, TDT

pytestmark = pytest.mark.gpu
W64 = dict(H=64, P=64, E=64, D=32)
W640 = dict(H=640, P=640, E=640, D=64)


def _equal_logits(c, above):
    """Weights whose tokens all have the same logit, `above` of them (spread over the vocabulary) a higher one."""
    w = S.make_weights(c, 5)
    w["W_out"][: c["V"] + 1] = 0
    w["b_out"][: c["V"]] = 0.5
    if above:
        w["b_out"][np.linspace(0, c["V"] - 1, above).astype(int)] = 1.25
    w["b_out"][c["V"]] = 1.0
    return w


def _rising_logits(c):
    """Weights whose logits rise with the token index by more than float32 rounds them: the Beam best of a row are its last tokens, all in one
    of the sets that bound the K-th best, so that a pass over the candidates that reach the bound raises it by some 55 places only."""
    w = _equal_logits(c, 0)
    w["b_out"][: c["V"]] = np.linspace(-1.0, 1.0, c["V"])
    return w


def _assert_best_of_each_parent(g, w, V):
    """Tokens kept from one hypothesis at one step are its best ones, of equal logits the smallest, in the order of the slots (their scores
    differ by the logits alone, so this holds bit for bit).  Returns how many tokens were looked at."""
    order = np.lexsort((np.arange(V), -w["b_out"][:V].astype(np.float64)))
    seen = 0
    for b in range(g["n_steps"].shape[0]):
        for st in range(int(g["n_steps"][b])):
            parent, token = g["parent"][st, b], g["token"][st, b]
            for p in np.unique(parent[parent >= 0]):
                kept = token[(parent == p) & (token >= 0)]
                np.testing.assert_array_equal(kept, order[: kept.size], err_msg=f"utterance {b}, step {st}, parent {p}")
                seen += kept.size
    return seen


@pytest.mark.parametrize("above", [0, 3, 70])
@pytest.mark.parametrize("kw", [
    dict(beam=1, V=129, **W64), dict(beam=4, V=1024, **W640), dict(beam=5, V=90, algo="aes", gamma=2.3, **W64, **TDT),
    dict(beam=8, V=513, algo="aes", **W640), dict(beam=9, V=300, algo="aes", **W640), dict(beam=16, V=1024, **W640),
    dict(beam=8, V=700, prec="bf16", algo="aes", **W64, **ST, ctx=2),
], ids=lambda kw: f"k{kw['beam']}_v{kw['V']}_h{kw['H']}_{kw.get('algo', 'alsd')}")
def test_equal_logits_in_the_resident_loop(kw, above):
    import paper_2506_00185_amd as A
    c = S.custom_config(**dict(dict(B=3, T=7, T_min=3, s=3, blank_bias=0.0), **kw))
    w, L = _equal_logits(c, above), S.make_lengths(c, 7)
    enc = S.make_enc(c, L, 8)
    ref = gpu_decode(A.BeamDecoder(c, w, use_graph=False), enc, L)
    dec = A.BeamDecoder(c, w)
    r = gpu_decode(dec, enc, L)
    assert dec.last_step_loop() == "resident"
    for key in KEYS:
        np.testing.assert_array_equal(r[key], ref[key])


# Scores of the walk: float32 log-probabilities of some 20 steps, each right to 2^-22 of a value below 10 (soft-max statistics in float32);
# operands are bfloat16 but zero, so that their rounding does not come in.
@pytest.mark.parametrize("above", [0, 3, 70])
@pytest.mark.parametrize("beam,V,algo", [(1, 700, "alsd"), (4, 97, "aes"), (10, 1030, "aes"), (16, 1030, "alsd")])
def test_equal_logits_behind_materialised_ones(oracle, beam, V, algo, above):
    import paper_2506_00185_amd as A
    c = S.custom_config(B=3, T=6, T_min=3, V=V, beam=beam, algo=algo, s=2, prec="bf16", blank_bias=0.0, **W64, **ST, ctx=2)
    w, L = _equal_logits(c, above), S.make_lengths(c, 7)
    enc = S.make_enc(c, L, 8)
    g = gpu_decode(A.BeamDecoder(c, w, joint_path="materialized"), enc, L)
    o = oracle.decode(c, w, enc, L, log=True)
    tol = 20 * 10 * 2.0 ** -22
    compare(g, o, tol, tol, walk=make_walk(oracle, c, w, enc, L, g, tol))
    # (the oracle's margins are zero where candidates are equal, so that the order of equal ones is left to this)
    assert _assert_best_of_each_parent(g, w, V) >= (beam - 1) * int((L > 0).sum())


@pytest.mark.parametrize("kw", [
    dict(beam=4, V=1024, **W640), dict(beam=4, V=1024, algo="aes", **W64), dict(beam=8, V=700, algo="aes", **W640), dict(beam=10, V=1024, **W64),
    dict(beam=10, V=1023, algo="aes", **W640), dict(beam=16, V=1024, algo="aes", **W64), dict(beam=4, V=1024, prec="bf16", algo="aes", **W64, **ST, ctx=2),
], ids=lambda kw: f"k{kw['beam']}_v{kw['V']}_h{kw['H']}_{kw.get('algo', 'alsd')}")
def test_rising_logits_in_the_resident_loop(kw):
    import paper_2506_00185_amd as A
    c = S.custom_config(**dict(dict(B=3, T=7, T_min=3, s=3, blank_bias=0.0), **kw))
    w, L = _rising_logits(c), S.make_lengths(c, 7)
    enc = S.make_enc(c, L, 8)
    ref = gpu_decode(A.BeamDecoder(c, w, use_graph=False), enc, L)
    dec = A.BeamDecoder(c, w)
    r = gpu_decode(dec, enc, L)
    assert dec.last_step_loop() == "resident"
    for key in KEYS:
        np.testing.assert_array_equal(r[key], ref[key])
    assert _assert_best_of_each_parent(r, w, c["V"]) >= (c["beam"] - 1) * int((L > 0).sum())


@pytest.mark.parametrize("beam,V,algo", [(4, 8192, "alsd"), (10, 8192, "aes"), (10, 2500, "alsd"), (16, 8191, "aes")])
def test_rising_logits_behind_materialised_ones(oracle, beam, V, algo):
    """AES++ has one open row at the first step and few later on; b_out's steps of 2 / V and 2^-22 of a score keep apart."""
    import paper_2506_00185_amd as A
    c = S.custom_config(B=3, T=6, T_min=3, V=V, beam=beam, algo=algo, s=2, prec="bf16", blank_bias=0.0, **W64, **ST, ctx=2)
    w, L = _rising_logits(c), S.make_lengths(c, 7)
    enc = S.make_enc(c, L, 8)
    g = gpu_decode(A.BeamDecoder(c, w, joint_path="materialized"), enc, L)
    o = oracle.decode(c, w, enc, L, log=True)
    tol = 20 * 10 * 2.0 ** -22  # (see above)
    compare(g, o, tol, tol, walk=make_walk(oracle, c, w, enc, L, g, tol))
    assert _assert_best_of_each_parent(g, w, V) >= (beam - 1) * int((L > 0).sum())


def _bigrams(V, uniform):
    """A bigram model; uniform: equal unigrams, and of 40 contexts one successor each that differs."""
    if not uniform:
        return S.make_lm(V=V, order=2, n_target=3 * V, zipf_s=1.1, seed=5)
    ctx = np.linspace(0, V - 1, 40).astype(np.int32)
    tokens = np.concatenate([np.stack([np.arange(V), np.full(V, -1)], 1), np.stack([ctx, V - 1 - ctx], 1)]).astype(np.int32)
    n = tokens.shape[0]
    prob = np.where(np.arange(n) < V, -2.0, -1.5).astype(np.float32)
    return dict(tokens=tokens, order=(1 + (np.arange(n) >= V)).astype(np.int8), log10_prob=prob, log10_backoff=np.zeros(n, np.float32), V=V, max_order=2)


# What candidates are ranked by is not their score, or not their logit: late pruning (keys with the LM's term), early pruning (logits,
# scores with the LM's term), prefix search (a credit per hypothesis).
@pytest.mark.parametrize("blank", [1.0, 0.5, -2.0])
@pytest.mark.parametrize("kw,prune", [
    (dict(beam=4, V=1024, **W640), "late"), (dict(beam=9, V=300, algo="aes", **W64), "late"), (dict(beam=8, V=700, **W64), "late"),
    (dict(beam=4, V=1024, **W640), "early"), (dict(beam=9, V=300, algo="aes", **W64), "early"), (dict(beam=8, V=701, **W640), "early"),
    (dict(beam=5, V=129, algo="aes", aes_prefix=True, **W64), None), (dict(beam=12, V=1024, algo="aes", aes_prefix=True, **W640), None),
    (dict(beam=8, V=700, algo="aes", aes_prefix=True, **W64), "late"),
], ids=lambda x: x if not isinstance(x, dict) else f"k{x['beam']}_v{x['V']}_h{x['H']}_{x.get('algo', 'alsd')}")
def test_equal_logits_ranked_by_more_than_the_logit(kw, prune, blank):
    import paper_2506_00185_amd as A
    c = S.custom_config(**dict(dict(B=3, T=7, T_min=3, s=3, blank_bias=0.0), **kw))
    w, L = _equal_logits(c, 0), S.make_lengths(c, 7)
    w["b_out"][c["V"]] = blank
    enc = S.make_enc(c, L, 8)
    lm = A.NGramLM(_bigrams(c["V"], prune == "late")) if prune else None
    args = dict(lm=lm, lm_weight=0.3 if lm else 0.0)
    ref = gpu_decode(A.BeamDecoder(c, w, use_graph=False, lm_prune=prune or "late"), enc, L, **args)
    dec = A.BeamDecoder(c, w, lm_prune=prune or "late")
    r = gpu_decode(dec, enc, L, **args)
    assert dec.last_step_loop() == "resident"
    for key in KEYS:
        np.testing.assert_array_equal(r[key], ref[key])


@pytest.mark.parametrize("kw", [
    dict(beam=1, V=8192), dict(beam=8, V=40, algo="aes", gamma=2.3, **TDT), dict(beam=9, V=8191, algo="aes"),
    dict(beam=13, V=33, algo="aes", gamma=1.0), dict(beam=12, V=8192, algo="aes", **TDT),
    dict(beam=7, V=600, algo="aes", aes_prefix=True), dict(beam=7, V=600, aes_prefix=True),  # (k_utt_select; ALSD++ has no prefix search)
], ids=lambda kw: f"k{kw['beam']}_v{kw['V']}_{kw.get('algo', 'alsd')}_{kw.get('model', 'rnnt')}")
def test_materialised_logits_at_the_edges(oracle, kw):
    """Bars of the bf16 variant at 160 wide: see test_gpu_parity."""
    import paper_2506_00185_amd as A
    from test_gpu_parity import TIE_BF16, TOL_BF16
    c = S.custom_config(**dict(dict(B=3, T=8, T_min=1, s=2, prec="bf16", blank_bias=3.0, H=160, P=96, E=96, D=64, **ST, ctx=2), **kw))
    w = S.perturb_biases(S.make_weights(c, 5), 6)
    L = S.make_lengths(c, 7)
    enc = S.make_enc(c, L, 8)
    g = gpu_decode(A.BeamDecoder(c, w, joint_path="materialized"), enc, L)
    o = oracle.decode(c, w, enc, L, log=True)
    full, exempt = compare(g, o, TOL_BF16, TIE_BF16, walk=make_walk(oracle, c, w, enc, L, g, TOL_BF16))
    assert full + exempt == c["B"]


@pytest.mark.parametrize("kernel,kw,prune", [
    ("k_utt_few", dict(algo="aes"), None), ("k_utt_select", dict(algo="aes", aes_prefix=True), None), ("k_utt_few", dict(aes_prefix=True), None),
    ("k_utt_select", dict(), "early"), ("k_row_select", dict(), "late"),
])
def test_profile_names_the_kernel_that_ran(kernel, kw, prune):
    import paper_2506_00185_amd as A
    c = S.custom_config(**dict(dict(B=2, T=4, V=300, beam=4, s=2, prec="bf16", blank_bias=3.0, **W64, **ST, ctx=2), **kw))
    w, L = S.make_weights(c, 5), S.make_lengths(c, 7)
    lm = A.NGramLM(S.make_lm(V=300, order=2, n_target=900, zipf_s=1.1, seed=5)) if prune else None
    dec = A.BeamDecoder(c, w, joint_path="materialized", lm_prune=prune or "late")
    dec.set_profiling(True)
    gpu_decode(dec, S.make_enc(c, L, 8), L, lm=lm, lm_weight=0.3 if lm else 0.0)
    times = dec.kernel_times()
    assert {n for n in ("k_utt_few", "k_utt_select", "k_row_select") if times.get(n, (0, 0))[1]} == {kernel}
