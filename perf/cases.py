"""Workloads by which the speed of the batched Transducer beam search is judged.

A case is one batch of utterances of one decoder: ``prepare`` makes what a serving program holds before a batch arrives
(decoder handle, language model, the encoder output and the lengths in device memory), ``run`` is what it then does with
the batch: ``BeamDecoder.decode`` and ``BeamDecoder.results``.  The shapes are those of the framework's own workloads
(``synth_inputs.CONFIGS``), of its batch and beam sweeps (batches 1 to 32, beams 1 to 12) and of its tests; weights, encoder
output and n-gram models are synthetic, as everywhere in this repository.

Fields: ``model`` rnnt / tdt, ``pred`` lstm / stateless, ``algo`` alsd / aes, ``prec`` f32 / bf16 (operands of the joint),
``batch`` utterances of ``frames_min`` to ``frames`` encoder frames (80 ms each), ``beam`` hypotheses per utterance,
``enc`` encoder width, ``hidden`` width of the joint, the prediction network and its embedding, ``vocab`` tokens,
``symbols`` most tokens per frame, ``margin`` prune margin of AES++ (0: off), ``ngrams`` size of the 4-gram LM (0: none).
"""
from __future__ import annotations

import functools

import numpy as np
import torch

import paper_2506_00185_amd as A
import synth_inputs as S

LM_WEIGHT = 0.3
DURATIONS = (0, 1, 2, 3, 4)
#: hypotheses of a batch of the LSTM decoders, and of the stateless ones
MOST_ROWS = {"lstm": 256, "stateless": 1280}


def case(name, batch, frames, frames_min, beam, model="rnnt", pred="lstm", algo="alsd", prec="f32", enc=1024, hidden=640,
         vocab=1024, symbols=5, margin=0.0, ngrams=0):
    c = dict(model=model, pred=pred, algo=algo, prec=prec, batch=batch, frames=frames, frames_min=frames_min, beam=beam,
             enc=enc, hidden=hidden, vocab=vocab, symbols=symbols, margin=margin, ngrams=ngrams)
    return dict(c, name=name) if name else c


def listed():
    return [
        # a toy decoder on one short utterance: latency of the step loop and of the call itself
        case("tiny_b1_beam4", 1, 20, 20, 4, enc=64, hidden=64, vocab=16, symbols=3),
        # one utterance at a time, as an interactive service has it
        case("single_b1_beam4", 1, 125, 125, 4),
        # small batch of short commands on the TDT model, beam of the published batch sweeps, lengths ragged
        case("tdt_b4_beam6_ragged", 4, 77, 23, 6, model="tdt", algo="alsd", symbols=2),
        # a decoder of other widths, odd batch and vocabulary, frame-synchronous
        case("narrow_aes_b7_beam5", 7, 90, 31, 5, algo="aes", enc=512, hidden=320, vocab=500),
        # greedy search over a full batch
        case("greedy_b32", 32, 125, 125, 1),
        # the headline workload, and the same with the joint's operands in bfloat16
        case("rnnt_b32_beam4", 32, 125, 125, 4),
        case("rnnt_b32_beam4_bf16", 32, 125, 125, 4, prec="bf16"),
        # batch 16 with a wide beam (rescoring needs long n-best lists), lengths ragged
        case("rnnt_b16_beam12_ragged", 16, 125, 40, 12),
        # TDT, frame-synchronous with pruning, utterances of 4 to 20 seconds
        case("tdt_aes_b64_ragged", 64, 250, 50, 4, model="tdt", algo="aes", symbols=2, margin=2.3),
        # shallow fusion with a 4-gram model
        case("lm_b32_beam8", 32, 125, 125, 8, ngrams=500_000),
        # stateless decoder of a small batch: joint fused with the selection
        case("stateless_b8_beam4_bf16", 8, 125, 61, 4, pred="stateless", algo="aes", prec="bf16", symbols=2),
        # large vocabulary, large batch, stateless prediction network in bfloat16
        case("stateless_b128_v8192", 128, 250, 250, 10, pred="stateless", algo="aes", prec="bf16", vocab=8192, symbols=2),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    """A batch of 1 to 64 (stateless: 128) utterances of up to 250 frames at beams 1 to 12, in the mixes of options that
    the listed cases have."""
    kind = rng.choice(["rnnt", "rnnt", "rnnt", "bf16", "tdt", "tdt", "lm", "narrow", "stateless"])
    beam = rng.choice([1, 2, 3, 4, 4, 5, 6, 8, 8, 10, 12])
    rows = MOST_ROWS["stateless" if kind == "stateless" else "lstm"]
    batch = _log_int(rng, 1, min(128 if kind == "stateless" else 64, rows // beam))
    frames = _log_int(rng, 20, 250)
    ragged = rng.random() < 0.6
    frames_min = max(1, int(frames * rng.uniform(0.2, 0.9))) if ragged else frames
    algo = rng.choice(["alsd", "alsd", "aes"])
    c = dict(algo=algo)
    if kind == "bf16":
        c.update(prec="bf16")
    elif kind == "tdt":
        c.update(model="tdt", symbols=2, margin=rng.choice([0.0, 2.3]) if algo == "aes" else 0.0)
    elif kind == "lm":
        c.update(ngrams=500_000)
    elif kind == "narrow":
        c.update(enc=512, hidden=rng.choice([128, 256, 320, 512]), vocab=rng.choice([29, 128, 257, 500, 1000]))
    elif kind == "stateless":
        c.update(pred="stateless", prec="bf16", symbols=2, vocab=rng.choice([1024, 4096, 8192]))
    return case(None, batch, frames, frames_min, beam, **c)


@functools.lru_cache(maxsize=2)
def _language_model(vocab, ngrams):
    """The n-gram model is an asset of the program: loaded once, used by every decoder."""
    return A.NGramLM(S.make_lm(vocab, 4, ngrams, 1.1, 4003))


def _config(c):
    return S.custom_config(
        model=c["model"], pred=c["pred"], prec=c["prec"], B=c["batch"], T=c["frames"], T_min=c["frames_min"], D=c["enc"],
        H=c["hidden"], P=c["hidden"], E=c["hidden"], V=c["vocab"], durations=DURATIONS if c["model"] == "tdt" else (),
        beam=c["beam"], s=c["symbols"], algo=c["algo"], gamma=c["margin"] or float("inf"),
        blank_bias=2.0 if c["vocab"] < 64 else 3.0, ctx=2 if c["pred"] == "stateless" else 0)


def prepare(c, seed):
    cfg = _config(c)
    decoder = A.BeamDecoder(cfg, S.make_weights(cfg, seed))
    lengths = torch.as_tensor(S.make_lengths(cfg, seed + 1)).cuda()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed + 2)
    enc = torch.randn(cfg["B"], cfg["T"], cfg["D"], generator=gen, device="cuda", dtype=torch.float32)
    enc *= (torch.arange(cfg["T"], device="cuda")[None, :] < lengths[:, None])[:, :, None]  # zero behind each length
    lm = _language_model(c["vocab"], c["ngrams"]) if c["ngrams"] else None
    return dict(decoder=decoder, enc=enc, lengths=lengths, lm=lm)


def run(state):
    state["decoder"].decode(state["enc"], state["lengths"], lm=state["lm"], lm_weight=LM_WEIGHT if state["lm"] else 0.0)
    r = state["decoder"].results()
    return dict(tokens=r["tokens"], lens=r["lens"], scores=r["scores"], n_steps=r["n_steps"])


def _steps(c):
    """Steps of the search, from the lengths: these models emit close to ``symbols`` tokens per frame (RNN-T); with
    durations a step advances about one frame."""
    return c["frames"] * (1.0 if c["model"] == "tdt" else 0.9 * (c["symbols"] + 1))


def work(c):
    H, V, n_out = c["hidden"], c["vocab"], c["vocab"] + 1 + (len(DURATIONS) if c["model"] == "tdt" else 0)
    total_frames = c["batch"] * (c["frames"] + c["frames_min"]) / 2.0
    # hypothesis-steps: an utterance takes part until its own frames are over
    rows = _steps(c) * c["batch"] * c["beam"] * (1.0 + c["frames_min"] / c["frames"]) / 2.0
    per_row = 2.0 * H * n_out
    weights = H * c["enc"] + H * n_out
    if c["pred"] == "lstm":
        per_row += 2.0 * H * 4 * H + 2.0 * H * H  # recurrent gates, projection (the token half of the gates is a table)
        weights += 4 * H * H + H * H + 4 * H * (V + 1)
    else:
        weights += 2 * H * (V + 1)
    flops = 2.0 * total_frames * c["enc"] * H + rows * per_row
    n_best = 4.0 * c["batch"] * c["beam"] * (c["frames"] * c["symbols"] + 1)
    data = 4.0 * weights + 4.0 * total_frames * c["enc"] + n_best
    if c["ngrams"]:
        data += rows * 4.0 * V  # a row of unigram scores per hypothesis and step
    return {"bytes": data, "flops": flops}


def tolerance(c):
    # Scores are sums of some hundred float32 log-probabilities (bf16: of logits whose operands were rounded to 8 bits).
    # Two hypotheses that tie within that noise may change places, which changes the tokens of one list entry.
    if c["prec"] == "bf16":
        return {"rel": 1e-3, "max": 1e-2, "differ": 0.01}
    return {"rel": 2e-5, "max": 1e-3, "differ": 0.01}
