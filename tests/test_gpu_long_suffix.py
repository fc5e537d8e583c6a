"""A suffix whose projected rows take more than 4 GiB: the attention reads every own row, those past
the first 4 GiB too.

One layer, so only the last row's attention counts, over a document and 65 000 own rows of 96 KiB
(rows from 43 691 on lie past 4 GiB).  Keys and values of a one-layer model depend on the token alone,
so the reference weighs a value per token.  The suffix repeats one token and changes to
another one where the rows pass 4 GiB: reading other rows there changes the answer by far more than
the tolerance, which the test asserts of its reference.

Tolerance, relative to the larger logit: FP32 a few hundred roundings, 1e-4; BF16 some eight
roundings of 2^-9 in sequence (weights, normalised row, queries, keys, probabilities, values,
attention output, hidden row), with an FP8 cache the document's rows besides (40 of 65 040), 2^-4."""
import numpy as np
import pytest

from oracle import model as O
from paper_2602_04430_amd import synth
from tests.gpu_common import BOUND, Engine, say

D, ROWS, DOC = 128, 65000, 40
PITCH = 96 << 10
PAST = -(-(1 << 32) // PITCH)            # first row that starts past 4 GiB
CASES = [("f32", "f32", 64, 1e-4), ("bf16", "bf16", 128, 2.0 ** -4), ("bf16", "fp8", 128, 2.0 ** -4)]


def _shape(heads):
    return synth.ModelShape(n_layers=1, d_model=64, n_heads=heads, n_kv_heads=heads, head_dim=D, d_ffn=64, vocab=64)


def _weights(heads):
    w = synth.make_weights(_shape(heads), 11)
    w["L0.wq"] *= 4                        # keys of the last row's own token, all past 4 GiB, draw the attention
    w["L0.wk"] = w["L0.wq"]
    w["head"] *= 10
    return w


def _suffix(switch=PAST):
    s = np.full(ROWS, 3, np.int32)
    s[switch:] = 40
    return s


def _reference(w, heads, doc, suffix):
    """Logits of tokens 1 and 0 after the suffix, in float64."""
    w = {k: np.asarray(v, np.float64) for k, v in w.items()}
    norm = lambda x, g: x / np.sqrt(np.mean(x * x, -1, keepdims=True) + 1e-5) * g
    h = norm(w["embed"], w["L0.attn_norm"])
    tok = np.concatenate([doc, suffix])
    q, k, v = ((h @ w[f"L0.{n}"].T).reshape(-1, heads, D) for n in ("wq", "wk", "wv"))
    # q at the last position, k at position p: the angle is their distance
    ang = (len(tok) - 1 - np.arange(len(tok)))[:, None] * 10000.0 ** (-2.0 * np.arange(D // 2) / D)
    cos, sin = np.cos(ang), np.sin(ang)
    q1, q2 = q[tok[-1], :, :D // 2], q[tok[-1], :, D // 2:]
    out = np.empty((heads, D))
    used = np.unique(tok)
    for i in range(heads):
        k1, k2 = k[used, i, :D // 2], k[used, i, D // 2:]
        by_token = cos @ (q1[i] * k1 + q2[i] * k2).T - sin @ (q2[i] * k1 - q1[i] * k2).T
        s = by_token[np.arange(len(tok)), np.searchsorted(used, tok)] / np.sqrt(D)
        p = np.exp(s - s.max())
        out[i] = np.bincount(tok, p, len(w["embed"])) @ v[:, i] / p.sum()
    x = w["embed"][tok[-1]] + out.reshape(-1) @ w["L0.wo"].T
    f = norm(x, w["L0.ffn_norm"])
    g = f @ w["L0.w_gate"].T
    x = x + (g / (1 + np.exp(-g)) * (f @ w["L0.w_up"].T)) @ w["L0.w_down"].T
    return w["head"][[synth.YES_ID, synth.NO_ID]] @ norm(x, w["final_norm"])


def _doc():
    return synth.doc_tokens(np.asarray([DOC]), 64, 3)


@pytest.mark.parametrize("heads,tol", sorted({(h, t) for _, _, h, t in CASES}))
def test_the_rows_past_4_gib_decide_the_answer(heads, tol):
    """(host only) what the GPU test would compute without those rows is well outside its tolerance"""
    assert 3 * heads * D * (4 if heads == 64 else 2) == PITCH
    w, (doc, _) = _weights(heads), _doc()
    ref = _reference(w, heads, doc, _suffix())
    wrong = _suffix(ROWS - 1)              # the last token stays
    other = _reference(w, heads, doc, wrong)
    assert np.abs(ref - other).max() > 4 * tol * np.abs(ref).max(), (ref, other)


@pytest.mark.gpu
@pytest.mark.parametrize("compute,kv,heads,tol", CASES)
def test_own_rows_past_4_gib(device, compute, kv, heads, tol):
    w, (doc, offs) = _weights(heads), _doc()
    eng = Engine(_shape(heads), w, compute, kv, 64 << 20)
    say("long suffix", compute, kv, heads)
    handles = eng.build(synth.Docs(np.asarray([DOC]), doc, offs))
    lg, _ = eng.filter(handles, np.arange(DOC), [0, DOC], _suffix())
    ref = _reference(w, heads, doc, _suffix())
    eng.close()
    assert np.abs(lg[0] - ref).max() <= tol * np.abs(ref).max(), (lg[0], ref)


@pytest.mark.gpu
@pytest.mark.parametrize("compute,kv,D", [("f32", "f32", 32), ("f32", "f32", 128), ("bf16", "bf16", 64),
                                          ("bf16", "bf16", 128), ("bf16", "fp8", 128)])
def test_own_rows_where_the_base_moves(device, compute, kv, D):
    """The kernels move the own rows' base every 1024 rows: suffixes on both sides of that, every row's
    hidden state deciding the next layer's keys."""
    shape = synth.ModelShape(n_layers=2, d_model=128, n_heads=2, n_kv_heads=1, head_dim=D, d_ffn=128, vocab=64)
    w = synth.make_weights(shape, 5)
    doc, offs = synth.doc_tokens(np.asarray([70]), 64, 3)
    eng = Engine(shape, w, compute, kv, 64 << 20)
    handles = eng.build(synth.Docs(np.asarray([70]), doc, offs))
    m = O.Model(shape, w)
    cache = O.kv_build(m, doc)
    for S in (1023, 1024, 1025, 1057, 2050):
        say("own rows", compute, kv, D, S)
        suffix = synth.suffix_tokens(S, 64, 6)
        lg, _ = eng.filter(handles, np.arange(70), [0, 70], suffix)
        ref = O.filter_eval(m, cache, np.arange(70), suffix, synth.YES_ID, synth.NO_ID)
        assert np.abs(lg[0] - ref.logits).max() <= BOUND[(compute, kv)], (S, lg[0], ref.logits)
    eng.close()
