"""FP32 attention under large scores: the parts of a document that have softmax states of their own are
weighed as in float64.

The model makes every number up to the softmax exact: embeddings of +-1 and no epsilon (the norm
divides by one), queries and keys in the one rotary pair that does not turn (its frequency is
1e-28), of 256 and 256 +- 1/256.  Scores are then 65 536 +- 1, whose scaled maxima round by up to
2^-10, and the weight of a token's keys is 2^(its score).  Value and output matrices put the share of
token A's keys into one hidden dimension, and the feed-forward is off.

Tolerance: exp2 and the reciprocal within 2^-22, sums of n equal numbers within (steps of 16 keys)
2^-24, the norms and the head within 2^-22: 2^-18 of the logit covers them (1024 keys).  A state
taken at its unrounded maximum is wrong by 2^-12 and more, which the test asserts for its scores."""
import numpy as np
import pytest

from oracle import model as O
from paper_2602_04430_amd import kvop as K
from paper_2602_04430_amd import synth
from tests.gpu_common import Engine, say

TOL = 2.0 ** -18
A, B = 2, 3                              # tokens; the suffix is one B
ORDERS = {"low after high": [(A, 512), (B, 512)], "high after low": [(B, 512), (A, 512)],
          "inside a chunk": [(B, 300), (A, 400)], "three chunks": [(B, 512), (A, 100), (B, 600)]}


def _model(D):
    shape = synth.ModelShape(n_layers=1, d_model=64, n_heads=1, n_kv_heads=1, head_dim=D, d_ffn=64, vocab=8,
                             rms_eps=0.0, rope_theta=1e30)
    w = {k: np.zeros_like(v) for k, v in synth.make_weights(shape, 1).items()}
    w["embed"][:] = np.where(np.random.default_rng(2).random((8, 64)) < 0.5, -1, 1)
    w["embed"][[A, B], 0], w["embed"][A, 1], w["embed"][B, 1] = 1, 1, -1
    for k in w:
        if k.endswith("norm"):
            w[k][:] = 1
    pair = D // 2 - 1
    w["L0.wq"][pair, 0] = 256
    w["L0.wk"][pair, :2] = 256, 1 / 256
    w["L0.wv"][0, :2] = 0.5, 0.5         # 1 for A, 0 for B
    w["L0.wo"][5, 0] = 8
    w["head"][synth.YES_ID, 5], w["head"][synth.NO_ID, :5] = 1, 1
    return shape, w


@pytest.mark.parametrize("D", [32, 64, 128])
def test_an_unrounded_maximum_would_show(D):
    """(host only)"""
    c = np.float32(1.4426950408889634 / np.sqrt(D))
    err = [float(np.float32(np.float32(s) * c)) - s * float(c) for s in (65537.0, 65535.0)]
    # the share of A moves by a quarter of it, the logit by at least a quarter of that
    assert abs(err[0] - err[1]) * np.log(2) / 16 > 4 * TOL, err


@pytest.mark.gpu
@pytest.mark.parametrize("D", [32, 64, 128])
@pytest.mark.parametrize("order", sorted(ORDERS))
def test_shares_of_the_chunks(device, D, order):
    shape, w = _model(D)
    doc = np.concatenate([np.full(n, t, np.int32) for t, n in ORDERS[order]])
    n, suffix = len(doc), np.array([B], np.int32)
    m = O.Model(shape, w)
    ref = O.filter_eval(m, O.kv_build(m, doc), np.arange(n), suffix, synth.YES_ID, synth.NO_ID).logits
    eng = Engine(shape, w, "f32", "f32", 64 << 20)
    handles = eng.build(synth.Docs(np.asarray([n]), doc, np.asarray([0, n])))
    say("scores", D, order)
    alone, _ = eng.filter(handles, np.arange(n), [0, n], suffix)
    many = 700
    lg, _ = eng.filter(np.tile(handles, many), np.tile(np.arange(n, dtype=np.int32), many),
                       np.arange(many + 1, dtype=np.int64) * n, suffix)
    eng.close()
    assert np.abs(alone[0] - ref).max() <= TOL * np.abs(ref).max(), (alone[0], ref)
    np.testing.assert_array_equal(lg, np.tile(alone, (many, 1)))
