"""The map head at the edges of its splits (items of 2 or, beyond 8192 columns, 1 per workgroup,
labels of 32): logits
against the FP64 oracle within the FP32 bound, the same bits alone and among many, ids the first
maximum of the item's logits."""
import numpy as np
import pytest

from oracle import model as om
from paper_2602_04430_amd import synth
from tests.gpu_common import E_F32, Engine, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,labels,items", [(128, 1, 1), (128, 31, 9), (128, 33, 17), (128, 100, 8), (2112, 40, 5), (8256, 33, 3)])
def test_map_head_splits(device, d, labels, items):
    shape = synth.ModelShape(n_layers=1, d_model=d, n_heads=2, n_kv_heads=1, head_dim=32, d_ffn=64, vocab=160)
    w = synth.make_weights(shape, 3, gain_jitter=0.1)
    docs = synth.make_docs_uniform(items, 3, 20, shape.vocab, seed=2)
    eng = Engine(shape, w, "f32", "f32", 16 << 20)
    handles = eng.build(docs)
    idx, offs = synth.full_lists(docs.lengths)
    suffix = synth.suffix_tokens(5, shape.vocab, 1)
    lo, n_gen = 20, 2
    say("map head", d, labels, items)
    lg, tk = eng.map(handles, idx, offs, suffix, lo, labels, n_gen)
    assert np.array_equal(tk, lo + np.argmax(lg, axis=2))
    m = om.Model(shape, w)
    for i in range(items):
        ref = om.map_eval(m, om.kv_build(m, docs.doc(i)), np.arange(docs.lengths[i]), suffix, lo, labels, n_gen)
        assert np.max(np.abs(lg[i, 0] - np.asarray(ref.step_logits)[0])) <= E_F32
    one, _ = eng.map(handles[:1], idx[:offs[1]], offs[:2], suffix, lo, labels, n_gen)
    np.testing.assert_array_equal(one[0], lg[0])
