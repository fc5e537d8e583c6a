"""Pooled document features at the edges of their row chunks (64 rows) and column blocks (2048)."""
import numpy as np
import pytest

from oracle import model as om
from paper_2602_04430_amd import synth
from tests.gpu_common import Engine, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [128, 2048, 2112, 4160])
def test_pooled_features_at_chunk_edges(device, d):
    """Against the FP64 oracle within 1e-4 of the largest feature (FP32 model), and a document's
    features the same bits whatever documents it is built with."""
    shape = synth.ModelShape(n_layers=1, d_model=d, n_heads=2, n_kv_heads=1, head_dim=32, d_ffn=64, vocab=64)
    lengths = np.asarray([1, 2, 63, 64, 65, 127, 128, 129, 200], np.int64)
    toks, offs = synth.doc_tokens(lengths, shape.vocab, 3)
    docs = synth.Docs(lengths, toks, offs)
    w = synth.make_weights(shape, 1, gain_jitter=0.1)
    eng = Engine(shape, w, "f32", "f32", 16 << 20)
    _, pooled = eng.build(docs, pooled=True)
    pooled = pooled.cpu().numpy()
    m = om.Model(shape, w)
    for i in range(len(lengths)):
        say("pooled", d, int(lengths[i]))
        ref = om.kv_build(m, docs.doc(i)).pooled
        assert np.max(np.abs(pooled[i] - ref)) <= 1e-4 * np.max(np.abs(ref)), (d, lengths[i])
        _, alone = eng.build(docs.subset([i]), pooled=True)
        np.testing.assert_array_equal(alone.cpu().numpy()[0], pooled[i])
