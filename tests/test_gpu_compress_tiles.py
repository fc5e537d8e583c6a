"""Expected-attention scores at the edges of the query tiles (64 rows, four stages) and key groups
(32 keys, 1024-row segments), for every head width, against the FP64 oracle with the bounds of
the score test (FP32 rtol 1e-3; BF16 against the emulated BF16 form rtol 3e-2)."""
import numpy as np
import pytest

from oracle import codecs
from oracle import compress as oc
from oracle import model as om
from paper_2602_04430_amd import synth
from tests.gpu_common import Engine, say
from tests.test_gpu_compress import _docs, _scored

pytestmark = pytest.mark.gpu
LENGTHS = np.array([1, 31, 32, 33, 63, 95, 127, 128, 129, 191, 192, 193, 256, 257, 1023, 1024, 1025, 1057], np.int64)


@pytest.mark.parametrize("D", [32, 64, 128])
@pytest.mark.parametrize("compute", ["f32", "bf16"])
def test_scores_at_tile_edges(device, compute, D):
    shape = synth.ModelShape(n_layers=1, d_model=128, n_heads=4, n_kv_heads=2, head_dim=D, d_ffn=128, vocab=256)
    w = synth.make_weights(shape, 5, gain_jitter=0.1)
    docs = _docs(shape, 6, LENGTHS)
    eng = Engine(shape, w, compute, compute, 64 << 20)
    say("ea tiles", compute, D)
    _, scores = _scored(eng, docs, 7)
    got = scores.cpu().numpy().astype(np.float64)
    eng.close()
    if compute == "f32":
        m, rtol = om.Model(shape, w), 1e-3
    else:
        m, rtol = om.Model(shape, {k: codecs.bf16_round(v) if v.ndim == 2 else v for k, v in w.items()},
                           act=codecs.bf16_round), 3e-2
    for i, L in enumerate(docs.lengths):
        ref = oc.ea_scores(m, docs.doc(i), 7)
        np.testing.assert_allclose(got[docs.offsets[i]:docs.offsets[i + 1]], ref, rtol=rtol, atol=1e-6,
                                   err_msg=f"document {i} L {L}")
