"""FP32 attention: the keys of long items go to several workgroups where few items are long.  The
split changes no bits: documents alone (split) and among many (whole), at the edges of tiles (16
and 32 keys) and of chunks (512 keys), through lists and joins, at every head dimension, and
suffixes of one and of several blocks of query rows.  (Among many, the first layer's projection is
shared by all items; alone it is not.)"""
import numpy as np
import pytest

from paper_2602_04430_amd import kvop as K
from paper_2602_04430_amd import synth
from tests.gpu_common import Engine, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [32, 64, 128])
def test_alone_equals_among_many(device, D):
    shape = synth.ModelShape(n_layers=2, d_model=4 * D, n_heads=4, n_kv_heads=2, head_dim=D, d_ffn=256, vocab=512)
    rng = np.random.default_rng(6)
    special = [1, 15, 16, 17, 479, 480, 481, 495, 496, 497, 511, 512, 513, 1008, 1024, 1025, 2100]
    lengths = np.asarray(special + [int(x) for x in rng.integers(500, 600, 300)], np.int64)
    toks, offs = synth.doc_tokens(lengths, shape.vocab, 3)
    eng = Engine(shape, synth.make_weights(shape, 2), "f32", "f32", 2 << 30)
    handles = eng.build(synth.Docs(lengths, toks, offs))
    for r, S in ((1.0, 16), (0.5, 1), (1.0, 45)):
        idx, lo = synth.retained_lists(lengths, r, 7)
        suffix = synth.suffix_tokens(S, shape.vocab, 4)
        all_lg, all_dec = eng.filter(handles, idx, lo, suffix, r)
        for i in range(len(special)):
            say("document", D, r, S, int(lengths[i]))
            lg, dec = eng.filter(handles[i:i + 1], idx[lo[i]:lo[i + 1]], [0, lo[i + 1] - lo[i]], suffix, r)
            np.testing.assert_array_equal(lg[0], all_lg[i])
            assert dec[0] == all_dec[i]
        pairs = [(0, 16), (5, 12), (16, 3), (13, 9), (11, 11)]
        ph = np.asarray([handles[j] for ab in pairs for j in ab])
        pidx = np.concatenate([idx[lo[j]:lo[j + 1]] for ab in pairs for j in ab])
        po = np.concatenate([[0], np.cumsum([lo[j + 1] - lo[j] for ab in pairs for j in ab])])
        many = 60
        lg_m, _ = eng.filter(np.tile(ph, many), np.tile(pidx, many),
                             np.concatenate([[0], np.cumsum(np.tile(np.diff(po), many))]), suffix, r, kind=K.KVOP_JOIN)
        for q in range(len(pairs)):
            lg, _ = eng.filter(ph[2 * q:2 * q + 2], pidx[po[2 * q]:po[2 * q + 2]],
                               [0, po[2 * q + 1] - po[2 * q], po[2 * q + 2] - po[2 * q]], suffix, r, kind=K.KVOP_JOIN)
            np.testing.assert_array_equal(lg[0], lg_m[q])
