"""The stages the attention keeps in flight, chosen from the work list, change no bits: short and
long documents, alone (the deeper form) and among many (the shallow form), filters and joins."""
import numpy as np
import pytest
import torch

from paper_2602_04430_amd import kvop as K
from paper_2602_04430_amd import synth
from tests.gpu_common import Engine, say

pytestmark = pytest.mark.gpu
SHAPE = synth.ModelShape(n_layers=2, d_model=256, n_heads=4, n_kv_heads=2, head_dim=128, d_ffn=256, vocab=512)


@pytest.mark.parametrize("kv", ["bf16", "fp8"])
def test_alone_equals_among_many(device, kv):
    rng = np.random.default_rng(5)
    # tile edges of 32 and 64 keys, one to five tiles, and one long document
    special = [1, 4, 31, 32, 33, 63, 64, 65, 96, 97, 129, 160, 1500]
    lengths = np.asarray(special + [int(x) for x in rng.integers(40, 70, 500)], np.int64)
    toks, offs = synth.doc_tokens(lengths, SHAPE.vocab, 3)
    eng = Engine(SHAPE, synth.make_weights(SHAPE, 2), "bf16", kv, 256 << 20)
    handles = eng.build(synth.Docs(lengths, toks, offs))
    for r, S in ((1.0, 32), (0.5, 7)):
        idx, lo = synth.retained_lists(lengths, r, 7)
        suffix = synth.suffix_tokens(S, SHAPE.vocab, 4)
        all_lg, all_dec = eng.filter(handles, idx, lo, suffix, r)
        for i in range(len(special)):
            say("document", kv, r, int(lengths[i]))
            lg, dec = eng.filter(handles[i:i + 1], idx[lo[i]:lo[i + 1]], [0, lo[i + 1] - lo[i]], suffix, r)
            np.testing.assert_array_equal(lg[0], all_lg[i])
            assert dec[0] == all_dec[i]
        pairs = [(0, 12), (5, 6), (12, 3), (7, 9)]
        ph = np.asarray([handles[j] for ab in pairs for j in ab])
        pidx = np.concatenate([idx[lo[j]:lo[j + 1]] for ab in pairs for j in ab])
        po = np.concatenate([[0], np.cumsum([lo[j + 1] - lo[j] for ab in pairs for j in ab])])
        many = 200
        lg_m, _ = eng.filter(np.tile(ph, many), np.tile(pidx, many),
                             np.concatenate([[0], np.cumsum(np.tile(np.diff(po), many))]), suffix, r, kind=K.KVOP_JOIN)
        for q in range(len(pairs)):
            lg, _ = eng.filter(ph[2 * q:2 * q + 2], pidx[po[2 * q]:po[2 * q + 2]],
                               [0, po[2 * q + 1] - po[2 * q], po[2 * q + 2] - po[2 * q]], suffix, r, kind=K.KVOP_JOIN)
            np.testing.assert_array_equal(lg[0], lg_m[q])
