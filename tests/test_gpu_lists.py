"""Retained lists are checked wherever the fault lies: at the ends of a list, and on both sides of the
rows that the check's workgroup takes at a time (256 and 1024)."""
import numpy as np
import pytest

from paper_2602_04430_amd import kvop as K
from paper_2602_04430_amd import synth
from tests.gpu_common import Engine

pytestmark = pytest.mark.gpu


def test_faults_are_found_at_every_edge(device):
    shape = synth.ModelShape(n_layers=1, d_model=128, n_heads=2, n_kv_heads=1, head_dim=64, d_ffn=128, vocab=256)
    lengths = np.array([1, 300, 2500], np.int64)
    toks, offs = synth.doc_tokens(lengths, shape.vocab, 3)
    eng = Engine(shape, synth.make_weights(shape, 2), "bf16", "bf16", 64 << 20)
    handles = eng.build(synth.Docs(lengths, toks, offs))
    suffix = synth.suffix_tokens(4, shape.vocab, 4)
    idx = np.concatenate([np.arange(L, dtype=np.int32) for L in lengths])
    lo = np.concatenate([[0], np.cumsum(lengths)])
    good, _ = eng.filter(handles, idx, lo, suffix)
    for doc, rows in ((0, (0,)), (1, (0, 1, 255, 256, 299)), (2, (0, 255, 256, 1023, 1024, 1025, 2047, 2048, 2499))):
        for row in rows:
            for value in (-1, int(lengths[doc]), row - 1):     # negative, past the end, equal to the row before
                if value == row - 1 and row == 0:
                    continue
                bad = idx.copy()
                bad[lo[doc] + row] = value
                with pytest.raises(K.KvopError, match="1 index list"):
                    eng.filter(handles, bad, lo, suffix)
    again, _ = eng.filter(handles, idx, lo, suffix)
    np.testing.assert_array_equal(good, again)
    eng.close()
