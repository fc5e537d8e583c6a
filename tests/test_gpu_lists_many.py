"""Retained lists are checked in both forms of the check (few or long lists: a workgroup each; many
short ones: a wavefront each), wherever the fault lies."""
import numpy as np
import pytest

from paper_2602_04430_amd import kvop as K
from paper_2602_04430_amd import synth
from tests.gpu_common import Engine, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lengths", [[3] * 7, [3] * 41 + [5], [300] * 4 + [2] * 599, [300] * 4 + [2] * 593])
def test_every_list_of_many(device, lengths):
    """7 and 42 lists of up to 3 and 5 rows and 603 of up to 300 run as wavefronts, 597 as workgroups."""
    shape = synth.ModelShape(n_layers=1, d_model=64, n_heads=1, n_kv_heads=1, head_dim=64, d_ffn=64, vocab=64)
    lengths = np.asarray(lengths, np.int64)
    toks, offs = synth.doc_tokens(lengths, shape.vocab, 3)
    eng = Engine(shape, synth.make_weights(shape, 2), "bf16", "bf16", 8 << 20)
    handles = eng.build(synth.Docs(lengths, toks, offs))
    suffix = synth.suffix_tokens(2, shape.vocab, 4)
    idx = np.concatenate([np.arange(n, dtype=np.int32) for n in lengths])
    lo = np.concatenate([[0], np.cumsum(lengths)])
    n = len(lengths)
    good, _ = eng.filter(handles, idx, lo, suffix)
    for doc in sorted({0, 1, 2, 3, 4, 5, n // 2, n - 2, n - 1}):
        for row in sorted({0, 1, int(lengths[doc]) - 1}):
            for value in (-1, int(lengths[doc])):
                bad = idx.copy()
                bad[lo[doc] + row] = value
                with pytest.raises(K.KvopError, match="1 index list"):
                    eng.filter(handles, bad, lo, suffix)
    say("two faults", n)
    bad = idx.copy()
    bad[lo[[1, n - 1]]] = -1
    with pytest.raises(K.KvopError, match="2 index list"):
        eng.filter(handles, bad, lo, suffix)
    again, _ = eng.filter(handles, idx, lo, suffix)
    eng.close()
    np.testing.assert_array_equal(good, again)
