"""FP32 attention without room for the chunks' states: they take at most 256 MiB beyond the feed-forward
buffer, and where they would take more, one workgroup takes all keys of its unit, with the same
bits.  Two documents of 16 000 rows under a suffix of 1024: alone 134 MiB of states (split),
together 268 MiB (whole), although the keys alone would split them."""
import numpy as np
import pytest

from paper_2602_04430_amd import kvop as K
from paper_2602_04430_amd import synth
from tests.gpu_common import Engine, say

HEADS, D, L, S = 8, 128, 16000, 1024
SHAPE = synth.ModelShape(n_layers=2, d_model=64, n_heads=HEADS, n_kv_heads=HEADS, head_dim=D, d_ffn=64, vocab=64)


def _items(docs):
    """Keys of the work items (blocks of 64 query rows) and the bytes of their chunks' states."""
    keys = [L + q + 64 for q in range(0, S, 64)] * docs
    chunks = sum(-(-(-(-L // 16) + -(-(k - L) // 16)) // 32) for k in keys)     # tiles of 16, chunks of 32 tiles
    return keys, chunks * 64 * HEADS * (D + 2) * 4


def test_the_sizes_are_on_both_sides_of_the_limit():
    """(host only)"""
    for docs, fits in ((1, True), (2, False)):
        keys, need = _items(docs)
        assert (need <= 256 << 20) == fits and need > docs * S * SHAPE.d_ffn * 4
        assert K.kvop_attention_form(K.KVOP_F32, K.KVOP_KV_F32, D, HEADS, 64, max(keys), sum(keys)) == 2


@pytest.mark.gpu
def test_without_room_the_bits_are_the_same(device):
    toks, offs = synth.doc_tokens(np.asarray([L, L]), 64, 3)
    eng = Engine(SHAPE, synth.make_weights(SHAPE, 2), "f32", "f32", 2 << 30)
    handles = eng.build(synth.Docs(np.asarray([L, L]), toks, offs))
    suffix = synth.suffix_tokens(S, 64, 4)
    rows = np.arange(L, dtype=np.int32)
    say("one by one")
    alone = [eng.filter(handles[i:i + 1], rows, [0, L], suffix)[0][0] for i in range(2)]
    say("together")
    both, _ = eng.filter(handles, np.tile(rows, 2), [0, L, 2 * L], suffix)
    again, _ = eng.filter(handles[1:], rows, [0, L], suffix)
    eng.close()
    np.testing.assert_array_equal(both, np.stack(alone))
    np.testing.assert_array_equal(again[0], alone[1])
    assert np.all(np.isfinite(both))
