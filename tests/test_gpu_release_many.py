"""Releasing many documents in one call: each handle once, nothing released when one is refused, and time
in proportion to their number."""
import time

import numpy as np
import pytest

from paper_2602_04430_amd import kvop as K
from paper_2602_04430_amd import synth
from tests.gpu_common import Engine, say

pytestmark = pytest.mark.gpu


def test_release_of_many(device):
    shape = synth.ModelShape(n_layers=1, d_model=64, n_heads=1, n_kv_heads=1, head_dim=32, d_ffn=64, vocab=64)
    eng = Engine(shape, synth.make_weights(shape, 1), "bf16", "bf16", 64 << 20)
    took = {}
    for n in 3 * (2000, 40000):
        lengths = np.full(n, 2, np.int64)
        toks, offs = synth.doc_tokens(lengths, shape.vocab, 3)
        handles = eng.build(synth.Docs(lengths, toks, offs))
        for bad in (np.concatenate([handles, handles[:1]]), np.concatenate([handles, handles[-1:]])):
            with pytest.raises(K.KvopError, match="twice"):
                K.kvop_kv_release(eng.pool, bad)
        start = time.perf_counter()
        K.kvop_kv_release(eng.pool, handles)
        took[n] = min(took.get(n, 1e9), time.perf_counter() - start)
        say("released", n, took[n])
        assert K.kvop_pool_stats(eng.pool)[2] == 0
        with pytest.raises(K.KvopError, match="not live"):
            K.kvop_kv_release(eng.pool, handles[:1])
    eng.close()
    assert took[40000] < 100 * took[2000], took       # 20 times the documents; 400 times with a search each
