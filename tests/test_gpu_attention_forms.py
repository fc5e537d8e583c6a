"""The forms of the attention that the work list decides give the same bits, each form seen to be the one
that runs: documents alone take the form for few long items, the same documents among many the
form for many keys, in the suffix layers and in the last one.  Lengths at the edges of tiles
(16 and 32 keys) and of the FP32 chunks (512 keys)."""
import numpy as np
import pytest

from paper_2602_04430_amd import kvop as K
from paper_2602_04430_amd import synth
from tests.gpu_common import COMPUTE, KVDT, Engine, say

SPECIAL = {"f32": [1, 15, 16, 17, 479, 480, 481, 495, 496, 497, 511, 512, 513, 1008, 1024, 1025, 2100],
           "bf16": [1, 4, 31, 32, 33, 63, 64, 65, 96, 97, 129, 160, 1500]}
OTHERS = {"f32": (500, 600), "bf16": (280, 320)}
COPIES = 5
ALONE, MANY = {"f32": 2, "bf16": 4}, {"f32": 3, "bf16": 2}
CASES = [("f32", 32), ("f32", 64), ("f32", 128), ("bf16", 128)]
EVALS = {"f32": [(1.0, 16), (0.5, 1), (1.0, 45)], "bf16": [(1.0, 32), (0.5, 7), (1.0, 45)]}


def _shape(D):
    return synth.ModelShape(n_layers=2, d_model=4 * D, n_heads=4, n_kv_heads=2, head_dim=D, d_ffn=256, vocab=512)


def _lengths(kind):
    return np.asarray(SPECIAL[kind] + [int(x) for x in np.random.default_rng(6).integers(*OTHERS[kind], 300)], np.int64)


def _forms(kind, D, keys, S):
    """The forms of the suffix layers and of the last layer over items of `keys` retained rows (two
    query heads share a kv head: blocks of 32 query rows)."""
    block = min(S, 32)
    blocks = [k + min(S, q + block) for k in keys for q in range(0, S, block)]
    ask = lambda rows, n: K.kvop_attention_form(COMPUTE[kind], KVDT[kind], D, 2, rows, max(n), int(sum(n)))
    return ask(2 * block, blocks), ask(2, [k + S for k in keys])


def _check_choice(kind, D, kept, S):
    assert _forms(kind, D, list(kept) * COPIES, S) == (MANY[kind], MANY[kind])
    alone = [_forms(kind, D, [k], S) for k in kept[:len(SPECIAL[kind])]]
    several = [f for k, f in zip(kept, alone) if kind != "f32" or k > 512]   # (FP32: items of several chunks)
    assert several and set(several) == {(ALONE[kind], ALONE[kind])}


@pytest.mark.parametrize("kind,D", CASES)
def test_the_lists_take_both_forms(kind, D):
    """(host only)"""
    for r, S in EVALS[kind]:
        _check_choice(kind, D, [synth.retained_count(r, int(n)) for n in _lengths(kind)], S)


@pytest.mark.gpu
@pytest.mark.parametrize("kind,D", CASES)
def test_few_and_many_agree(device, kind, D):
    lengths = _lengths(kind)
    toks, offs = synth.doc_tokens(lengths, 512, 3)
    eng = Engine(_shape(D), synth.make_weights(_shape(D), 2), kind, kind, 2 << 30)
    handles = eng.build(synth.Docs(lengths, toks, offs))
    for r, S in EVALS[kind]:
        idx, lo = synth.retained_lists(lengths, r, 7)
        suffix = synth.suffix_tokens(S, 512, 4)
        _check_choice(kind, D, np.diff(lo), S)
        many_lo = np.concatenate([[0], np.cumsum(np.tile(np.diff(lo), COPIES))])
        all_lg, all_dec = eng.filter(np.tile(handles, COPIES), np.tile(idx, COPIES), many_lo, suffix, r)
        n = len(lengths)
        for c in range(1, COPIES):
            np.testing.assert_array_equal(all_lg[c * n:(c + 1) * n], all_lg[:n])
        for i in range(len(SPECIAL[kind])):
            say("document", kind, D, r, S, int(lengths[i]))
            lg, dec = eng.filter(handles[i:i + 1], idx[lo[i]:lo[i + 1]], [0, lo[i + 1] - lo[i]], suffix, r)
            np.testing.assert_array_equal(lg[0], all_lg[i])
            assert dec[0] == all_dec[i]
    eng.close()
