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


def test_select_at_register_and_segment_edges(device):
    """Selection against the oracle's top-k of the same FP32 values: lengths at the edges of a wavefront,
    a workgroup, the rows that one wavefront (1024) and one workgroup (4096) keep in registers, scores that differ in every bit or in one,
    all equal, signed zeros, infinities and the type's extremes."""
    import torch

    from paper_2602_04430_amd import kvop as K
    lengths = np.array([2, 63, 64, 65, 255, 256, 257, 511, 513, 1023, 1024, 1025, 4095, 4096, 4097, 8192, 8193], np.int64)
    rng = np.random.default_rng(9)
    eng = Engine(synth.ModelShape(n_layers=1, d_model=128, n_heads=4, n_kv_heads=2, head_dim=64, d_ffn=128, vocab=256),
                 synth.make_weights(synth.ModelShape(n_layers=1, d_model=128, n_heads=4, n_kv_heads=2, head_dim=64,
                                                     d_ffn=128, vocab=256), 1), "f32", "f32", pool_bytes=1 << 24)
    n, offs = int(lengths.sum()), np.concatenate([[0], np.cumsum(lengths)])
    big = np.finfo(np.float32).max
    kinds = {"distinct": rng.standard_normal(n).astype(np.float32),
             "one bit": np.where(rng.random(n) < 0.5, np.float32(1.0), np.nextafter(np.float32(1.0), np.float32(2.0))),
             "equal": np.full(n, 0.25, np.float32),
             "extremes": rng.choice(np.array([0.0, big, -big, np.inf, -np.inf, 1e-45], np.float32), n)}
    for name, sc in kinds.items():
        dsc = torch.from_numpy(sc.astype(np.float32)).cuda()
        for r in (0.99, 0.5, 0.03):
            ks = [synth.retained_count(r, int(L)) for L in lengths]
            idx = torch.full((sum(ks) + 1,), -1, dtype=torch.int32, device="cuda")
            io = K.kvop_ea_select(eng.pool, dsc, offs, r, idx)
            torch.cuda.synchronize()
            got = idx.cpu().numpy()
            assert got[-1] == -1
            for i, L in enumerate(lengths):
                want = oc.ea_select(sc[offs[i]:offs[i + 1]].astype(np.float64), ks[i])
                np.testing.assert_array_equal(got[io[i]:io[i + 1]], want, err_msg=f"{name} r {r} L {L}")
    eng.close()
