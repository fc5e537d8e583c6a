"""The proxy's one-pass inference, standardiser and batch reductions at the edges of their splits."""
import numpy as np
import pytest
import torch

from paper_2602_04430_amd import kvop as K
from paper_2602_04430_amd import synth

pytestmark = pytest.mark.gpu


def _proxy(d, h, seed):
    rng = np.random.default_rng(seed)
    p = synth.proxy_init(d, h, 2, seed)
    p["b1"] = (rng.standard_normal(h) * 0.05).astype(np.float32)
    p["w2"] = (rng.standard_normal((2, h)) * 0.4).astype(np.float32)
    flat = np.concatenate([p["w1"].ravel(), p["b1"], p["w2"].ravel(), p["b2"]]).astype(np.float32)
    return p, K.kvop_proxy_create(d, h, torch.from_numpy(flat).cuda())


def _infer(px, f, tau=0.6):
    n = f.shape[0]
    out = [torch.full((n,), 7, dtype=torch.int8, device="cuda"), torch.full((n,), np.nan, device="cuda"),
           torch.full((n,), 7, dtype=torch.int8, device="cuda")]
    K.kvop_proxy_infer(px, f, tau, *out)
    torch.cuda.synchronize()
    return [x.cpu().numpy() for x in out]


@pytest.mark.parametrize("d,h", [(64, 64), (192, 128), (2048, 256), (320, 512)])
def test_row_counts_and_widths(device, d, h):
    """Every split of the rows gives a row the same answer, equal to the oracle's within the BF16
    rounding of features and weights (h = 512 takes the separate passes).  The bound: z is a sum
    of h products with relative input error 2^-8 twice, so |dz| <= 2^-6 sum |W2| |gelu| <=
    2^-6 (sum W2^2)^1/2 (sum gelu^2)^1/2, and |dp| <= |dz| / 2 for two classes (two logits)."""
    p, px = _proxy(d, h, d + h)
    rng = np.random.default_rng(1)
    n = 4096 * 5 + 7
    feats = (rng.standard_normal((n, d)) * 0.7).astype(np.float32)
    f = torch.from_numpy(feats).cuda()
    cls, conf, ans = _infer(px, f)
    for m in (1, 15, 17, 33, 4097, 8191, 8192, 8193, 12288, 12289, 16385):
        if m > n:
            break
        c2, f2, a2 = _infer(px, f[:m])
        np.testing.assert_array_equal(c2, cls[:m])
        np.testing.assert_array_equal(f2, conf[:m])
        np.testing.assert_array_equal(a2, ans[:m])
    k = 200
    w = {q: np.asarray(v, np.float64) for q, v in p.items()}
    x = feats[-k:].astype(np.float64)
    pre = x @ w["w1"].T + w["b1"]
    act = 0.5 * pre * (1 + np.vectorize(__import__("math").erf)(pre / np.sqrt(2)))
    z = act @ w["w2"].T + w["b2"]
    pr = np.exp(z - z.max(1, keepdims=True))
    ref = (pr / pr.sum(1, keepdims=True)).max(1)
    spread = np.sqrt((w["w2"] ** 2).sum()) * np.sqrt((act ** 2).sum(1) + (x ** 2).sum(1) * (w["w1"] ** 2).sum(1).max())
    assert np.all(np.abs(conf[-k:] - ref) <= 2.0 ** -6 * spread)
    assert np.array_equal(ans, (conf > np.float32(0.6)).astype(np.int8))
    K.kvop_proxy_destroy(px)


@pytest.mark.parametrize("n", [1, 2, 255, 256, 257, 1791, 1792, 1793, 2048, 2049])
def test_standardiser_streams_the_same_sums(device, n):
    """The streaming standardiser and the one-thread-per-column one (features off a 16-byte
    boundary) add the same rows in the same order: bit-equal answers afterwards."""
    d, h = 128, 64
    rng = np.random.default_rng(n)
    base = torch.from_numpy((rng.standard_normal(n * d + 1) * 2 + 0.5).astype(np.float32)).cuda()
    off = base[1:].view(n, d)                       # 4 bytes past a 16-byte boundary
    on = off.clone()
    assert off.data_ptr() % 16 == 4 and on.data_ptr() % 16 == 0
    outs = []
    for f in (on, off):
        _, px = _proxy(d, h, 9)
        K.kvop_proxy_fit_standardizer(px, f)
        outs.append(_infer(px, f))
        K.kvop_proxy_destroy(px)
    for a, b in zip(*outs):
        np.testing.assert_array_equal(a, b)
    assert np.all(np.isfinite(outs[0][1]))


@pytest.mark.parametrize("batch,h", [(8, 64), (64, 128), (72, 64), (1032, 256), (512, 512)])
def test_gradients_over_batch_remainders(device, batch, h):
    """Bias, head and loss gradients against sums in float64 over the batch.  Bound: the FP32 terms
    carry the BF16 roundings of x and W1 (relative 2^-8 each, 2^-6 of the sum of magnitudes covers
    both layers)."""
    d = 128
    p, px = _proxy(d, h, batch)
    rng = np.random.default_rng(batch)
    feats = rng.standard_normal((batch + 5, d)).astype(np.float32)
    labels = rng.integers(0, 2, batch + 5).astype(np.int32)
    rows = rng.permutation(batch + 5)[:batch].astype(np.int32)
    g = torch.empty(h * d + 3 * h + 2, device="cuda")
    loss = torch.empty(1, device="cuda")
    K.kvop_proxy_grads(px, torch.from_numpy(feats).cuda(), torch.from_numpy(labels).cuda(),
                       torch.from_numpy(rows).cuda(), batch, g, loss)
    torch.cuda.synchronize()
    got = g.cpu().numpy().astype(np.float64)
    t = {q: torch.tensor(np.asarray(v, np.float64), requires_grad=True) for q, v in p.items()}
    x = torch.tensor(feats[rows].astype(np.float64))
    z = torch.nn.functional.gelu(x @ t["w1"].T + t["b1"]) @ t["w2"].T + t["b2"]
    ref = torch.nn.functional.cross_entropy(z, torch.tensor(labels[rows].astype(np.int64)))
    ref.backward()
    o = h * d
    for lo, hi, name in ((0, o, "w1"), (o, o + h, "b1"), (o + h, o + 3 * h, "w2"), (o + 3 * h, o + 3 * h + 2, "b2")):
        e = got[lo:hi] - t[name].grad.numpy().ravel()
        assert np.linalg.norm(e) <= 2.0 ** -6 * (np.linalg.norm(t[name].grad.numpy()) + 2.0 ** -6), name
    assert abs(float(loss[0]) - float(ref)) <= 2.0 ** -6
    K.kvop_proxy_destroy(px)
