"""The proxy's one-pass inference (from 8192 rows on) with a standardiser of its own mean and spread per
column: against the oracle, bit for bit against the separate passes, on features off a 16-byte
boundary, without allocation, and at the largest sizes it takes; and the standardiser over several
column groups an XCD."""
import numpy as np
import pytest
import torch

from oracle import codecs
from oracle import proxy as op
from paper_2602_04430_amd import kvop as K
from paper_2602_04430_amd import synth
from tests.gpu_common import say

pytestmark = pytest.mark.gpu
TAU = 0.6


def _proxy(d, h, seed):
    rng = np.random.default_rng(seed)
    p = synth.proxy_init(d, h, 2, seed)
    p["b1"] = (rng.standard_normal(h) * 0.05).astype(np.float32)
    p["w2"] = (rng.standard_normal((2, h)) * 0.4).astype(np.float32)
    flat = np.concatenate([p["w1"].ravel(), p["b1"], p["w2"].ravel(), p["b2"]]).astype(np.float32)
    return p, K.kvop_proxy_create(d, h, torch.from_numpy(flat).cuda())


def _features(n, d, seed, lead=0):
    """[n, d] with its own mean and spread per column, `lead` floats past a 16-byte boundary."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    mean = torch.randn(d, generator=g, device="cuda")
    std = torch.rand(d, generator=g, device="cuda") * 2 + 0.2
    f = torch.empty(n * d + lead, device="cuda")[lead:].view(n, d)
    f.copy_(torch.randn(n, d, generator=g, device="cuda") * std + mean)
    assert f.data_ptr() % 16 == 4 * lead
    return f, mean, 1.0 / std


def _infer(px, f, call=None):
    n = f.shape[0]
    out = [torch.full((n,), 7, dtype=torch.int8, device="cuda"), torch.full((n,), np.nan, device="cuda"),
           torch.full((n,), 7, dtype=torch.int8, device="cuda")]
    (call or K.kvop_proxy_infer)(px, f, TAU, *out)
    torch.cuda.synchronize()
    return [x.cpu().numpy() for x in out]


def _equal(a, b):
    for x, y in zip(a, b):
        np.testing.assert_array_equal(x, y)


def _check_oracle(p, f, mean, istd, rows, got):
    """conf of `rows` against float64 on the same 16-bit features and weights (FP32 sums: 1e-5)."""
    w = {k: np.asarray(v, np.float64) for k, v in p.items()}
    w["w1"] = codecs.bf16_round(p["w1"]).astype(np.float64)
    x = ((f[rows] - mean) * istd).cpu().numpy()
    _, _, _, probs = op.forward(w, codecs.bf16_round(x).astype(np.float64))
    cls, conf, ans = (g[rows.cpu().numpy()] for g in got)
    np.testing.assert_allclose(conf, probs.max(axis=1), rtol=0, atol=1e-5)
    clear = np.abs(probs[:, 1] - probs[:, 0]) > 1e-4
    np.testing.assert_array_equal(cls[clear], np.argmax(probs, axis=1)[clear])
    np.testing.assert_array_equal(ans, (conf > np.float32(TAU)).astype(np.int8))
    # a column's mean or spread taken from its neighbour would show
    for m, s in ((mean.roll(1), istd), (mean, istd.roll(1))):
        _, _, _, other = op.forward(w, ((f[rows] - m) * s).cpu().numpy().astype(np.float64))
        assert np.abs(other.max(axis=1) - probs.max(axis=1)).max() > 1e-3


@pytest.mark.parametrize("d,h", [(64, 64), (192, 128), (2048, 256), (4096, 64), (4096, 256)])
def test_fused_equals_oracle_and_separate_passes(device, d, h):
    p, px = _proxy(d, h, d + h)
    n = 12289                              # a row in a tile of its own, and several tiles a workgroup
    f, mean, istd = _features(n, d, 3)
    K.kvop_proxy_set_standardizer(px, mean, istd)
    say("fused inference", d, h)
    got = _infer(px, f)
    rows = torch.cat([torch.arange(0, 40), torch.arange(n // 2, n // 2 + 40), torch.arange(n - 60, n)]).cuda()
    _check_oracle(p, f, mean, istd, rows, got)
    for r0, r1 in ((0, 4096), (4096, 8191), (8191, n)):       # fewer than 8192 rows: the separate passes
        _equal(_infer(px, f[r0:r1]), [x[r0:r1] for x in got])
    for m in (8192, 8193, 8207, 8209):
        _equal(_infer(px, f[:m]), [x[:m] for x in got])
    K.kvop_proxy_destroy(px)


@pytest.mark.parametrize("lead", [1, 2, 3])
@pytest.mark.parametrize("n", [300, 8200])
def test_features_off_a_16_byte_boundary(device, n, lead):
    _, px = _proxy(320, 128, 4)
    f, mean, istd = _features(n, 320, 5, lead)
    K.kvop_proxy_set_standardizer(px, mean, istd)
    say("off boundary", n, lead)
    _equal(_infer(px, f), _infer(px, f.clone()))
    K.kvop_proxy_destroy(px)


def test_fused_without_allocation(device):
    """9000 rows of 64 columns are within the scratch's limit and take the one-pass form."""
    p, px = _proxy(64, 64, 6)
    f, mean, istd = _features(9000, 64, 7)
    K.kvop_proxy_set_standardizer(px, mean, istd)
    say("no allocation")
    got = _infer(px, f, K.kvop_proxy_infer_noalloc)
    _check_oracle(p, f, mean, istd, torch.arange(8900, 9000).cuda(), got)
    _equal(got, _infer(px, f))
    K.kvop_proxy_destroy(px)


@pytest.mark.parametrize("d", [64, 192, 1088, 2048])
@pytest.mark.parametrize("n", [3, 700, 2049])
def test_standardiser_over_column_groups(device, d, n):
    """4 to 128 groups of 16 columns over eight XCDs, with remainders: bit-equal to the kernel for
    features off a boundary, and each column's own mean and spread (two-pass float64, on rounded
    inputs; FP32 sums of n rows move a standardised feature by less than its 16-bit rounding, which
    the oracle's tolerance of 2^-6 of a probability covers)."""
    p, px = _proxy(d, 64, d)
    on, _, _ = _features(n, d, n)
    off = torch.empty(n * d + 1, device="cuda")[1:].view(n, d)
    off.copy_(on)
    say("standardiser", d, n)
    outs = []
    for f in (on, off):
        K.kvop_proxy_fit_standardizer(px, f)
        outs.append(_infer(px, on))
    _equal(*outs)
    x = on.double()
    x = ((x - x.mean(0)) / x.std(0, correction=0).clamp_min(1e-6)).cpu().numpy()
    _, _, _, probs = op.forward({k: np.asarray(v, np.float64) for k, v in p.items()}, x[:50])
    np.testing.assert_allclose(outs[0][1][:50], probs.max(axis=1), rtol=0, atol=2.0 ** -6)
    K.kvop_proxy_destroy(px)
