"""The proxy's gradients are written straight into the caller's buffer: the same bits wherever it starts and
nothing beside it."""
import numpy as np
import pytest
import torch

from paper_2602_04430_amd import kvop as K
from paper_2602_04430_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,h,batch", [(64, 64, 8), (192, 128, 72), (1024, 256, 264)])
def test_any_start(device, d, h, batch):
    p = synth.proxy_init(d, h, 2, 1)
    flat = np.concatenate([p["w1"].ravel(), p["b1"], p["w2"].ravel(), p["b2"]]).astype(np.float32)
    px = K.kvop_proxy_create(d, h, torch.from_numpy(flat).cuda())
    g = torch.Generator(device="cuda").manual_seed(2)
    f = torch.randn(batch, d, generator=g, device="cuda")
    y = torch.randint(0, 2, (batch,), generator=g, device="cuda", dtype=torch.int32)
    rows = torch.arange(batch, device="cuda", dtype=torch.int32)
    n, loss, outs = len(flat), torch.empty(2, device="cuda"), []
    for lead in (0, 1, 2, 3, 4):
        buf = torch.full((n + 8,), 7.0, device="cuda")
        K.kvop_proxy_grads(px, f, y, rows, batch, buf[lead:lead + n], loss[lead % 2:])
        torch.cuda.synchronize()
        outs.append(buf[lead:lead + n].clone())
        assert torch.all(buf[:lead] == 7) and torch.all(buf[lead + n:] == 7), lead
        assert torch.equal(outs[0], outs[-1]), lead
    assert torch.isfinite(outs[0]).all() and loss[0] == loss[1]
    K.kvop_proxy_destroy(px)
