"""The residual add on tiles with wavefronts that only load: in place over several row tiles, each
output is added to once, with the bits of the general register-staged tile."""
import pytest
import torch

from paper_2602_04430_amd import kvop as K

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,general", [("bf16_32x16x256_8w_swz2_lds4", 7), ("bf16_32x32x256_8w_swz2_lds4", 7),
                                          ("f32_32x16x128_8w_swz2_lds4", 0), ("f32_32x32x128_8w_swz2_lds4", 0)])
def test_row_tiles_add_in_place(device, name, general):
    bf16 = name.startswith("bf16")
    dt, ty = (K.KVOP_BF16, torch.bfloat16) if bf16 else (K.KVOP_F32, torch.float32)
    tile = [K.kvop_gemm_tile_name(dt, t) for t in range(K.kvop_gemm_num_tiles(dt))].index(name)
    g = torch.Generator().manual_seed(3)
    N, Kd = 208, 320
    for M in (1, 31, 32, 33, 127, 128, 129, 500):
        A = torch.randn(M, Kd, generator=g).to(device, ty)
        B = (torch.randn(N, Kd, generator=g) * 0.05).to(device, ty)
        C0 = torch.randn(M, N + 8, generator=g).to(device)
        outs = []
        for t in (general, tile):
            C = C0.clone()
            K.kvop_debug_gemm(dt, K.KVOP_F32, 1, t, A, B, C, M, N, Kd, Kd, Kd, N + 8)
            outs.append(C)
        torch.cuda.synchronize()
        assert torch.equal(outs[0], outs[1]), M
        assert torch.equal(outs[0][:, N:], C0[:, N:]), M
