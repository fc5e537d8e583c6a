"""The tile the library chooses for a projection: the same bits as the general register-staged
tile whatever rows, columns, depth, strides and alignment, at the edges of the narrow tiles."""
import numpy as np
import pytest
import torch

from paper_2602_04430_amd import kvop as K

pytestmark = pytest.mark.gpu
GENERAL = 7      # 128x128 register-staged


@pytest.mark.parametrize("epi", [0, 1, 2, 3])
@pytest.mark.parametrize("N,Kd", [(2048, 2048), (384, 320), (640, 5632), (256, 64)])
def test_chosen_tile_gives_the_general_tiles_bits(device, epi, N, Kd):
    rng = np.random.default_rng(N + Kd + epi)
    D = 128
    g = torch.Generator().manual_seed(1)
    cos = torch.randn(64, D // 2, generator=g).to(device)
    sin = torch.randn(64, D // 2, generator=g).to(device)
    out_dt = torch.float32 if epi == 1 else torch.bfloat16
    Nc = N // 2 if epi == 2 else N
    seen = set()
    for M in (1, 15, 16, 17, 31, 32, 33, 64, 65, 129, 200, 257, 513, 1100, 2049):
        lda = Kd if epi == 3 else Kd + 8
        A = torch.from_numpy(rng.standard_normal((M, lda)).astype(np.float32)).to(device).bfloat16()
        B = torch.from_numpy(rng.standard_normal((N, Kd)).astype(np.float32) * 0.05).to(device).bfloat16()
        C0 = torch.from_numpy(rng.standard_normal((M, Nc)).astype(np.float32)).to(device).to(out_dt)
        pos = torch.from_numpy(rng.integers(0, 64, M).astype(np.int32)).to(device)
        outs = []
        for tile in (GENERAL, -1):
            C = C0.clone()
            if epi == 3:
                K.kvop_debug_gemm_rope(tile, A, B, C, M, N, Kd, D, N - D, pos, cos, sin, True)
            else:
                K.kvop_debug_gemm(K.KVOP_BF16, K.KVOP_F32 if epi == 1 else K.KVOP_BF16, epi, tile, A, B, C, M, N, Kd,
                                  lda, Kd, Nc)
            outs.append(C)
        seen.add(K.kvop_gemm_pick_tile(K.KVOP_BF16, epi, M, N, Kd))
        torch.cuda.synchronize()
        assert torch.equal(outs[0], outs[1]), (epi, M, N, Kd, sorted(seen))
    assert len(seen) >= 2, seen


def test_operands_off_16_byte_boundaries(device):
    """A view that starts 8 bytes into a row is read by the register-staged tiles, as before."""
    g = torch.Generator().manual_seed(2)
    M, N, Kd = 40, 256, 256
    A = torch.randn(M, Kd + 8, generator=g).to(device).bfloat16()
    B = torch.randn(N, Kd, generator=g).to(device).bfloat16()
    C = torch.empty(M, N, device=device, dtype=torch.bfloat16)
    ref = torch.empty_like(C)
    K.kvop_debug_gemm(K.KVOP_BF16, K.KVOP_BF16, 0, -1, A[:, 4:], B, C, M, N, Kd, Kd + 8, Kd, N)
    K.kvop_debug_gemm(K.KVOP_BF16, K.KVOP_BF16, 0, -1, A[:, 4:Kd + 4].contiguous(), B, ref, M, N, Kd, Kd, Kd, N)
    torch.cuda.synchronize()
    assert torch.equal(C, ref)


@pytest.mark.parametrize("epi", [0, 1, 2])
@pytest.mark.parametrize("N,Kd", [(2048, 2048), (384, 320), (2080, 192), (640, 5632), (256, 64), (96, 96), (64, 36)])
def test_chosen_fp32_tile_gives_the_general_tiles_bits(device, epi, N, Kd):
    """FP32: whole and partial slabs of 128 and 64, slabs of 32 only, and no direct-load tile."""
    rng = np.random.default_rng(N + Kd + epi)
    Nc = N // 2 if epi == 2 else N
    seen = set()
    for M in (1, 16, 17, 32, 33, 64, 65, 129, 257, 513, 1100, 2049):
        A = torch.from_numpy(rng.standard_normal((M, Kd + 4)).astype(np.float32)).to(device)
        B = torch.from_numpy(rng.standard_normal((N, Kd)).astype(np.float32) * 0.05).to(device)
        C0 = torch.from_numpy(rng.standard_normal((M, Nc)).astype(np.float32)).to(device)
        outs = []
        for tile in (0, -1):
            C = C0.clone()
            K.kvop_debug_gemm(K.KVOP_F32, K.KVOP_F32, epi, tile, A, B, C, M, N, Kd, Kd + 4, Kd, Nc)
            outs.append(C)
        seen.add(K.kvop_gemm_pick_tile(K.KVOP_F32, epi, M, N, Kd))
        torch.cuda.synchronize()
        assert torch.equal(outs[0], outs[1]), (epi, M, N, Kd, sorted(seen))
    assert Kd < 2048 or len(seen) >= 4, seen
