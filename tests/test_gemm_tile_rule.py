"""The built-in tile choice (host only): near ties between the largest tile over a few rounds and a
smaller one go to the largest, which is the faster there."""
import pytest

from paper_2602_04430_amd import kvop as K


@pytest.mark.parametrize("epi,M,N,Kd", [(1, 17000, 2048, 2048), (1, 20000, 2048, 2048), (1, 17000, 2048, 5632),
                                        (1, 18000, 2048, 5632), (1, 20000, 2048, 5632), (0, 10000, 4096, 2048),
                                        (1, 9000, 4096, 11008), (1, 10000, 4096, 11008)])
def test_near_ties_over_several_rounds_go_to_the_largest_tile(epi, M, N, Kd):
    # times of 256x128 over 256x256: 1.03, 1.07, 1.03, 1.08, 1.15, 1.03, 1.09, 1.13
    name = K.kvop_gemm_tile_name(K.KVOP_BF16, K.kvop_gemm_pick_tile(K.KVOP_BF16, epi, M, N, Kd))
    assert name.startswith("bf16_256x256x64"), name


@pytest.mark.parametrize("M,N,Kd", [(9000, 2048, 5632), (10000, 2048, 2048)])
def test_a_clearly_faster_smaller_tile_is_kept(M, N, Kd):
    # 232 us against 253, 104 against 111: the 256x256 tile's second round is nearly empty
    name = K.kvop_gemm_tile_name(K.KVOP_BF16, K.kvop_gemm_pick_tile(K.KVOP_BF16, 1, M, N, Kd))
    assert not name.startswith("bf16_256x256x64"), name
