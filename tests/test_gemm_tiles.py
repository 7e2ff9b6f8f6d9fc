"""Which output tile a bf16 product takes (host only: the choice itself, no launch)."""
import pytest

import paper_2506_06472_amd as tio


@pytest.mark.parametrize("a_km,b_km", [(0, 0), (0, 1), (1, 1), (1, 0)])
@pytest.mark.parametrize("M,N,K", [(8192, 22016, 4096), (4096, 4096, 4096), (8192, 4096, 11008)])
def test_row_sums_do_not_cost_the_large_tile(M, N, K, a_km, b_km):
    args = (a_km, b_km, M, N, K, M if a_km else K, N if b_km else K)
    assert tio.tio_op_gemm_tile(*args, rowsum=False) == (256, 256)
    assert tio.tio_op_gemm_tile(*args, rowsum=True) == (256, 256)


def test_operands_beyond_32_bit_offsets_take_no_tile():
    assert tio.tio_op_gemm_tile(1, 0, 136, 72, 8200, 65544, 8200) == (0, 0)
