"""GPU: bf16 attention on the matrix cores at the edges of the key blocks of its backward pass (128 rows at head size 64, 256 at
head size 128) with a head count that is no multiple of the eight XCDs; oracle, comparison and bounds are those of
test_gpu_ops.test_attention_forward_backward."""
import pytest
from test_gpu_ops import test_attention_forward_backward as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,T,H,dh", [(1, 1, 1, 128), (1, 33, 9, 128), (2, 255, 1, 128), (1, 256, 3, 128), (1, 257, 2, 128),
                                      (1, 500, 1, 128), (1, 129, 9, 64), (1, 255, 2, 64)])
def test_bf16_attention_edges(B, T, H, dh):
    check("bf16", B, T, H, dh, 1)


# the loops over the tiles on the diagonal and the others: none of the others, one, a partial one
@pytest.mark.parametrize("B,T,H,dh", [(1, 64, 3, 64), (1, 128, 9, 64), (1, 192, 2, 64), (2, 321, 1, 64), (1, 64, 1, 128), (1, 128, 2, 128),
                                      (1, 320, 9, 128), (2, 321, 1, 128), (1, 577, 1, 128)])
def test_bf16_attention_tiles_on_and_off_the_diagonal(B, T, H, dh):
    check("bf16", B, T, H, dh, 1)
