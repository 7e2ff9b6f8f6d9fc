"""GPU: the fp32-arithmetic attention kernels at the edges of their 32-row blocks and of the four wavefronts that share a
block's tiles, with a head count that is no multiple of the eight XCDs; the oracle, the comparison and its bounds are those of
test_gpu_ops.test_attention_forward_backward."""
import pytest
from test_gpu_ops import test_attention_forward_backward as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,B,T,H,dh", [
    ("fp32", 1, 1, 1, 32), ("fp32", 1, 31, 9, 32), ("fp32", 2, 32, 2, 64), ("fp32", 1, 33, 3, 128), ("fp32", 1, 128, 1, 32),
    ("fp32", 1, 161, 3, 64), ("bf16", 1, 1, 1, 32), ("bf16", 3, 65, 3, 32), ("bf16", 1, 300, 2, 32),
    # four and eight wavefronts to a block: up to four tiles, five, more than eight; more workgroups than eight are taken for
    ("fp32", 1, 129, 8, 32), ("fp32", 2, 289, 4, 32), ("fp32", 8, 160, 8, 32), ("fp32", 3, 192, 1, 128)])
def test_fp32_attention_edges(dtype, B, T, H, dh):
    check(dtype, B, T, H, dh, 1)


def test_scores_of_minus_infinity():
    """A key whose score is -inf takes no part; the rows that see only such keys are as they were before (no finite value)."""
    import torch
    import paper_2506_06472_amd as tio
    T, dh = 70, 32
    g = torch.Generator(device="cuda").manual_seed(3)
    qkv = torch.randn((T, 3 * dh), device="cuda", generator=g)
    qkv[:, 0] = qkv[:, 0].abs() + 0.1
    qkv[:40, dh] = float("-inf")
    o, lse = torch.full((T, dh), 7.0, device="cuda"), torch.zeros(T, device="cuda")
    tio.tio_op_attention(0, "fp32", 1, T, 1, dh, qkv.data_ptr(), o.data_ptr(), lse.data_ptr())
    torch.cuda.synchronize()
    q, k, v = (x.double() for x in qkv.split(dh, 1))
    s = (q @ k.t() / dh ** 0.5).masked_fill(torch.ones((T, T), device="cuda").triu(1).bool(), float("-inf"))
    p = torch.softmax(s[40:], -1)
    assert (o[40:] - p @ v).abs().max() < 1e-5 and (lse[40:] - torch.logsumexp(s[40:], -1)).abs().max() < 1e-5
    assert not torch.isfinite(o[:40]).any() and (lse[:40] == float("-inf")).all()
