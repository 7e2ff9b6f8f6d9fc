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


@pytest.mark.parametrize("dtype,T,H,dh", [("fp32", 33, 365000, 32), ("bf16", 40, 730000, 32), ("fp32", 32, 182500, 64), ("bf16", 33, 365000, 64)])
def test_rows_whose_tile_spans_more_than_4_GiB(dtype, T, H, dh):
    """So many heads that 32-bit offsets do not reach over a tile of 32 rows: the first and the last heads have the bits they have in
    a layer of their own (bf16 with heads of 64 runs on other kernels then: fp32-rounded probabilities against bf16 ones, 2^-8 each
    for them, their gradients and the outputs)."""
    import torch
    import paper_2506_06472_amd as tio
    print(f"wide attention {dtype} T={T} H={H} dh={dh}", flush=True)
    t = torch.float32 if dtype == "fp32" else torch.bfloat16
    g = torch.Generator(device="cuda").manual_seed(T)
    qkv, dO = torch.zeros((T, 3, H, dh), device="cuda", dtype=t), torch.zeros((T, H, dh), device="cuda", dtype=t)
    ends = [slice(0, 3), slice(H // 2, H // 2 + 3), slice(H - 3, H)]
    for s in ends:
        qkv[:, :, s] = torch.randn((T, 3, 3, dh), device="cuda", generator=g).to(t)
        dO[:, s] = torch.randn((T, 3, dh), device="cuda", generator=g).to(t)

    def run(qkv, dO):
        n = dO.shape[1]
        o, dqkv = torch.full_like(dO, 7.0), torch.full_like(qkv, 7.0)
        lse, delta = (torch.full((n, T), 7.0, device="cuda") for _ in range(2))
        torch.cuda.synchronize()
        tio.tio_op_attention(0, dtype, 1, T, n, dh, qkv.data_ptr(), o.data_ptr(), lse.data_ptr(), dO.data_ptr(), delta.data_ptr(),
                             dqkv.data_ptr())
        torch.cuda.synchronize()
        return o, lse, delta, dqkv
    o, lse, delta, dqkv = run(qkv, dO)
    same = dtype == "fp32" or dh == 32
    for s in ends:
        alone = run(qkv[:, :, s].contiguous(), dO[:, s].contiguous())
        for name, a, b in zip(("o", "lse", "delta", "dqkv"), (o[:, s], lse[s], delta[s], dqkv[:, :, s]), alone):
            a, b = a.double(), b.double()
            assert torch.equal(a, b) if same else ((a - b).norm() <= 3 * 2.0 ** -8 * b.norm()).item(), (name, s)


@pytest.mark.parametrize("dtype,T,H,dh", [("fp32", 1, 2, 32), ("fp32", 7, 3, 32), ("fp32", 33, 2, 32), ("fp32", 129, 2, 32), ("fp32", 1, 2, 64),
                                          ("fp32", 65, 1, 64), ("fp32", 5, 1, 128), ("fp32", 97, 2, 128), ("bf16", 1, 2, 32), ("bf16", 33, 3, 32),
                                          ("bf16", 161, 1, 32)])
def test_what_lies_behind_the_buffers_does_not_matter(dtype, T, H, dh):
    """Tiles of 32 rows reach up to 31 rows past a sequence: behind qkv, dO and the rows of o lie zeros in one run and NaN in the other, in
    the same allocations, and every output has to be finite and the same to the bit."""
    import torch
    import paper_2506_06472_amd as tio
    print(f"attention behind the buffer {dtype} T={T} H={H} dh={dh}", flush=True)
    t, d = torch.float32 if dtype == "fp32" else torch.bfloat16, H * dh
    g = torch.Generator(device="cuda").manual_seed(T + dh)
    qkv, dO = torch.randn((T, 3 * d), device="cuda", generator=g).to(t), torch.randn((T, d), device="cuda", generator=g).to(t)
    outs = []
    for fill in (0.0, float("nan")):
        big_q, big_g, big_o = (torch.full((T + 64, n), fill, device="cuda", dtype=t) for n in (3 * d, d, d))
        big_q[:T], big_g[:T] = qkv, dO
        dqkv = torch.full((T, 3 * d), 7.0, device="cuda", dtype=t)
        lse, delta = (torch.full((H * T + 64,), fill, device="cuda") for _ in range(2))
        torch.cuda.synchronize()
        tio.tio_op_attention(0, dtype, 1, T, H, dh, big_q.data_ptr(), big_o.data_ptr(), lse.data_ptr(), big_g.data_ptr(), delta.data_ptr(),
                             dqkv.data_ptr())
        torch.cuda.synchronize()
        outs.append([big_o[:T], lse[:H * T], delta[:H * T], dqkv])
        assert torch.equal(big_o[T:].isnan(), torch.full_like(big_o[T:], fill).isnan())
    for name, a, b in zip(("o", "lse", "delta", "dqkv"), *outs):
        assert torch.isfinite(b).all() and torch.equal(a, b), name


def test_more_heads_than_one_grid_has_room_for():
    """Sequences of one token, so that o = v and dV = dO but for the rounding of a probability of one: 8.4 million blocks of dK/dV and as many of dQ, of 256 threads, where
    a grid has fewer than 2^32 of them."""
    import torch
    import paper_2506_06472_amd as tio
    B, H, dh = 1 << 13, 1032, 32
    print(f"attention B={B} T=1 H={H}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(3)
    qkv, dO = torch.randn((B, 3, H, dh), device="cuda", generator=g), torch.randn((B, H, dh), device="cuda", generator=g)
    o, dqkv = torch.full_like(dO, 7.0), torch.full_like(qkv, 7.0)
    lse, delta = (torch.full((B, H), 7.0, device="cuda") for _ in range(2))
    torch.cuda.synchronize()
    tio.tio_op_attention(0, "fp32", B, 1, H, dh, qkv.data_ptr(), o.data_ptr(), lse.data_ptr(), dO.data_ptr(), delta.data_ptr(), dqkv.data_ptr())
    torch.cuda.synchronize()
    # exp(s - max) and exp(s - lse) of |s| < 16: its rounding, 2^-21, and a few more
    assert ((o - qkv[:, 2]).abs() <= 2.0 ** -20 * qkv[:, 2].abs()).all() and ((dqkv[:, 2] - dO).abs() <= 2.0 ** -20 * dO.abs()).all()
    # P (dP - delta) is the difference of two sums of 32 products, of v and of o; dK and dQ that times q / sqrt(32) and k / sqrt(32)
    bound = (2 * 32 * 2.0 ** -24 + 2.0 ** -20) * (dO * o).abs().sum(-1, keepdim=True) / 32 ** 0.5
    assert (dqkv[:, 0].abs() <= bound * qkv[:, 1].abs() + 1e-30).all() and (dqkv[:, 1].abs() <= bound * qkv[:, 0].abs() + 1e-30).all()
