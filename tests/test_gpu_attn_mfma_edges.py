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


# one launch for both gradients (head size 128: four wavefronts, eight) and two, beside the sizes above
@pytest.mark.parametrize("B,T,H,dh", [(2, 257, 9, 64), (4, 333, 6, 128), (1, 1025, 3, 128), (7, 300, 16, 128), (5, 129, 9, 128), (8, 261, 21, 64)])
def test_bf16_attention_gradients_in_one_launch_or_two(B, T, H, dh):
    check("bf16", B, T, H, dh, 1)


# sixteen rows to a wavefront (few workgroups of 64 rows) and thirty-two, in the forward pass and in the backward one: sequences that end in
# the first, second and last row of a wavefront's group, in either half of a tile of 32 keys, and tiles of which only later wavefronts have use
@pytest.mark.parametrize("B,T,H,dh", [(1, 16, 2, 64), (1, 17, 1, 64), (3, 31, 2, 64), (1, 81, 2, 64), (1, 97, 9, 64), (2, 176, 1, 64), (1, 16, 1, 128),
                                      (1, 17, 2, 128), (1, 47, 2, 128), (2, 81, 1, 128), (1, 113, 9, 128), (1, 240, 1, 128), (8, 177, 54, 64),
                                      (8, 273, 32, 64), (8, 257, 21, 128), (8, 145, 32, 128)])
def test_bf16_attention_rows_of_a_wavefront(B, T, H, dh):
    check("bf16", B, T, H, dh, 1)


# orders of the workgroups: all resident with every other row of units turned round (whole rows only; a row short of one), not all
# resident, heads taken eight and one at a time.  No result depends on the order: each sequence alone gives the same bits
@pytest.mark.parametrize("B,T,H,dh", [(3, 300, 11, 64), (8, 520, 13, 64), (7, 1000, 5, 64), (8, 1025, 17, 64), (8, 520, 13, 128), (8, 4096, 9, 128)])
def test_bf16_attention_does_not_depend_on_the_order_of_its_blocks(B, T, H, dh):
    import torch
    import paper_2506_06472_amd as tio
    print(f"attention order B={B} T={T} H={H} dh={dh}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(T + H)
    d = H * dh
    qkv = torch.randn((B, T, 3 * d), device="cuda", generator=g).bfloat16()
    dO = torch.randn((B, T, d), device="cuda", generator=g).bfloat16()

    def run(qkv, dO):
        n = qkv.shape[0]
        o, dqkv = torch.full_like(dO, 7.0), torch.full_like(qkv, 7.0)
        lse, delta = (torch.full((n, H, T), 7.0, device="cuda") for _ in range(2))
        tio.tio_op_attention(0, "bf16", n, T, H, dh, qkv.data_ptr(), o.data_ptr(), lse.data_ptr(), dO.data_ptr(), delta.data_ptr(),
                             dqkv.data_ptr())
        torch.cuda.synchronize()
        return o, lse, dqkv
    whole = run(qkv, dO)
    for b in range(B):
        for name, w, one in zip(("o", "lse", "dqkv"), whole, run(qkv[b:b + 1].contiguous(), dO[b:b + 1].contiguous())):
            assert torch.equal(w[b], one[0]), (name, b)


# one launch for both gradients (head size 128: four wavefronts, eight) and two; sequences that end inside a tile of 64 rows and inside a
# workgroup's first tiles, and a whole one
@pytest.mark.parametrize("B,T,H,dh", [(2, 333, 3, 64), (1, 50, 2, 64), (8, 1000, 9, 64), (2, 320, 1, 64), (2, 333, 3, 128), (1, 50, 2, 128),
                                      (4, 300, 16, 128), (8, 1000, 20, 128), (2, 384, 1, 128)])
def test_gradients_of_keys_at_minus_infinity(B, T, H, dh):
    """A key whose scores are all -inf takes part in nothing: dK and dV are those of a key far below every other.  The forward pass
    rescales at other tiles then, which changes the rounding of probabilities, their gradients and the outputs to bf16: 2^-8 each."""
    import torch
    import paper_2506_06472_amd as tio
    print(f"attention, infinite keys B={B} T={T} H={H} dh={dh}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(T + H)
    x = torch.randn((B, T, 3, H, dh), device="cuda", generator=g)
    x[:, :, 0, :, 5] = x[:, :, 0, :, 5].abs() + 0.25
    keys = sorted({1, T // 2, T - 2})
    dO = torch.randn((B, T, H * dh), device="cuda", generator=g).bfloat16()

    def run(value):
        q = x.clone()
        q[:, keys, 1, :, 5] = value
        q = q.bfloat16().contiguous()
        o, dqkv = torch.full_like(dO, 7.0), torch.full_like(q, 7.0)
        lse, delta = (torch.full((B, H, T), 7.0, device="cuda") for _ in range(2))
        torch.cuda.synchronize()
        tio.tio_op_attention(0, "bf16", B, T, H, dh, q.data_ptr(), o.data_ptr(), lse.data_ptr(), dO.data_ptr(), delta.data_ptr(), dqkv.data_ptr())
        torch.cuda.synchronize()
        return o, lse, dqkv[:, :, 1:]
    for name, a, b in zip(("o", "lse", "dk, dv"), run(float("-inf")), run(-1e30)):
        assert torch.isfinite(a).all(), name
        a, b = a.double(), b.double()
        assert ((a - b).norm() <= 3 * 2.0 ** -8 * b.norm()).item(), name


# one launch for both gradients and two, delta in the launch of dQ, of both, in one of its own; o at the start, the end and across
@pytest.mark.parametrize("dtype,B,T,H,dh", [("bf16", 2, 333, 3, 64), ("bf16", 8, 1000, 9, 64), ("bf16", 4, 300, 16, 128), ("bf16", 8, 1000, 20, 128),
                                            ("bf16", 2, 200, 3, 32), ("fp32", 2, 333, 3, 32), ("fp32", 2, 200, 3, 64)])
@pytest.mark.parametrize("at", [0, 2, "across"])
def test_gradients_written_over_the_output(dtype, B, T, H, dh, at):
    """o may lie where dqkv goes: the backward pass has the bits that it has with buffers of their own."""
    import torch
    import paper_2506_06472_amd as tio
    print(f"attention, dqkv over o {dtype} B={B} T={T} H={H} dh={dh}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(T + H)
    t, n = torch.float32 if dtype == "fp32" else torch.bfloat16, B * T * H * dh
    qkv, dO = torch.randn(3 * n, device="cuda", generator=g).to(t), torch.randn(n, device="cuda", generator=g).to(t)
    outs = []
    for alone in (True, False):
        buf = torch.full((4 * n,), 7.0, device="cuda", dtype=t)
        dqkv = buf[:3 * n]
        o = buf[3 * n:] if alone else buf[n * at:] if at != "across" else buf[3 * n - 64:]
        lse, delta = (torch.full((B * H * T,), 7.0, device="cuda") for _ in range(2))
        torch.cuda.synchronize()
        tio.tio_op_attention(0, dtype, B, T, H, dh, qkv.data_ptr(), o.data_ptr(), lse.data_ptr(), dO.data_ptr(), delta.data_ptr(), dqkv.data_ptr())
        torch.cuda.synchronize()
        outs.append((dqkv.clone(), lse, delta))
    for name, a, b in zip(("dqkv", "lse", "delta"), *outs):
        assert torch.equal(a, b), name
