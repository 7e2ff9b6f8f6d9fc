"""GPU: fp32 products at the sizes where the dispatch changes its tile (16 or 32 square, 64x32, 64 square) and at the edges of tiles and of
contraction tiles, against numpy in 64 bits."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

CASES = [  # M, N, K: 16x16, 32x32, then 64x64 tiles; whole, one short, one over
    (32, 32, 128), (1, 1, 1), (31, 33, 127), (65, 97, 300), (17, 15, 129),
    (512, 512, 64), (509, 423, 63), (64, 3000, 200),
    (896, 1024, 32), (1024, 1024, 64), (1021, 1019, 97),
    # 64x32 tiles; 64x64 ones; k-major rows that end inside a chunk, contractions of whole tiles and of one more
    (1024, 1024, 65), (1021, 1022, 31), (1023, 1021, 96), (1500, 901, 33), (1022, 3070, 64), (1021, 3071, 129), (717, 1307, 128),
]


@pytest.mark.parametrize("a_km,b_km", [(0, 0), (0, 1), (1, 1), (1, 0)])
@pytest.mark.parametrize("M,N,K", CASES)
def test_fp32_products(M, N, K, a_km, b_km):
    import torch
    import paper_2506_06472_amd as tio
    print(f"fp32 gemm M={M} N={N} K={K} a_km={a_km} b_km={b_km}", flush=True)
    r8 = lambda n: (n + 7) // 8 * 8
    g = torch.Generator(device="cuda").manual_seed(M + 3 * N + 7 * K)
    A = torch.randn((M, K), device="cuda", generator=g)
    B = torch.randn((N, K), device="cuda", generator=g)

    def stored(X, km):                      # padding is NaN: it must never leak
        X = X.t() if km else X
        t = torch.full((X.shape[0], r8(X.shape[1])), float("nan"), device="cuda")
        t[:, :X.shape[1]] = X
        return t
    dA, dB = stored(A, a_km), stored(B, b_km)
    bias = torch.randn(r8(N), device="cuda", generator=g)
    R = torch.randn((M, r8(N)), device="cuda", generator=g)
    C, rs = torch.full((M, r8(N)), 7.0, device="cuda"), torch.full((r8(M) + 8,), 7.0, device="cuda")
    tio.tio_op_gemm(0, "fp32", a_km, b_km, M, N, K, dA.data_ptr(), dA.shape[1], dB.data_ptr(), dB.shape[1], bias.data_ptr(),
                    R.data_ptr(), r8(N), C.data_ptr(), r8(N), rs.data_ptr())
    torch.cuda.synchronize()
    ref = (A.double() @ B.double().t() + bias[:N].double() + R[:, :N].double()).cpu().numpy()
    mag = (A.abs().double() @ B.abs().double().t()).cpu().numpy() + np.abs(ref)
    got = C.cpu().numpy().astype(np.float64)
    # one rounding of 2^-24 per addition of a chain of K products and two epilogue terms
    assert np.all(np.abs(got[:, :N] - ref) <= (K + 3) * 2.0 ** -24 * mag)
    assert np.all(got[:, N:] == 7.0)
    sums = rs.cpu().numpy().astype(np.float64)
    assert np.all(np.abs(sums[:M] - A.double().sum(1).cpu().numpy()) <= (K + 3) * 2.0 ** -24 * A.abs().double().sum(1).cpu().numpy() + 1e-30)
    assert np.all(sums[M:] == 7.0)


@pytest.mark.parametrize("M,N", [(1, (1 << 29) + 5), (1, (1 << 29) - 261), ((1 << 29) + 5, 1)])
def test_more_small_tiles_than_one_grid_has_room_for(M, N):
    """2^24 tiles of 256 threads and more are one grid too many; a contraction of one element is rounded once."""
    import torch
    import paper_2506_06472_amd as tio
    print(f"fp32 gemm M={M} N={N} K=1", flush=True)
    r8 = lambda n: (n + 7) // 8 * 8
    g = torch.Generator(device="cuda").manual_seed(1)
    A, B = torch.randn((1, r8(M)), device="cuda", generator=g), torch.randn((1, r8(N)), device="cuda", generator=g)
    C = torch.full((M, r8(N)) if M == 1 else (M, 4), 7.0, device="cuda")
    torch.cuda.synchronize()
    tio.tio_op_gemm(0, "fp32", 1, 1, M, N, 1, A.data_ptr(), A.shape[1], B.data_ptr(), B.shape[1], 0, 0, 0, C.data_ptr(), C.shape[1])
    torch.cuda.synchronize()
    want = A[0, 0] * B[0, :N] if M == 1 else A[0, :M] * B[0, 0]
    assert torch.equal(C[0, :N] if M == 1 else C[:, 0], want)
    assert (C[0, N:] == 7.0).all()
