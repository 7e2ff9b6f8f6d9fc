"""GPU: the bf16 product kernel at the edges of its tiles: contractions of 1 to 4 tiles with every kind of remainder (whole,
a multiple of 8, odd), outputs one short of and one over a tile, with and without row sums and split contraction, against
float64; padding is NaN and must never leak."""
import pytest

pytestmark = pytest.mark.gpu


r8 = lambda n: (n + 7) // 8 * 8


def _tile(M, N, K, a_km, b_km, rowsum, splits=1):
    import paper_2506_06472_amd as tio
    return tio.tio_op_gemm_tile(a_km, b_km, M, N, K, r8(M) if a_km else r8(K), r8(N) if b_km else r8(K), rowsum, splits)


def _run(M, N, K, a_km, b_km, rowsum, splits=1):
    import torch
    import paper_2506_06472_amd as tio
    print(f"bf16 gemm M={M} N={N} K={K} a_km={a_km} b_km={b_km} rowsum={rowsum} splits={splits}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(M + 3 * N + 7 * K + a_km + 2 * b_km)
    A = torch.randn((M, K), device="cuda", generator=g).bfloat16()
    B = torch.randn((N, K), device="cuda", generator=g).bfloat16()

    def stored(X, km):
        X = X.t() if km else X
        t = torch.full((X.shape[0], r8(X.shape[1])), float("nan"), device="cuda", dtype=torch.bfloat16)
        t[:, :X.shape[1]] = X
        return t
    dA, dB = stored(A, a_km), stored(B, b_km)
    C = torch.full((M, r8(N)), 7.0, device="cuda", dtype=torch.bfloat16)
    rs = torch.full((r8(M) + 8,), 7.0, device="cuda", dtype=torch.bfloat16)
    ws = torch.full((splits * (M * N + M) + 64,), float("nan"), device="cuda") if splits > 1 else None
    tio.tio_op_gemm(0, "bf16", a_km, b_km, M, N, K, dA.data_ptr(), dA.shape[1], dB.data_ptr(), dB.shape[1], 0, 0, 0, C.data_ptr(),
                    r8(N), rs.data_ptr() if rowsum else 0, ws.data_ptr() if ws is not None else 0, splits)
    torch.cuda.synchronize()
    ref, mag = A.double() @ B.double().t(), A.abs().double() @ B.abs().double().t()
    # one fp32 rounding per addition of the chain, one bf16 rounding of the result
    bound = (K + 8) * 2.0 ** -24 * mag + 2.0 ** -8 * ref.abs()
    assert ((C[:, :N].double() - ref).abs() <= bound).all() and (C[:, N:] == 7.0).all()
    if rowsum:
        s = A.double().sum(1)
        assert ((rs[:M].double() - s).abs() <= (K + 8) * 2.0 ** -24 * A.abs().double().sum(1) + 2.0 ** -8 * s.abs()).all()
        assert (rs[M:] == 7.0).all()
    if ws is not None:
        assert torch.isnan(ws[splits * (M * N + M):]).all()


@pytest.mark.parametrize("a_km,b_km", [(0, 0), (0, 1), (1, 1), (1, 0)])
@pytest.mark.parametrize("K", [1, 8, 31, 64, 65, 96, 127, 128, 129, 191, 192, 200, 256, 319])
def test_contraction_remainders(K, a_km, b_km):
    _run(127, 129, K, a_km, b_km, rowsum=K % 2 == 1)


# output sizes that get each of the tiles: 256x256, 256x192, 128x192, 128x128, 64x64
@pytest.mark.parametrize("a_km,b_km", [(0, 0), (0, 1), (1, 1), (1, 0)])
@pytest.mark.parametrize("M,N,K", [(4096, 4096, 1024), (4095, 3841, 1031), (8192, 3072, 768), (8100, 3070, 777), (2047, 3072, 3000),
                                   (4000, 1500, 640), (3100, 1000, 200), (2048, 2048, 300), (500, 700, 391), (1021, 768, 5025)])
def test_every_tile(M, N, K, a_km, b_km):
    _run(M, N, K, a_km, b_km, rowsum=a_km == b_km == 1)


@pytest.mark.parametrize("M,N,K,splits", [(256, 128, 1000, 3), (129, 68, 517, 2), (200, 136, 64, 8), (130, 64, 4097, 4)])
def test_split_contraction_remainders(M, N, K, splits):
    _run(M, N, K, 1, 1, rowsum=True, splits=splits)


@pytest.mark.parametrize("a_km,b_km", [(0, 0), (0, 1), (1, 0)])
@pytest.mark.parametrize("M,N,K", [(4096, 4096, 1024), (4095, 3841, 1031)])
def test_row_sums_of_the_large_tile_in_every_layout(M, N, K, a_km, b_km):
    assert _tile(M, N, K, a_km, b_km, True) == (256, 256)
    _run(M, N, K, a_km, b_km, rowsum=True)
