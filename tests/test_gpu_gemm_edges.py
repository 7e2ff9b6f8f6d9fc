"""GPU: the bf16 product kernels at the edges of their tiles: contractions of one to a dozen tiles with every kind of remainder
(whole, a multiple of 8, odd), outputs one short of and one over a tile, every epilogue (plain, bias and residual on rows of 8k and
8k + 4 elements, row sums, split contraction with short and empty ranges), against float64; padding is NaN and must never leak.  Every
test states the output tile or the route (ranges of the contraction, one launch or two) it is about and checks that the dispatch takes it."""
import pytest

pytestmark = pytest.mark.gpu

LAYOUTS = [(0, 0), (0, 1), (1, 1), (1, 0)]
r8 = lambda n: (n + 7) // 8 * 8


def route(M, N, K, a_km, b_km, rowsum=False):
    """"rows" / "columns": two launches, the first with whole rows or columns; otherwise the ranges the contraction is cut into."""
    import paper_2506_06472_amd as tio
    ranges, rows, cols = tio.tio_op_gemm_route(a_km, b_km, M, N, K, r8(M) if a_km else r8(K), r8(N) if b_km else r8(K), rowsum)
    return "rows" if rows else "columns" if cols else ranges


def _run(M, N, K, a_km, b_km, rowsum=False, splits=1, tile=None, epilogue=(), pad=0):
    import torch
    import paper_2506_06472_amd as tio
    print(f"bf16 gemm M={M} N={N} K={K} a_km={a_km} b_km={b_km} rowsum={rowsum} splits={splits} tile={tile} epilogue={epilogue} pad={pad}",
          flush=True)
    lda, ldb, ldc = r8(M) if a_km else r8(K), r8(N) if b_km else r8(K), r8(N) + pad
    if tile:
        assert tio.tio_op_gemm_tile(a_km, b_km, M, N, K, lda, ldb, rowsum, splits) == tile
    g = torch.Generator(device="cuda").manual_seed(M + 3 * N + 7 * K + a_km + 2 * b_km)
    A = torch.randn((M, K), device="cuda", generator=g).bfloat16()
    B = torch.randn((N, K), device="cuda", generator=g).bfloat16()

    def stored(X, ld):
        t = torch.full((X.shape[0], ld), float("nan"), device="cuda", dtype=torch.bfloat16)
        t[:, :X.shape[1]] = X
        return t
    dA, dB = stored(A.t() if a_km else A, lda), stored(B.t() if b_km else B, ldb)
    C = torch.full((M, ldc), 7.0, device="cuda", dtype=torch.bfloat16)
    rs = torch.full((r8(M) + 8,), 7.0, device="cuda", dtype=torch.bfloat16)
    ws = torch.full((splits * (M * N + M) + 64,), float("nan"), device="cuda") if splits > 1 else None
    ref, mag = A.double() @ B.double().t(), A.abs().double() @ B.abs().double().t()
    bias = resid = None
    if epilogue:
        b, R = (torch.randn(n, device="cuda", generator=g).bfloat16() * 8 for n in ((1, N), (M, N)))
        if "bias" in epilogue:
            bias, ref, mag = stored(b, r8(N)), ref + b.double(), mag + b.abs().double()
        if "resid" in epilogue:
            resid, ref, mag = stored(R, ldc), ref + R.double(), mag + R.abs().double()
    tio.tio_op_gemm(0, "bf16", a_km, b_km, M, N, K, dA.data_ptr(), lda, dB.data_ptr(), ldb, bias.data_ptr() if bias is not None else 0,
                    resid.data_ptr() if resid is not None else 0, ldc, C.data_ptr(), ldc, rs.data_ptr() if rowsum else 0,
                    ws.data_ptr() if ws is not None else 0, splits)
    torch.cuda.synchronize()
    # one fp32 rounding per addition of the chain, one bf16 rounding of the result
    bound = (K + 8) * 2.0 ** -24 * mag + 2.0 ** -8 * ref.abs()
    assert ((C[:, :N].double() - ref).abs() <= bound).all() and (C[:, N:] == 7.0).all()
    if rowsum:
        s = A.double().sum(1)
        assert ((rs[:M].double() - s).abs() <= (K + 8) * 2.0 ** -24 * A.abs().double().sum(1) + 2.0 ** -8 * s.abs()).all()
        assert (rs[M:] == 7.0).all()
    if ws is not None:
        assert torch.isnan(ws[splits * (M * N + M):]).all()


@pytest.mark.parametrize("a_km,b_km", LAYOUTS)
@pytest.mark.parametrize("K", [1, 8, 31, 64, 65, 96, 127, 128, 129, 191, 192, 200, 256, 319])
def test_contraction_remainders(K, a_km, b_km):
    rowsum = K % 2 == 1                              # with row sums only k-major operands have the 64x64 tile
    _run(127, 129, K, a_km, b_km, rowsum, tile=(128, 128) if rowsum and not (a_km and b_km) else (64, 64))


# one short of and one over whole tiles; contractions from one tile (less than the ring of tiles in LDS holds) to several, as short
# as the dispatch gives each tile
@pytest.mark.parametrize("a_km,b_km", LAYOUTS)
@pytest.mark.parametrize("tile,M,N,K", [
    *(((256, 256), 8100, 8170, K) for K in (65, 96, 127, 128, 129, 191)), *(((256, 256), 3990, 4010, K) for K in (257, 319, 385)),
    *(((128, 128), 3100, 1010, K) for K in (1, 31, 64, 65, 128, 129, 191, 391)),
    *(((256, 192), 8100, 3010, K) for K in (641, 648, 703, 704)),
    *(((128, 192), 2047, 3070, K) for K in (833, 840, 896, 897, 959))])
def test_contraction_remainders_of_the_larger_tiles(tile, M, N, K, a_km, b_km):
    _run(M, N, K, a_km, b_km, tile=tile)
    if a_km and b_km:
        _run(M, N, K, a_km, b_km, rowsum=True, tile=tile)


EVERY_TILE = [((256, 256), 4096, 4096, 1024), ((256, 256), 4095, 3841, 1031), ((256, 256), 8100, 8170, 200),
              ((256, 192), 8192, 3072, 768), ((256, 192), 8100, 3070, 777),
              ((128, 192), 2047, 3072, 3000), ((128, 192), 2048, 3072, 704), ((128, 128), 4000, 1500, 640), ((128, 128), 3100, 1000, 200),
              ((128, 128), 2048, 2048, 300), ((64, 64), 500, 700, 391), ((64, 64), 1021, 768, 5025), ((64, 64), 512, 640, 384)]


@pytest.mark.parametrize("a_km,b_km", LAYOUTS)
@pytest.mark.parametrize("tile,M,N,K", EVERY_TILE)
def test_every_tile(tile, M, N, K, a_km, b_km):
    _run(M, N, K, a_km, b_km, rowsum=a_km == b_km == 1, tile=tile)


@pytest.mark.parametrize("a_km,b_km", LAYOUTS)
@pytest.mark.parametrize("pad", [0, 4])              # rows of 8k + 4 elements: output and residual move element by element
@pytest.mark.parametrize("tile,M,N,K", EVERY_TILE)
def test_every_tile_with_bias_and_residual(tile, M, N, K, pad, a_km, b_km):
    _run(M, N, K, a_km, b_km, tile=tile, epilogue=("bias", "resid"), pad=pad)


@pytest.mark.parametrize("epilogue", ["bias", "resid"])          # each set of operands has code of its own
@pytest.mark.parametrize("tile,M,N,K", EVERY_TILE)
def test_every_tile_with_bias_or_residual(tile, M, N, K, epilogue):
    _run(M, N, K, 0, 0, tile=tile, epilogue=(epilogue,))


@pytest.mark.parametrize("tile,M,N,K,splits", [
    ((64, 64), 256, 128, 1000, 3), ((64, 64), 129, 68, 517, 2), ((64, 64), 200, 136, 64, 8), ((64, 64), 130, 64, 4097, 4),
    ((128, 128), 768, 768, 2048, 8), ((256, 256), 840, 6980, 500, 2), ((128, 128), 832, 6976, 128, 2), ((256, 192), 840, 4680, 2000, 2),
    ((128, 192), 768, 3072, 8192, 2), ((128, 192), 3070, 764, 4161, 2), ((128, 192), 200, 2068, 5121, 8),
    # ranges of 640: the last of sixteen is one element long, or empty behind one of 257
    ((128, 192), 256, 1152, 9601, 16), ((128, 192), 256, 1152, 9217, 16), ((256, 192), 380, 1324, 9601, 16),
    ((256, 256), 500, 1544, 9601, 16), ((256, 256), 500, 1544, 9217, 16)])
@pytest.mark.parametrize("rowsum", [False, True])
def test_split_contraction_remainders(tile, M, N, K, splits, rowsum):
    _run(M, N, K, 1, 1, rowsum=rowsum, splits=splits, tile=tile)


@pytest.mark.parametrize("a_km,b_km", [(0, 0), (0, 1), (1, 0)])
@pytest.mark.parametrize("M,N,K", [(4096, 4096, 1024), (4095, 3841, 1031), (8100, 8170, 65)])
def test_row_sums_of_the_large_tile_in_every_layout(M, N, K, a_km, b_km):
    _run(M, N, K, a_km, b_km, rowsum=True, tile=(256, 256))


# an output of just under 2^27 elements, and of as many, which is stored past the caches: parts inside it and at its ragged ends
@pytest.mark.parametrize("M,N", [(4095, 32776), (4096, 32768), (4099, 32777)])
def test_outputs_larger_than_the_caches(M, N):
    assert route(M, N, 72, 0, 0) == 1
    _run(M, N, 72, 0, 0)


# the same in two launches, of which the first alone is under that size
def test_outputs_larger_than_the_caches_in_two_launches():
    assert route(8176, 16470, 1211, 0, 0) == "columns"
    _run(8176, 16470, 1211, 0, 0)


# products in two launches, whole rounds of tiles and what is left: cut by columns and by rows, what is left ragged and less than a tile
@pytest.mark.parametrize("M,N,K,a_km,b_km,rowsum,epilogue,pad,cut", [
    (1021, 50257, 768, 0, 0, False, ("bias", "resid"), 0, "columns"), (1021, 50261, 770, 0, 0, False, ("resid",), 4, "columns"),
    (1792, 9664, 1000, 0, 1, False, ("bias",), 0, "columns"), (50257, 768, 1021, 1, 1, True, (), 0, "rows"),
    (16001, 3130, 1161, 1, 1, True, (), 0, "columns"), (4224, 12277, 1200, 0, 0, False, (), 4, "rows"),
    (6200, 8449, 1000, 1, 0, False, ("bias", "resid"), 0, "rows"), (2508, 6720, 3968, 0, 1, False, ("bias", "resid"), 0, "columns")])
def test_products_in_two_launches(M, N, K, a_km, b_km, rowsum, epilogue, pad, cut):
    assert route(M, N, K, a_km, b_km, rowsum) == cut
    _run(M, N, K, a_km, b_km, rowsum=rowsum, epilogue=epilogue, pad=pad)
