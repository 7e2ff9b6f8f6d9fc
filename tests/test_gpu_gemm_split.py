"""GPU: bf16 products whose long contraction is cut into ranges without a workspace from the caller: edges of rows, ranges and
epilogues against float64 (the comparison and its bound are those of test_gpu_gemm_edges), the bits of the same cut with a caller's
workspace, and the scratch space under more streams than it has parts, under threads, and under graph capture."""
import threading

import pytest
from test_gpu_gemm_edges import _run, r8, route

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K,a_km,b_km,rowsum,epilogue,pad", [
    (200, 300, 15000, 0, 0, False, (), 0), (199, 301, 15001, 0, 1, False, ("bias", "resid"), 0), (65, 1022, 22017, 0, 1, False, ("resid",), 4),
    (1, 1, 20000, 0, 0, False, ("bias",), 0), (3, 7, 16385, 1, 0, False, ("bias", "resid"), 4), (300, 301, 15999, 1, 1, True, (), 0),
    (512, 130, 30011, 1, 1, True, (), 0), (1021, 768, 50257, 0, 1, False, (), 0)])
def test_long_contractions(M, N, K, a_km, b_km, rowsum, epilogue, pad):
    assert route(M, N, K, a_km, b_km, rowsum) == 8
    _run(M, N, K, a_km, b_km, rowsum=rowsum, epilogue=epilogue, pad=pad)


# two, four and eight ranges with 45 to 64 MiB of partials, ragged and not, row sums behind them; the last is next to the line and not cut
@pytest.mark.parametrize("M,N,K,a_km,b_km,rowsum,epilogue,ranges", [
    (4096, 1792, 12940, 0, 1, False, (), 2), (4093, 1790, 12941, 0, 1, False, ("bias", "resid"), 2), (4096, 1024, 32000, 0, 1, False, (), 4),
    (3330, 1791, 16001, 1, 1, True, (), 2), (2300, 1791, 24001, 1, 1, True, (), 4), (1536, 1280, 24001, 1, 1, True, (), 8),
    (2050, 2047, 16001, 1, 1, True, (), 1)])
def test_large_partials(M, N, K, a_km, b_km, rowsum, epilogue, ranges):
    assert route(M, N, K, a_km, b_km, rowsum) == ranges
    _run(M, N, K, a_km, b_km, rowsum=rowsum, epilogue=epilogue)


class _Product:
    def __init__(self, torch, M, N, K, seed):
        g = torch.Generator(device="cuda").manual_seed(seed)
        self.torch, self.M, self.N, self.K = torch, M, N, K
        self.A = torch.randn((M, r8(K)), device="cuda", generator=g).bfloat16()
        self.B = torch.randn((N, r8(K)), device="cuda", generator=g).bfloat16()

    def run(self, out, stream=0, ws=None, splits=1):
        import paper_2506_06472_amd as tio
        tio.tio_op_gemm(stream, "bf16", 0, 0, self.M, self.N, self.K, self.A.data_ptr(), self.A.shape[1], self.B.data_ptr(), self.B.shape[1],
                        0, 0, 0, out.data_ptr(), out.shape[1], 0, ws.data_ptr() if ws is not None else 0, splits)

    def out(self):
        return self.torch.empty((self.M, r8(self.N)), device="cuda", dtype=self.torch.bfloat16)


def test_the_cut_is_the_one_a_caller_can_ask_for():
    import torch
    p = _Product(torch, 200, 304, 15000, 1)
    a, b = p.out(), p.out()
    p.run(a)
    p.run(b, ws=torch.empty(8 * (200 * 304 + 200), device="cuda"), splits=8)
    torch.cuda.synchronize()
    assert torch.equal(a, b)


def test_streams_and_threads_do_not_share_partials():
    import torch
    products = [_Product(torch, 200 + 8 * i, 304, 15000, i) for i in range(6)]
    want = [p.out() for p in products]
    for p, w in zip(products, want):
        p.run(w)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in products]          # more than the scratch space has parts
    got = [[p.out() for _ in range(4)] for p in products]
    for j in range(4):
        for i, p in enumerate(products):
            p.run(got[i][j], streams[(i + j) % 6].cuda_stream)
    torch.cuda.synchronize()
    for w, outs in zip(want, got):
        assert all(torch.equal(w, o) for o in outs)
    # threads: four on one stream, two on streams of their own
    for outs in got:
        for o in outs:
            o.zero_()
    torch.cuda.synchronize()

    def work(i):
        for o in got[i]:
            products[i].run(o, streams[0 if i < 4 else i].cuda_stream)
    threads = [threading.Thread(target=work, args=(i,)) for i in range(6)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    for w, outs in zip(want, got):
        assert all(torch.equal(w, o) for o in outs)


def test_under_graph_capture():
    """A captured product keeps to one range, so that its replays use no scratch space that others may be using: it does not have the
    bits of the cut (eager) product, and has the same ones in every replay while cut products of six other streams are under way."""
    import torch
    p = _Product(torch, 200, 304, 15000, 5)
    ref = p.A[:, :p.K].double() @ p.B[:, :p.K].double().t()
    mag = p.A[:, :p.K].abs().double() @ p.B[:, :p.K].abs().double().t()
    bound = (p.K + 8) * 2.0 ** -24 * mag + 2.0 ** -8 * ref.abs()
    out, eager = p.out(), p.out()
    p.run(out)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        p.run(out, torch.cuda.current_stream().cuda_stream)
    others = [_Product(torch, 200 + 8 * i, 304, 15000, 10 + i) for i in range(6)]
    want = [q.out() for q in others]
    for q, w in zip(others, want):
        q.run(w)
    got = [q.out() for q in others]
    streams = [torch.cuda.Stream() for _ in others]
    first = None
    for _ in range(4):
        out.zero_()
        for g in got:
            g.zero_()
        torch.cuda.synchronize()
        for when in (0, 1):
            for q, g, s in zip(others, got, streams):
                q.run(g, s.cuda_stream)
            if when == 0:
                graph.replay()
                p.run(eager, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        for o in (out, eager):
            assert ((o[:, :304].double() - ref).abs() <= bound).all()
        first = out.clone() if first is None else first
        assert torch.equal(out, first)
        assert not torch.equal(out, eager)
        assert all(torch.equal(w, g) for w, g in zip(want, got))


def test_cut_products_of_all_sizes_on_many_streams():
    import torch
    products = [_Product(torch, M, N, K, i) for i, (M, N, K) in enumerate(
        [(200, 304, 15000), (4096, 1792, 12940), (216, 304, 15000), (4096, 1024, 32000), (232, 304, 15000), (2304, 1280, 16000)])]
    assert all(route(p.M, p.N, p.K, 0, 0) > 1 for p in products)
    want = [p.out() for p in products]
    for p, w in zip(products, want):
        p.run(w)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in products]
    got = [[p.out() for _ in range(3)] for p in products]
    for j in range(3):
        for i, p in enumerate(products):
            p.run(got[i][j], streams[(i + j) % 6].cuda_stream)
    torch.cuda.synchronize()
    for w, outs in zip(want, got):
        assert all(torch.equal(w, o) for o in outs)
