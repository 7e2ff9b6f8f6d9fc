"""GPU: the AdamW update has one rounding for each sum, the one written in the kernel, to the bit: m = fma(1 - b1, g, b1 m),
v = fma((1 - b2) g, g, b2 v), theta = fma(-lr, fma(wd, theta, m / bc1 / (sqrt(v / bc2) + eps)), theta).  The launcher is called through the
built library's own C++ name."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
F = np.float32


class _Tensor(ctypes.Structure):
    _fields_ = [("g", ctypes.c_void_p), ("w", ctypes.c_void_p), ("master", ctypes.c_void_p), ("m", ctypes.c_void_p), ("v", ctypes.c_void_p),
                ("n", ctypes.c_int64)]


def _fma(a, b, c):
    """Exact product, sum to 64 bits of mantissa, then to fp32 (that the first rounding decides the second is a matter of 2^-40)."""
    return (np.longdouble(a) * np.longdouble(b) + np.longdouble(c)).astype(F)


def _want(t, g, lr, b1, b2, eps, wd, bc1, bc2):
    th, m, v = t
    m = _fma(F(1) - b1, g, b1 * m)
    v = _fma((F(1) - b2) * g, g, b2 * v)
    q = m * (F(1) / bc1) / (np.sqrt(v * (F(1) / bc2)) + eps)
    return _fma(-lr, _fma(wd, th, q), th), m, v


# ordinary and non-temporal accesses, each with a remainder behind the groups of four, in one launch and alone
@pytest.mark.parametrize("sizes", [(64,), (1000, 3, 1 << 20), (1003,), ((1 << 20) + 6,), (7, (1 << 20) + 4, 130, 8, 64, 1, 2, 512)])
@pytest.mark.parametrize("precision", ["fp32", "bf16"])
def test_update(precision, sizes):
    import torch
    from paper_2506_06472_amd import binding, build
    binding.lib()
    run = ctypes.CDLL(build.LIB)["_ZN3tio1k5adamwEP12ihipStream_tiPKNS0_11AdamwTensorEifffffff"]
    run.argtypes, run.restype = [ctypes.c_void_p, ctypes.c_int, ctypes.c_void_p, ctypes.c_int] + [ctypes.c_float] * 7, None
    bf16 = precision == "bf16"
    rng = np.random.default_rng(sum(sizes))
    hyper = [F(x) for x in (3e-4, 0.9, 0.999, 1e-8, 0.01, 1 - 0.9 ** 3, 1 - 0.999 ** 3)]
    dev, state, grads = [], [], []
    for n in sizes:
        th, m = rng.standard_normal(n).astype(F), (rng.standard_normal(n) * 1e-3).astype(F)
        v = (rng.random(n) * 1e-6).astype(F)
        g = torch.from_numpy((rng.standard_normal(n) * 1e-3).astype(F))
        g = g.bfloat16() if bf16 else g
        grads.append(g.float().numpy())
        state.append((th, m, v))
        d = [g.cuda(), *(torch.from_numpy(x.copy()).cuda() for x in (th, m, v))]
        dev.append(d + ([torch.zeros(n, device="cuda", dtype=torch.bfloat16)] if bf16 else []))
    batch = (_Tensor * len(sizes))(*(
        _Tensor(d[0].data_ptr(), d[4].data_ptr() if bf16 else d[1].data_ptr(), d[1].data_ptr() if bf16 else None, d[2].data_ptr(), d[3].data_ptr(), n)
        for d, n in zip(dev, sizes)))
    torch.cuda.synchronize()
    run(None, binding.PREC[precision], batch, len(sizes), *hyper)
    torch.cuda.synchronize()
    for d, t, g, n in zip(dev, state, grads, sizes):
        want = _want(t, g, *hyper)
        for name, w, a in zip(("theta", "m", "v"), want, d[1:4]):
            assert np.array_equal(a.cpu().numpy(), w), (name, n)
        if bf16:
            assert torch.equal(d[4].cpu(), torch.from_numpy(want[0]).bfloat16())
