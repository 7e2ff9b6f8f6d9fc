"""GPU: the sums over many tokens have one order whatever their length, to the bit: the loss in 256 chains, a norm's gradients in eight.
The launchers are called through the built library's own C++ names."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
F = np.float32
FP32 = 0          # TIO_PREC_FP32


def _kernel(name, *argtypes):
    from paper_2506_06472_amd import binding, build
    binding.lib()
    f = getattr(ctypes.CDLL(build.LIB), name)
    f.argtypes, f.restype = argtypes, None
    return f


def _chains(x, n):
    """n running sums over the rows of x, row i to sum i % n, each in row order."""
    s = np.zeros((n,) + x.shape[1:], F)
    for i in range(0, len(x), n):
        rows = x[i:i + n]
        s[:len(rows)] = s[:len(rows)] + rows
    return s


# around a round of 8 and of 32 loads of a thread, and a remainder behind each
@pytest.mark.parametrize("S", [1, 2047, 2048, 2049, 2305, 8191, 8192, 8200, 18450])
def test_loss(S):
    import torch
    x = (np.random.default_rng(S).random(S) * 10).astype(F)
    s = _chains(x, 256).reshape(4, 64)
    for o in (32, 16, 8, 4, 2, 1):
        s = s + s[:, np.arange(64) ^ o]
    want = F(0)
    for w in range(4):
        want = want + s[w, 0]
    d, out = torch.from_numpy(x).cuda(), torch.full((1,), 3.0, device="cuda")
    run = _kernel("_ZN3tio1k11loss_reduceEP12ihipStream_tPKfPfllb", ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_int64,
                  ctypes.c_int64, ctypes.c_bool)
    torch.cuda.synchronize()
    run(None, d.data_ptr(), out.data_ptr(), S, 4096, False)      # a power of two: the division is exact
    torch.cuda.synchronize()
    assert out.item() == want / F(4096)


@pytest.mark.parametrize("rms", [False, True])
@pytest.mark.parametrize("rows", [1, 63, 64, 65, 127, 128, 250, 256, 257, 329, 1024, 1100])
def test_norm_gradients(rows, rms):
    import torch
    d = 104                                                      # three workgroups of 32 columns and a partial one
    part = np.random.default_rng(rows).standard_normal((rows, 1 if rms else 2, d)).astype(F)
    want = np.zeros(part.shape[1:], F)
    for chain in _chains(part, 8):
        want = want + chain
    p = torch.from_numpy(part).cuda()
    out = torch.full((2, d), 7.0, device="cuda")
    run = _kernel("_ZN3tio1k15norm_bwd_paramsEP12ihipStream_tibPKfPvS5_llb", ctypes.c_void_p, ctypes.c_int, ctypes.c_bool, ctypes.c_void_p,
                  ctypes.c_void_p, ctypes.c_void_p, ctypes.c_int64, ctypes.c_int64, ctypes.c_bool)
    torch.cuda.synchronize()
    run(None, FP32, rms, p.data_ptr(), out[0].data_ptr(), out[1].data_ptr(), rows, d, False)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    assert np.array_equal(got[:len(want)], want)
    if rms:
        assert (got[1] == 7.0).all()
