"""GPU: cross entropy at the vocabulary sizes where its kernel changes (rows of 4096 and 8192 chunks of 16 bytes, one chunk more),
and the embedding gradient with one token id in most or all positions, through one fp32 training step against the oracle."""
import numpy as np
import pytest

from gpulib import make_inputs, plans_for
from oracle import model as om

pytestmark = pytest.mark.gpu


def _step_matches(cfg, tokens=None, loss_bar=1e-5, grad_bar=1e-4, more=None):          # the bars of the fp32 parity tests
    import paper_2506_06472_amd as tio
    params, tok, lab = make_inputs(cfg, seed=1)
    if tokens is not None:
        tok = tokens(tok)
    pe = plans_for(cfg)[2].export()
    ctx = tio.tio_ctx_create(cfg, pe["arena_needed"], pe["host_needed"] + (1 << 20), 0)
    ctx.tio_params_load(params)
    loss = ctx.tio_train_step(tok, lab, None, capture_grads=True)["loss"]
    ref, grads = om.forward_backward(cfg, params, tok, lab)
    assert abs(loss - ref) <= loss_bar * abs(ref), (loss, ref)
    for n in ("w_head", "wte", "lnf_g"):
        g, r = ctx.tio_grads_read(n).astype(np.float64).ravel(), grads[n].ravel()
        assert np.abs(g - r).max() <= grad_bar * np.abs(r).max(), (n, np.abs(g - r).max() / np.abs(r).max())
    if more:
        more(ctx, grads, lab)
    ctx.close()


@pytest.mark.parametrize("V", [16384, 16385, 32768, 32769])
def test_cross_entropy_kernels_meet(V):
    print(f"vocabulary {V}", flush=True)
    _step_matches(dict(arch="gpt", L=1, d=64, H=2, f=128, V=V, T=24, B=1, precision="fp32", lr=1e-3))


# long rows of just under 2^28 bytes together, and of as many, which go past the caches
@pytest.mark.parametrize("B,V", [(255, 32768), (256, 32761)])
def test_cross_entropy_of_many_long_rows(B, V):
    print(f"vocabulary {V} batch {B}", flush=True)
    _step_matches(dict(arch="gpt", L=1, d=64, H=2, f=128, V=V, T=8, B=B, precision="fp32", lr=1e-3))


# The softmax part of the head's gradient: the columns that are no token's label, 8192 at a time (what 1024 threads hold in one register
# each).  Such a row is a sum of products of a rounded dlogits and a rounded hf, rounded again: three relative errors of at most 2^-9, and
# those of what hf is made from; 8 * 2^-9 holds all of them (measured: 1.8e-3), and eight columns without their gradient make 3e-2.
def _softmax_part(ctx, grads, lab):
    r = grads["w_head"]
    g = ctx.tio_grads_read("w_head").astype(np.float64).reshape(r.shape)
    other = np.ones(len(r), bool)
    other[lab.ravel()] = False
    for c in range(0, len(r), 8192):
        columns = np.arange(c, min(c + 8192, len(r)))
        columns = columns[other[columns]]
        assert np.linalg.norm((g - r)[columns]) <= 8 * 2.0 ** -9 * np.linalg.norm(r[columns]), c


# the same in bf16, whose rows of this length take 1024 threads.  Loss: the logits lie within 0.8 and are rounded by at most 2^-9 of that,
# each row by itself, so that the mean over 2656 rows moves by 3e-5, 3e-6 of it (measured: 1.1e-6); eight of the columns less in the sums
# make 1.5e-5.  The bar of the gradients' largest entries, which the labels' columns set, is that of the bf16 parity tests
@pytest.mark.parametrize("B", [166, 167])
def test_bf16_cross_entropy_of_many_long_rows(B):
    print(f"bf16, vocabulary 50257 batch {B}", flush=True)
    _step_matches(dict(arch="gpt", L=1, d=64, H=1, f=128, V=50257, T=16, B=B, precision="bf16", lr=1e-3), loss_bar=1e-5, grad_bar=6e-2,
                  more=_softmax_part)


@pytest.mark.parametrize("B,keep", [(1, 0), (1, 3), (20, 7), (20, 0)])
def test_embedding_gradient_of_repeated_tokens(B, keep):
    print(f"repeated tokens B={B} keep={keep}", flush=True)

    def repeat(tok):
        t = np.full_like(tok, 5)
        t.ravel()[:keep] = tok.ravel()[:keep]
        return t
    _step_matches(dict(arch="gpt", L=1, d=64, H=2, f=128, V=300, T=64, B=B, precision="fp32", lr=1e-3), repeat)


# partial rows of the norm's gradients around 128 (eight groups of rows, 32) and 256 (a whole round of loads), and losses around 2048
# (256 threads, 1024) and past a whole round of loads
@pytest.mark.parametrize("T", [1016, 1024, 2048, 2056, 2064, 8200])
def test_sums_over_many_tokens(T):
    print(f"tokens {T}", flush=True)
    _step_matches(dict(arch="gpt", L=1, d=64, H=2, f=128, V=300, T=8, B=T // 8, precision="fp32", lr=1e-3))


@pytest.mark.parametrize("precision", ["fp32", "bf16"])
@pytest.mark.parametrize("V", [16383, 16384])        # embedding and head of one row less than 2^20 parameters, and of 2^20
def test_optimizer_where_its_accesses_become_non_temporal(V, precision):
    from test_gpu_train import test_optimizer_state_follows_the_oracle_from_the_gpu_gradients as check
    check(dict(arch="gpt", L=1, d=64, H=1 if precision == "bf16" else 2, f=128, V=V, T=24, B=1, precision=precision, lr=1e-3))


# rotations where a thread takes one row, two (from 1023 rows), four, eight (from 4089), and sixteen (from 8177), whole groups of rows and
# not.  bf16: q, k and v by their norms, each rounded a handful of times by at most 2^-9 (measured: 7e-3; with the last of every eight rows
# not rotated q and k are off by 0.2 and more)
@pytest.mark.parametrize("precision,B", [*(("fp32", B) for B in (1, 127, 128, 255, 256, 257, 600, 1023, 1025)), *(("bf16", B) for B in (1, 128, 256, 600, 1025))])
def test_rotations_of_few_and_many_rows(precision, B):
    import paper_2506_06472_amd as tio
    print(f"rotations, {precision}, {8 * B} rows", flush=True)
    cfg = dict(arch="llama", L=1, d=64, H=2 if precision == "fp32" else 1, f=128, V=300, T=8, B=B, precision=precision, lr=1e-3)
    params, tok, lab = make_inputs(cfg, seed=1)
    pe = plans_for(cfg)[2].export()
    ctx = tio.tio_ctx_create(cfg, pe["arena_needed"], pe["host_needed"] + (1 << 20), 0)
    ctx.tio_params_load(params)
    loss = ctx.tio_train_step(tok, lab, None, capture_grads=True)["loss"]
    ref, grads = om.forward_backward(cfg, params, tok, lab)
    assert abs(loss - ref) <= (1e-5 if precision == "fp32" else 2e-2) * abs(ref), (loss, ref)
    r = grads["l0.w_qkv"]
    g = ctx.tio_grads_read("l0.w_qkv").astype(np.float64).reshape(r.shape)
    if precision == "fp32":
        assert np.abs(g - r).max() <= 1e-4 * np.abs(r).max(), np.abs(g - r).max() / np.abs(r).max()
    else:
        for i in (0, 64, 128):
            assert np.linalg.norm((g - r)[i:i + 64]) <= 8 * 2.0 ** -9 * np.linalg.norm(r[i:i + 64]), i
    ctx.close()
