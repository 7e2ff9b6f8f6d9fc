"""The work a user of this library has it do, as cases that can be timed and checked.

Three kinds of call reach the library's kernels:

  step       one training iteration (`Context.tio_train_step`) of a GPT- or Llama-shaped decoder: embedding, norms,
             attention, MLP, head, cross entropy, backward pass and AdamW; without migration, or under a memory cap
             with a plan (`tio_build_plan`) and pinned host memory as the slow tier at 25 GB/s per direction;
  linear     one linear layer through `tio_op_gemm`: y = x W^T (+ bias) (+ residual), and in training dx = dy W,
             dW = dy^T x and the bias gradient from the launch of dW;
  attention  one causal self-attention layer through `tio_op_attention`, forward alone or forward and backward.

Sizes are those of the repository's workloads (`synth.CONFIGS`: tiny GPT in fp32, GPT-2 small, Llama 7B and 30B widths
in bf16; the models at reduced depth, as `bench.py --layers` runs them) and ragged ones in between.
"""
import math

import torch

import paper_2506_06472_amd as tio

DEV = "cuda:0"
TYPES = {"bf16": torch.bfloat16, "fp32": torch.float32}
SLOW_TIER_BW = 25 * 10**9


def _linear(name, dtype, tokens, n_in, n_out, bias=False, resid=False, train=True, splits=1):
    return dict(name=name, kind="linear", dtype=dtype, tokens=tokens, n_in=n_in, n_out=n_out, bias=bias, resid=resid,
                train=train, splits=splits)


def _attention(name, dtype, B, T, H, dh, train=True):
    return dict(name=name, kind="attention", dtype=dtype, B=B, T=T, H=H, dh=dh, train=train)


def _step(name, arch, dtype, L, d, H, f, V, T, B, cap_frac=0.0, lr=3e-4):
    return dict(name=name, kind="step", arch=arch, dtype=dtype, L=L, d=d, H=H, f=f, V=V, T=T, B=B, cap_frac=cap_frac, lr=lr)


def listed():
    return [
        # the smallest training step the library is used for: 86 launches of a few microseconds each
        _step("step_tiny_gpt_fp32", "gpt", "fp32", 2, 128, 4, 512, 1024, 64, 2, lr=1e-3),
        # GPT-2-small widths, batch and vocabulary, two of the twelve layers, everything resident
        _step("step_gpt2_small_bf16", "gpt", "bf16", 2, 768, 12, 3072, 50257, 1024, 8),
        # the same step under a cap of 60 % of its uncapped peak: what the library exists for.  Its time is set by the
        # emulated slow tier; the kernels share the device with the copies
        _step("step_gpt2_small_capped", "gpt", "bf16", 2, 768, 12, 3072, 50257, 1024, 8, cap_frac=0.6),
        # Llama-7B widths, batch and vocabulary, one of the 32 layers: RMSNorm, RoPE, SwiGLU, head size 128
        _step("step_llama_7b_bf16", "llama", "bf16", 1, 4096, 32, 11008, 32000, 2048, 4),
        # fp32 training of a layer at GPT-2-small widths on one sequence
        _linear("linear_fp32", "fp32", 1024, 768, 3072, bias=True),
        # the first MLP layer of GPT-2 small on the whole batch (splits: what the training step takes for this dW)
        _linear("linear_gpt2_small_fc1", "bf16", 8192, 768, 3072, bias=True, splits=2),
        # gate and up projection of Llama 7B: the largest product of a layer
        _linear("linear_llama_7b_gate_up", "bf16", 8192, 4096, 22016),
        # a vocabulary of odd size as the output of a head, on a batch whose token count is odd too
        _linear("linear_ragged_head", "bf16", 1021, 768, 50257),
        # attention layers of GPT-2 small, Llama 7B (training) and Llama 30B (forward alone, as in evaluation)
        _attention("attention_gpt2_small", "bf16", 8, 1024, 12, 64),
        _attention("attention_llama_7b", "bf16", 4, 2048, 32, 128),
        _attention("attention_llama_30b_forward", "bf16", 2, 4096, 52, 128, train=False),
        # fp32 attention at the tiny workloads' head size, sequences of odd length
        _attention("attention_ragged_fp32", "fp32", 4, 333, 4, 32),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng, lo, hi):
    """Half of the sizes are whatever comes, half multiples of 64 where the range allows them."""
    n = _log_uniform(rng, lo, hi)
    return n if rng.random() < 0.5 else max(lo, n // 64 * 64)


def draw(rng):
    kind = rng.choice(["linear"] * 5 + ["attention"] * 4 + ["step"] * 3)
    if kind == "linear":
        dtype = rng.choice(["bf16", "bf16", "bf16", "fp32"])
        hi = (8192, 22016, 4e12) if dtype == "bf16" else (2048, 3072, 3e10)
        while True:
            tokens, n_in, n_out = _size(rng, 64, hi[0]), _size(rng, 128, hi[1]), _size(rng, 128, hi[1])
            if 6.0 * tokens * n_in * n_out <= hi[2]:
                break
        train = rng.random() < 0.75
        splits = rng.choice([1, 2, 4, 8]) if train and dtype == "bf16" and tokens >= 2048 and n_in * n_out < 1 << 24 else 1
        c = _linear("", dtype, tokens, n_in, n_out, rng.random() < 0.5, rng.random() < 0.5, train, splits)
    elif kind == "attention":
        dtype, dh = rng.choice([("bf16", 64), ("bf16", 128), ("bf16", 64), ("bf16", 128), ("bf16", 32), ("fp32", 32), ("fp32", 64)])
        fast = dtype == "bf16" and dh > 32
        while True:
            B, T, H = rng.randint(1, 8), _size(rng, 48, 4096 if fast else 512), _log_uniform(rng, 1, 52 if fast else 12)
            if B * H * T * T * dh <= 104 * 4096 * 4096 * 128 / 2:
                break
        c = _attention("", dtype, B, T, H, dh, rng.random() < 0.75)
    else:
        arch = rng.choice(["gpt", "llama"])
        dtype = rng.choice(["bf16", "bf16", "fp32"])
        dh = rng.choice([64, 128]) if dtype == "bf16" else 32
        H = rng.randint(2, 16 if dtype == "bf16" else 8)
        d = H * dh
        f = int(d * rng.uniform(2.6, 4.0)) // 8 * 8
        B = rng.randint(1, 4)
        T = _log_uniform(rng, 40, 1024 if dtype == "bf16" else 192) // 8 * 8 + 8 // math.gcd(B, 8)
        V = _log_uniform(rng, 500, 32000 if dtype == "bf16" else 4000)
        c = _step("", arch, dtype, rng.randint(1, 2), d, H, f, V, T, B, cap_frac=0.7 if rng.random() < 0.2 else 0.0,
                  lr=3e-4 if dtype == "bf16" else 1e-3)
    del c["name"]
    return c


# ------------------------------------------------------------------ inputs
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _normal(g, shape, dtype, std=1.0, mean=0.0):
    return (torch.randn(shape, device=DEV, generator=g) * std + mean).to(TYPES[dtype])


def _up8(n):
    return (n + 7) // 8 * 8


def _padded(g, rows, cols, dtype, std=1.0):
    """[rows, cols] values in rows of a multiple of eight elements; the padding is zero."""
    t = torch.zeros((rows, _up8(cols)), device=DEV, dtype=TYPES[dtype])
    t[:, :cols] = _normal(g, (rows, cols), dtype, std)
    return t


def _linear_inputs(c, seed):
    g = _gen(seed)
    S, n, m, dt = c["tokens"], c["n_in"], c["n_out"], c["dtype"]
    x, w = _padded(g, S, n, dt), _padded(g, m, n, dt, 0.02)          # a norm's output, weights at their initial scale
    bias = _padded(g, 1, m, dt, 0.02) if c["bias"] else None
    resid = _padded(g, S, m, dt) if c["resid"] else None
    dy = _padded(g, S, m, dt, 1e-2) if c["train"] else None
    return x, w, bias, resid, dy


def _attention_inputs(c, seed):
    g = _gen(seed)
    d = c["H"] * c["dh"]
    qkv = _normal(g, (c["B"] * c["T"], 3 * d), c["dtype"])
    do = _normal(g, (c["B"] * c["T"], d), c["dtype"], 1e-2) if c["train"] else None
    return qkv, do


def _model(c):
    # epsilon 1e-5, as the Llama models were trained with: with the usual 1e-8 the first update of a parameter whose
    # gradient is zero but for rounding (the key bias) is that rounding's sign
    return dict(arch=c["arch"], L=c["L"], d=c["d"], H=c["H"], f=c["f"], V=c["V"], T=c["T"], B=c["B"], precision=c["dtype"],
                lr=c["lr"], adam_eps=1e-5, weight_decay=0.01)


def _step_inputs(c, seed):
    """Parameters on the GPU in fp32, with the values the compute type can hold, tokens and labels on the host."""
    g = _gen(seed)
    params = {}
    for name, rows, cols in tio.tio_param_list(_model(c)):
        shape = (rows, cols) if rows > 1 else (cols,)
        gain = name.endswith("_g")
        params[name] = _normal(g, shape, c["dtype"], 0.02, 1.0 if gain else 0.0).float()
    tok = torch.randint(0, c["V"], (c["B"], c["T"] + 1), device=DEV, generator=g).cpu().numpy().astype("int32")
    return params, tok[:, :-1].copy(), tok[:, 1:].copy()


class _Step:
    """A training context with its plan, and where the plan keeps the state that stays on the GPU."""

    def __init__(self, c, seed):
        cfg = _model(c)
        params, self.tokens, self.labels = _step_inputs(c, seed)
        trace = tio.tio_trace_build(cfg)
        life = tio.tio_analyze_lifetimes(trace)
        peak = int(life.export()["M"].max())
        if c["cap_frac"]:
            cap = int(peak * c["cap_frac"]) // 256 * 256
            self.plan = tio.tio_build_plan(trace, life, cap, SLOW_TIER_BW, min_bytes=min(1 << 20, cap >> 8))
        else:
            self.plan = tio.tio_build_plan(trace, life, 2 * peak, 0)
        p = self.plan.export()
        self.ctx = tio.tio_ctx_create(cfg, max(p["arena_needed"], 1 << 16), p["host_needed"] + (1 << 16),
                                      SLOW_TIER_BW if c["cap_frac"] else 0, pool_on_device=not c["cap_frac"])
        for name in params:
            self.ctx.tio_params_load({name: params[name].cpu().numpy()})
        # persistent tensors in parameter order: weight, (fp32 master,) first and second moment; those the plan never
        # moves keep one address for the whole iteration
        moved = {e[0] for e in p["entries"]}
        at = {a[0]: a[3] for a in p["allocs"]}
        per = 4 if c["dtype"] == "bf16" else 3
        self.views = {}
        for i, (name, rows, cols) in enumerate(tio.tio_param_list(cfg)):
            for key, t in (("weight", i * per + (per - 3)), ("moment", i * per + (per - 2))):
                if t not in moved:
                    shape = (rows, cols) if rows > 1 else (cols,)
                    raw = self.ctx.arena[at[t]:at[t] + rows * cols * 4]
                    self.views[f"{name}.{key}"] = raw.view(torch.float32).view(shape)

    def run(self):
        st = self.ctx.tio_train_step(self.tokens, self.labels, self.plan)
        return {"loss": st["loss"], "state": self.views}


class _Linear:
    def __init__(self, c, seed):
        self.c = c
        self.x, self.w, self.bias, self.resid, self.dy = _linear_inputs(c, seed)
        S, n, m, t = c["tokens"], c["n_in"], c["n_out"], TYPES[c["dtype"]]
        self.y = torch.empty((S, _up8(m)), device=DEV, dtype=t)
        if c["train"]:
            self.dx = torch.empty((S, _up8(n)), device=DEV, dtype=t)
            self.dw = torch.empty((m, _up8(n)), device=DEV, dtype=t)
            self.db = torch.empty(_up8(m), device=DEV, dtype=t)
            self.ws = torch.empty(c["splits"] * (m * n + m), device=DEV) if c["splits"] > 1 else None

    def run(self):
        c = self.c
        S, n, m, dt = c["tokens"], c["n_in"], c["n_out"], c["dtype"]
        ld_n, ld_m = _up8(n), _up8(m)
        stream = torch.cuda.current_stream().cuda_stream
        ptr = lambda t: 0 if t is None else t.data_ptr()
        tio.tio_op_gemm(stream, dt, 0, 0, S, m, n, ptr(self.x), ld_n, ptr(self.w), ld_n, ptr(self.bias), ptr(self.resid), ld_m,
                        ptr(self.y), ld_m)
        out = {"y": self.y[:, :m]}
        if c["train"]:
            tio.tio_op_gemm(stream, dt, 0, 1, S, n, m, ptr(self.dy), ld_m, ptr(self.w), ld_n, 0, 0, 0, ptr(self.dx), ld_n)
            tio.tio_op_gemm(stream, dt, 1, 1, m, n, S, ptr(self.dy), ld_m, ptr(self.x), ld_n, 0, 0, 0, ptr(self.dw), ld_n,
                            ptr(self.db) if c["bias"] else 0, ptr(self.ws), c["splits"])
            out["dx"], out["dw"] = self.dx[:, :n], self.dw[:, :n]
            if c["bias"]:
                out["db"] = self.db[:m]
        return out


class _Attention:
    def __init__(self, c, seed):
        self.c = c
        self.qkv, self.do = _attention_inputs(c, seed)
        B, T, H, dh = c["B"], c["T"], c["H"], c["dh"]
        self.o = torch.empty((B * T, H * dh), device=DEV, dtype=self.qkv.dtype)
        self.lse = torch.empty((B, H, T), device=DEV)
        if c["train"]:
            self.delta = torch.empty((B, H, T), device=DEV)
            self.dqkv = torch.empty_like(self.qkv)

    def run(self):
        c = self.c
        stream = torch.cuda.current_stream().cuda_stream
        if not c["train"]:
            tio.tio_op_attention(stream, c["dtype"], c["B"], c["T"], c["H"], c["dh"], self.qkv.data_ptr(), self.o.data_ptr(),
                                 self.lse.data_ptr())
            return {"o": self.o, "lse": self.lse}
        tio.tio_op_attention(stream, c["dtype"], c["B"], c["T"], c["H"], c["dh"], self.qkv.data_ptr(), self.o.data_ptr(),
                             self.lse.data_ptr(), self.do.data_ptr(), self.delta.data_ptr(), self.dqkv.data_ptr())
        return {"o": self.o, "lse": self.lse, "dqkv": self.dqkv}


def prepare(case, seed):
    state = {"step": _Step, "linear": _Linear, "attention": _Attention}[case["kind"]](case, seed)
    torch.cuda.synchronize()
    return state


def run(state):
    return state.run()


# ------------------------------------------------------------------ what a pass cannot do without
def _weight_count(c):
    return sum(r * k for _, r, k in tio.tio_param_list(_model(c)))


def work(case):
    c = case
    e = 2 if c["dtype"] == "bf16" else 4
    if c["kind"] == "linear":
        S, n, m = c["tokens"], c["n_in"], c["n_out"]
        elems = S * n + n * m + S * m + (m if c["bias"] else 0) + (S * m if c["resid"] else 0)
        if c["train"]:
            elems += S * m + S * n + n * m + (m if c["bias"] else 0)
        return {"bytes": elems * e, "flops": (3 if c["train"] else 1) * 2.0 * S * n * m}
    if c["kind"] == "attention":
        rows, d = c["B"] * c["T"], c["H"] * c["dh"]
        flops = 2.0 * c["B"] * c["H"] * c["T"] ** 2 * c["dh"]              # the causal half of two products
        nbytes = rows * 4 * d * e + rows * c["H"] * 4
        if c["train"]:
            nbytes += rows * 4 * d * e + rows * c["H"] * 4
            flops *= 3.5
        return {"bytes": nbytes, "flops": flops}
    S, d, f, L, V = c["B"] * c["T"], c["d"], c["f"], c["L"], c["V"]
    per_layer = 4 * d * d + (2 if c["arch"] == "gpt" else 3) * d * f
    flops = 6.0 * S * (L * per_layer + V * d) + 3.5 * L * 2.0 * c["B"] * c["T"] ** 2 * d
    # AdamW reads and writes every state tensor once (bf16: master, two moments, the weight written; fp32: weight, two
    # moments); the forward pass reads the weights.  Activations could stay on chip
    return {"bytes": _weight_count(c) * (2 + 24 + 2 if c["dtype"] == "bf16" else 24 + 4), "flops": flops}


def tolerance(case):
    """About four times the largest error against `exact`: fp32 sums 1.3e-6 (single operators) and a few 1e-6 (gradients of
    a whole step); bf16 1.7e-3 (products), 2.4e-3 (attention) and 1.3e-2 (gradients of a whole step)."""
    if case["kind"] == "step":
        return {"rel": 3e-2} if case["dtype"] == "bf16" else {"rel": 2e-5}
    if case["dtype"] == "fp32":
        return {"rel": 5e-6}
    return {"rel": 7e-3} if case["kind"] == "linear" else {"rel": 1e-2}


# ------------------------------------------------------------------ the same in 64 bits
def _exact_linear(c, seed):
    x, w, bias, resid, dy = (None if t is None else t.double() for t in _linear_inputs(c, seed))
    S, n, m = c["tokens"], c["n_in"], c["n_out"]
    x, w = x[:, :n], w[:, :n]
    y = x @ w.t()
    if bias is not None:
        y += bias[0, :m]
    if resid is not None:
        y += resid[:, :m]
    out = {"y": y}
    if dy is not None:
        dy = dy[:, :m].contiguous()
        out["dx"], out["dw"] = dy @ w, dy.t().contiguous() @ x
        if c["bias"]:
            out["db"] = dy.sum(0)
    return out


def _attend(q, k, v):
    """[B, H, T, dh] each, in the type they come in; a few heads at a time."""
    T, dh = q.shape[2], q.shape[3]
    mask = torch.ones((T, T), dtype=torch.bool, device=q.device).triu(1)
    s = torch.matmul(q, k.transpose(2, 3).contiguous()).div_(math.sqrt(dh)).masked_fill_(mask, -math.inf)
    lse = torch.logsumexp(s, -1)
    return torch.matmul(torch.exp(s - lse.unsqueeze(-1)), v), lse


def _exact_attention(c, seed):
    B, T, H, dh = c["B"], c["T"], c["H"], c["dh"]
    qkv, do = _attention_inputs(c, seed)
    o = torch.empty((B, T, H, dh), device=DEV, dtype=torch.float64)
    lse = torch.empty((B, H, T), device=DEV, dtype=torch.float64)
    dqkv = torch.empty((B, T, 3, H, dh), device=DEV, dtype=torch.float64) if c["train"] else None
    heads = max(1, min(H, (1 << 28) // (T * T)))
    for b in range(B):
        for h in range(0, H, heads):
            part = qkv.view(B, T, 3, H, dh)[b, :, :, h:h + heads].double().permute(1, 2, 0, 3).contiguous()
            part = part.unsqueeze(1).requires_grad_(c["train"])                 # [3, 1, heads, T, dh]
            ob, lb = _attend(part[0], part[1], part[2])
            o[b, :, h:h + heads] = ob[0].detach().transpose(0, 1)
            lse[b, h:h + heads] = lb[0].detach()
            if c["train"]:
                go = do.view(B, T, H, dh)[b, :, h:h + heads].double().transpose(0, 1).unsqueeze(0).contiguous()
                (gp,) = torch.autograd.grad(ob, part, go)
                dqkv[b, :, :, h:h + heads] = gp[:, 0].permute(2, 0, 1, 3)
    out = {"o": o.view(B * T, H * dh), "lse": lse}
    if c["train"]:
        out["dqkv"] = dqkv.view(B * T, 3 * H * dh)
    return out


def _norm(c, x, g, b):
    if c["arch"] == "gpt":
        return torch.nn.functional.layer_norm(x, (x.shape[-1],), g, b, 1e-5)
    return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + 1e-5) * g


def _rope(x, theta=10000.0):
    """Rotation of adjacent pairs of [B, H, T, dh]."""
    T, dh = x.shape[2], x.shape[3]
    freq = theta ** (-torch.arange(0, dh, 2, device=x.device, dtype=x.dtype) / dh)
    ang = torch.arange(T, device=x.device, dtype=x.dtype)[:, None] * freq
    a, b = x[..., 0::2], x[..., 1::2]
    return torch.stack((a * ang.cos() - b * ang.sin(), a * ang.sin() + b * ang.cos()), -1).flatten(-2)


def _exact_step(c, seed):
    params, tok, lab = _step_inputs(c, seed)
    P = {k: v.double().requires_grad_() for k, v in params.items()}
    tok, lab = torch.from_numpy(tok).long().to(DEV), torch.from_numpy(lab).long().to(DEV)
    B, T, H, d, gpt = c["B"], c["T"], c["H"], c["d"], c["arch"] == "gpt"
    lin = torch.nn.functional.linear
    x = P["wte"][tok] + (P["wpe"] if gpt else 0.0)
    for i in range(c["L"]):
        l = lambda n: P.get(f"l{i}.{n}")
        n1, n2 = ("ln1", "ln2") if gpt else ("rms1", "rms2")
        qkv = lin(_norm(c, x, l(n1 + "_g"), l(n1 + "_b")), l("w_qkv"), l("b_qkv"))
        q, k, v = (t.contiguous() for t in qkv.view(B, T, 3, H, d // H).permute(2, 0, 3, 1, 4))
        if not gpt:
            q, k = _rope(q), _rope(k)
        a = _attend(q, k, v)[0].transpose(1, 2).reshape(B, T, d)
        x = x + lin(a, l("w_o"), l("b_o"))
        h = _norm(c, x, l(n2 + "_g"), l(n2 + "_b"))
        if gpt:
            u = torch.nn.functional.gelu(lin(h, l("w_fc1"), l("b_fc1")), approximate="tanh")
            x = x + lin(u, l("w_fc2"), l("b_fc2"))
        else:
            gate, up = lin(h, l("w_gu")).chunk(2, -1)
            x = x + lin(torch.nn.functional.silu(gate) * up, l("w_down"))
    h = _norm(c, x, P["lnf_g"], P["lnf_b"]) if gpt else _norm(c, x, P["rmsf_g"], None)
    loss = torch.nn.functional.cross_entropy(lin(h, P["w_head"]).view(B * T, -1), lab.view(-1))
    names = list(P)
    grads = torch.autograd.grad(loss, [P[n] for n in names])
    state = {}
    for n, g in zip(names, grads):
        w = P[n].detach()
        # first AdamW step: bias-corrected moments are the gradient and its square
        state[n + ".weight"] = w - c["lr"] * (g / (g.abs() + 1e-5) + 0.01 * w)
        state[n + ".moment"] = 0.1 * g
    return {"loss": float(loss), "state": state}      # the capped step returns the part that never leaves the GPU


def exact(case, seed):
    """What `run` returns, in 64 bits with plain torch operations."""
    return {"step": _exact_step, "linear": _exact_linear, "attention": _exact_attention}[case["kind"]](case, seed)
