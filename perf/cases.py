"""The work that a user has this framework do, as measurable cases.

A case is a dict of plain values; its "kind" says which public path one pass
takes:

  f32      one calibration step of a single fp32 linear layer
  step     one calibration step of a dense decoder block (DenseBlock.step)
  linear   a bf16 fake-ternary linear layer: forward, backward to its input and
           to the modulation factors
  mlp      the MLP half of a dense block, forward and backward
  attn     causal grouped-query attention, forward and backward
  moe      a routed-expert MLP: routing, forward and backward
  weights  the passes over a block's weights alone: group statistics with the
           softened ternarisation, then the final ternarisation and packing
  ternary  the deployment product on the 2-bit storage, over a block's layers

``exact`` is plain torch in 64 bits on the same inputs, written from the
paper's equations; it uses nothing of the package.
"""
from __future__ import annotations

import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_2606_26650_amd as lib
from paper_2606_26650_amd.block import DenseBlock

DEV = "cuda"
DELTA0, EPS = 0.5, 1e-6


# ------------------------------------------------------------------- cases

def listed():
    return [
        # the smallest calibration: one 256 x 256 fp32 linear, 8 samples of 128 tokens
        dict(name="f32-256", kind="f32", M=1024, N=256, K=256),
        # a block small enough that launches and host work are what counts; ragged tiles
        dict(name="step-small", kind="step", batch=2, seq=80, hidden=256, n_q=4, n_kv=2, d=64,
             ffn=384, qk_norm=True, hard=False, a8=False, input_grad=True),
        # a Qwen3-1.7B-shaped block on the paper's calibration batch, 3 samples of 2048 tokens
        dict(name="step-1.7b", kind="step", batch=3, seq=2048, hidden=2048, n_q=16, n_kv=8, d=128,
             ffn=6144, qk_norm=True, hard=False, a8=False, input_grad=False),
        # the benchmark's block: Qwen3-14B-shaped, 2 samples of 4096 tokens
        dict(name="step-14b", kind="step", batch=2, seq=4096, hidden=5120, n_q=40, n_kv=8, d=128,
             ffn=17408, qk_norm=True, hard=False, a8=False, input_grad=False),
        # an output projection (Llama-3-8B-shaped) on samples whose length is no tile multiple
        dict(name="linear-ragged", kind="linear", M=3000, N=4096, K=4096, res=True, hard=False),
        # one short sample through a fused q|k|v projection, in the hard epochs
        dict(name="linear-short", kind="linear", M=512, N=4096, K=2048, res=False, hard=True),
        # the MLP of a Llama-3-8B-shaped block on one sample
        dict(name="mlp-8b", kind="mlp", M=2048, h=4096, F=14336),
        # attention with 64-wide heads, no q/k norm, a sample length that is no tile multiple
        dict(name="attn-ragged", kind="attn", batch=3, seq=1000, n_q=16, n_kv=4, d=64,
             qk_norm=False, a8=False),
        # routed experts of a middling size, a ragged token count
        dict(name="moe", kind="moe", T=3000, h=2048, F=768, E=64, k=8),
        # all weights of a Qwen3-1.7B-shaped block: start and end of a calibration
        dict(name="weights-1.7b", kind="weights", rows=393216 // 16, cols=2048, g=128),
        # generating one token with a Qwen3-14B-shaped block's packed layers
        dict(name="ternary-decode", kind="ternary", M=1, hidden=5120, qkv=7168, ffn=17408,
             out_f32=False),
        # reading a prompt of 1000 tokens with the same layers
        dict(name="ternary-prefill", kind="ternary", M=1000, hidden=5120, qkv=7168, ffn=17408,
             out_f32=False),
    ]


def _log(rng, lo, hi, step=1):
    """An integer multiple of ``step`` from lo to hi, even over the logarithm."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(lo, min(hi, int(round(v / step)) * step))


def draw(rng):
    kind = rng.choice(["f32", "step", "linear", "mlp", "attn", "moe", "weights", "ternary"])
    if kind == "f32":
        return dict(kind=kind, M=_log(rng, 64, 4096), N=_log(rng, 128, 1024, 8),
                    K=_log(rng, 128, 1024, 128))
    if kind == "step":
        d = rng.choice([64, 128])
        n_kv = rng.choice([1, 2, 4, 8])
        n_q = n_kv * rng.choice([1, 2, 4])
        return dict(kind=kind, batch=rng.randint(1, 4), seq=_log(rng, 64, 2048, 8),
                    hidden=_log(rng, 256, 4096, 128), n_q=n_q, n_kv=n_kv, d=d if n_q * d >= 128 else 128,
                    ffn=_log(rng, 256, 12288, 128), qk_norm=rng.random() < 0.5,
                    hard=rng.random() < 0.25, a8=rng.random() < 0.25,
                    input_grad=rng.random() < 0.5)
    if kind == "linear":
        return dict(kind=kind, M=_log(rng, 64, 8192), N=_log(rng, 256, 8192, 8),
                    K=_log(rng, 256, 8192, 128), res=rng.random() < 0.5, hard=rng.random() < 0.25)
    if kind == "mlp":
        return dict(kind=kind, M=_log(rng, 64, 6144), h=_log(rng, 256, 5120, 128),
                    F=_log(rng, 384, 17408, 128))
    if kind == "attn":
        n_kv = rng.choice([1, 2, 4, 8])
        return dict(kind=kind, batch=rng.randint(1, 4), seq=_log(rng, 32, 4096, 8),
                    n_q=n_kv * rng.choice([1, 2, 4, 5]), n_kv=n_kv, d=rng.choice([64, 128]),
                    qk_norm=rng.random() < 0.5, a8=rng.random() < 0.2)
    if kind == "moe":
        E = rng.choice([8, 16, 32, 64, 128])
        return dict(kind=kind, T=_log(rng, 64, 4096), h=_log(rng, 256, 4096, 128),
                    F=_log(rng, 128, 1536, 128), E=E, k=rng.choice([1, 2, 4, 8]))
    if kind == "weights":
        return dict(kind=kind, rows=_log(rng, 16, 32768), cols=_log(rng, 512, 8192, 512),
                    g=rng.choice([64, 128, 128, 256]))
    return dict(kind=kind, M=_log(rng, 1, 2048), hidden=_log(rng, 512, 5120, 128),
                qkv=_log(rng, 512, 8192, 16), ffn=_log(rng, 512, 17408, 128),
                out_f32=rng.random() < 0.25)


# ------------------------------------------------------------ inputs (torch)

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _normal(g, shape, std=1.0, dtype=torch.bfloat16):
    return (torch.randn(shape, generator=g, device=DEV, dtype=torch.float32) * std).to(dtype)


def _acts(g, shape):
    """Calibration activations, Student-t with four degrees of freedom."""
    z = torch.randn(shape, generator=g, device=DEV)
    c = sum(torch.randn(shape, generator=g, device=DEV).square() for _ in range(4))
    return (z / (c / 4).sqrt()).to(torch.bfloat16)


def _factors(g, n):
    """Factors in the middle of a calibration, around the identity modulation."""
    u = torch.rand((3, n), generator=g, device=DEV) * 0.6 - 0.3
    return u[0].contiguous(), u[1].exp(), u[2].exp()


def _sharpness(case):
    return (lib.HARD, 0.0) if case.get("hard") else (lib.SOFT, 15.0)


def _params(case, g=128):
    mode, s = _sharpness(case)
    return lib.lmst_params(g, mode, DELTA0, s if s else 1.0, 30.0)


# ------------------------------------- Eq. 2-6 in 64 bits, with derivatives

def _stats(W, g=128):
    w = W.double().reshape(-1, g)
    mu0 = w.mean(1)
    a0 = (w - mu0[:, None]).abs().mean(1)
    return torch.stack([mu0, a0], 1).float()


def _scalars(stats, fac):
    """mu, alpha, Delta of every group, each rounded once to fp32."""
    mu0, a0 = stats[:, 0].double(), stats[:, 1].double()
    mu = (mu0 + fac[0].double() * a0).float().double()
    al = (fac[1].double() * a0).float().double()
    de = (fac[2].double() * DELTA0).float().double()
    return mu, al, de


def _lmst(W, stats, fac, hard, s, g=128):
    """alpha*T, T, f_W, f_Delta and W_hat, each [groups][g]; in the hard branch
    the derivatives are those of the transition at the last sharpness."""
    mu, al, de = (v[:, None] for v in _scalars(stats, fac))
    r = W.double().reshape(-1, g) - mu
    x = r / al.clamp_min(torch.finfo(torch.float32).tiny)
    sb = 30.0 if hard else s
    ta, tb = torch.tanh(sb * (x - de)), torch.tanh(sb * (x + de))
    k = 1.0 / (2.0 * math.tanh(sb))
    T = (ta + tb) * k
    da, db = 1.0 - ta * ta, 1.0 - tb * tb
    if hard:
        T = (r > de * al).double() - (r < -de * al).double()
    return al * T, T, sb * k * (da + db), sb * k * (db - da), x


def _factor_grads(G, W, stats, fac, hard, s, g=128):
    _, T, fw, fd, x = _lmst(W, stats, fac, hard, s, g)
    G = G.reshape(-1, g)
    a0 = stats[:, 1].double()
    gm = -a0 * (G * fw).sum(1)
    ga = a0 * ((G * T).sum(1) - (G * fw * x).sum(1))
    gd = DELTA0 * _scalars(stats, fac)[1] * (G * fd).sum(1)
    return gm, ga, gd


def _fake(W, stats, fac, hard, s):
    """The fake-ternary weight as the layers take it (bf16), in chunks of rows."""
    out = torch.empty_like(W)
    n = W.shape[-1] // 128
    for r0 in range(0, W.shape[0], 8192):
        r = slice(r0, r0 + 8192)
        q = slice(r0 * n, (r0 + 8192) * n)
        out[r] = _lmst(W[r], stats[q], [f[q] for f in fac], hard, s)[0].reshape(W[r].shape).to(W.dtype)
    return out


def _weight(g, rows, cols, std, case):
    """A frozen weight with its statistics, factors and fake-ternary weight."""
    W = _normal(g, (rows, cols), std)
    st = torch.cat([_stats(w) for w in W.split(8192)])
    fac = _factors(g, rows * cols // 128)
    mode, s = _sharpness(case)
    return SimpleNamespace(W=W, stats=st, fac=fac, Wf=_fake(W, st, fac, mode == lib.HARD, s),
                           g=[torch.empty_like(f) for f in fac])


def _grads64(G, w, case):
    """Factor gradients of a weight from dL/dW_fake, in 64 bits, in chunks of rows."""
    mode, s = _sharpness(case)
    n, out = w.W.shape[-1] // 128, []
    for r0 in range(0, w.W.shape[0], 8192):
        r, q = slice(r0, r0 + 8192), slice(r0 * n, (r0 + 8192) * n)
        out.append(_factor_grads(G[r], w.W[r], w.stats[q], [f[q] for f in w.fac], mode == lib.HARD, s))
    return tuple(torch.cat(t) for t in zip(*out))


def _swiglu64(gu):
    a, b = gu.chunk(2, -1)
    sg = torch.sigmoid(a)
    return a * sg * b


def _swiglu_bwd64(gu, da):
    a, b = gu.chunk(2, -1)
    sg = torch.sigmoid(a)
    return torch.cat([da * b * sg * (1 + a * (1 - sg)), da * a * sg], -1)


def _norm64(x):
    r = (x.square().mean(-1, keepdim=True) + EPS).rsqrt()
    return x * r, r


def _norm_bwd64(x, r, dy):
    return r * dy - x * r ** 3 * (dy * x).mean(-1, keepdim=True)


def _rope64(x, theta, back=False):
    S, d = x.shape[1], x.shape[-1]
    inv = theta ** (-2.0 * torch.arange(d // 2, device=x.device, dtype=torch.float64) / d)
    ang = torch.arange(S, device=x.device, dtype=torch.float64)[:, None] * inv
    c, s = ang.cos()[None, :, None], ang.sin()[None, :, None]
    s = -s if back else s
    a, b = x.chunk(2, -1)
    return torch.cat([a * c - b * s, b * c + a * s], -1)


class _Attn64:
    """Causal grouped-query attention on q|k|v rows; ``back`` gives dq|dk|dv."""

    def __init__(self, qkv, c, theta=1e6):
        B, S, H, Hk, d = c["batch"], c["seq"], c["n_q"], c["n_kv"], c["d"]
        self.c, self.theta, self.dims = c, theta, (B, S, H, Hk, d)
        x = qkv.reshape(B, S, H + 2 * Hk, d)
        self.qk = x[:, :, :H + Hk]
        if c["qk_norm"]:
            n, self.r = _norm64(self.qk)
        else:
            n, self.r = self.qk, None
        n = _rope64(n, theta)
        self.q, self.k, self.v = n[:, :, :H], n[:, :, H:], x[:, :, H + Hk:]
        self.o = torch.empty_like(self.q)
        for b in range(B):
            for h in range(H):
                self.o[b, :, h] = self._p(b, h) @ self.v[b, :, h * Hk // H]
        self.out = self.o.reshape(B * S, H * d)

    def _p(self, b, h):
        S, H, Hk, d = self.dims[1:]
        s = self.q[b, :, h] @ self.k[b, :, h * Hk // H].T / math.sqrt(d)
        s.masked_fill_(torch.ones(S, S, dtype=torch.bool, device=s.device).triu(1), -math.inf)
        return s.softmax(-1)

    def back(self, do):
        B, S, H, Hk, d = self.dims
        do = do.reshape(B, S, H, d)
        dq, dk, dv = (torch.zeros_like(t) for t in (self.q, self.k, self.v))
        for b in range(B):
            for h in range(H):
                j, p = h * Hk // H, self._p(b, h)
                dv[b, :, j] += p.T @ do[b, :, h]
                dp = do[b, :, h] @ self.v[b, :, j].T
                ds = p * (dp - (do[b, :, h] * self.o[b, :, h]).sum(-1, keepdim=True)) / math.sqrt(d)
                dq[b, :, h] = ds @ self.k[b, :, j]
                dk[b, :, j] += ds.T @ self.q[b, :, h]
        dqk = _rope64(torch.cat([dq, dk], 2), self.theta, back=True)
        if self.r is not None:
            dqk = _norm_bwd64(self.qk, self.r, dqk)
        return torch.cat([dqk, dv], 2).reshape(B * S, (H + 2 * Hk) * d)


# ---------------------------------------------------------------- f32 kind

def _f32_prepare(case, seed):
    g = _gen(seed)
    M, N, K = case["M"], case["N"], case["K"]
    W = _normal(g, (N, K), 0.02, torch.float32)
    X = _normal(g, (M, K), 1.0, torch.float32)
    X[:, torch.randperm(K, generator=g, device=DEV)[:4]] *= 20.0   # outlier channels
    f32 = dict(dtype=torch.float32, device=DEV)
    fac = _factors(g, N * K // 128)
    return SimpleNamespace(
        case=case, W=W, X=X, fac=fac, Y_fp=(X.double() @ W.double().T).float(), p=_params(case),
        stats=torch.empty((N * K // 128, 2), **f32), Wf=torch.empty_like(W),
        Y=torch.empty((M, N), **f32), dY=torch.empty((M, N), **f32), dX=torch.empty((M, K), **f32),
        loss=torch.empty(1, **f32), g=[torch.empty_like(f) for f in fac],
        loss_ws=torch.empty(lib.catq_workspace_size(lib.WS_LOSS, M * N, 1, 1), dtype=torch.uint8, device=DEV),
        ws=torch.empty(lib.catq_workspace_size(lib.WS_LINEAR_BWD, M, N, K), dtype=torch.uint8, device=DEV))


def _f32_run(s):
    M, N, K = s.case["M"], s.case["N"], s.case["K"]
    lib.catq_modulate_ternarize(s.W, *s.fac, s.p, s.stats, 0, W_fake=s.Wf)
    lib.catq_fakeq_linear_fwd(s.X, s.Wf, s.Y, M, N, K)
    lib.catq_block_recon_loss(s.Y, s.Y_fp, s.loss, s.dY, s.loss_ws)
    lib.catq_fakeq_linear_bwd(s.dY, s.X, s.Wf, M, N, K, s.W, s.stats, *s.fac, s.p, *s.g, s.ws, dX=s.dX)
    return dict(Wf=s.Wf, Y=s.Y, loss=s.loss, dX=s.dX, g=s.g)


def _f32_exact(case, seed):
    s = _f32_prepare(case, seed)
    st = _stats(s.W)
    Wf = _lmst(s.W, st, s.fac, False, 15.0)[0].reshape(s.W.shape)
    X = s.X.double()
    Y = X @ Wf.T
    d = Y - s.Y_fp.double()
    dY = d * (2.0 / d.numel())
    return dict(Wf=Wf, Y=Y, loss=d.square().mean().reshape(1), dX=dY @ Wf,
                g=list(_factor_grads(dY.T @ X, s.W, st, s.fac, False, 15.0)))


# --------------------------------------------------------------- step kind

def _block64(x, W, c, keep=False):
    """Pre-norm decoder block forward in 64 bits; ``keep``: what a backward needs."""
    h, hq = c["hidden"], c["n_q"] * c["d"]
    k = SimpleNamespace()
    xn1, k.r1 = _norm64(x)
    qkv = xn1 @ torch.cat([W["Wq"], W["Wk"], W["Wv"]]).T
    att = _Attn64(qkv, c)
    h1 = x + att.out @ W["Wo"].T
    xn2, k.r2 = _norm64(h1)
    gu = xn2 @ torch.cat([W["Wg"], W["Wu"]]).T
    a = _swiglu64(gu)
    y = h1 + a @ W["Wd"].T
    if keep:
        k.x, k.xn1, k.att, k.h1, k.xn2, k.gu, k.a = x, xn1, att, h1, xn2, gu, a
        return y, k
    return y


def _step_inputs(case, seed):
    g = _gen(seed)
    c = case
    h, hq, hk, F = c["hidden"], c["n_q"] * c["d"], c["n_kv"] * c["d"], c["ffn"]
    shapes = dict(Wq=(hq, h), Wk=(hk, h), Wv=(hk, h), Wo=(h, hq), Wg=(F, h), Wu=(F, h), Wd=(h, F))
    W = {k: _normal(g, s, 0.02) for k, s in shapes.items()}
    fac = _factors(g, sum(w.numel() for w in W.values()) // 128)
    x = _acts(g, (c["batch"] * c["seq"], h))
    y_fp = _block64(x.double(), {k: w.double() for k, w in W.items()}, c).float()
    return W, fac, x, y_fp


def _step_prepare(case, seed):
    W, fac, x, y_fp = _step_inputs(case, seed)
    cfg = SimpleNamespace(hidden=case["hidden"], n_q=case["n_q"], n_kv=case["n_kv"],
                          head_dim=case["d"], ffn=case["ffn"], qk_norm=case["qk_norm"],
                          rope_theta=1e6, batch=case["batch"], seq=case["seq"])
    bits = {k: w.view(torch.int16).cpu().numpy().view(np.uint16) for k, w in W.items()}
    blk = DenseBlock(cfg, bits, a8=case["a8"])
    A = blk.arena
    for t, f in zip((A.d_mu, A.d_alpha, A.d_delta), fac):
        t.copy_(f)
    blk.modulate_all(blk.params(lib.IDENTITY))   # as for the cached target: statistics ready
    return SimpleNamespace(case=case, blk=blk, x=x, y_fp=y_fp)


def _step_run(s):
    mode, sh = _sharpness(s.case)
    blk, A = s.blk, s.blk.arena
    loss = blk.step(s.x, s.y_fp, mode=mode, s=sh, s_bwd=30.0, input_grad=s.case["input_grad"])
    out = dict(loss=loss, y=blk.y, g=[A.g_mu, A.g_alpha, A.g_delta])
    if s.case["input_grad"]:
        out["dx"] = blk.dx
    return out


def _step_exact(case, seed):
    if case["a8"]:
        return None   # 8-bit codes near a half fall either way: no value to hold it to
    W, fac, x, y_fp = _step_inputs(case, seed)
    c = case
    mode, sh = _sharpness(case)
    hard = mode == lib.HARD
    ws, o = {}, 0
    for k, w in W.items():
        n = w.numel() // 128
        ws[k] = SimpleNamespace(W=w, stats=torch.cat([_stats(v) for v in w.split(8192)]),
                                fac=[f[o:o + n] for f in fac])
        ws[k].Wf = _fake(w, ws[k].stats, ws[k].fac, hard, sh).double()
        o += n
    T = {k: v.Wf for k, v in ws.items()}
    y, k = _block64(x.double(), T, c, keep=True)
    d = y - y_fp.double()
    dy = d * (2.0 / d.numel())
    G = {"Wd": dy.T @ k.a}
    dgu = _swiglu_bwd64(k.gu, dy @ T["Wd"])
    G["Wg"], G["Wu"] = (dgu.T @ k.xn2).split(c["ffn"])
    dh1 = dy + _norm_bwd64(k.h1, k.r2, dgu @ torch.cat([T["Wg"], T["Wu"]]))
    del dgu, k.gu, k.a
    G["Wo"] = dh1.T @ k.att.out
    dqkv = k.att.back(dh1 @ T["Wo"])
    hq, hk = c["n_q"] * c["d"], c["n_kv"] * c["d"]
    G["Wq"], G["Wk"], G["Wv"] = (dqkv.T @ k.xn1).split([hq, hk, hk])
    gs = [torch.cat(t) for t in zip(*(_grads64(G[n], ws[n], case) for n in W))]
    out = dict(loss=d.square().mean().reshape(1), y=y, g=gs)
    if c["input_grad"]:
        dxn = dqkv @ torch.cat([T["Wq"], T["Wk"], T["Wv"]])
        out["dx"] = dh1 + _norm_bwd64(k.x, k.r1, dxn)
    return out


# ------------------------------------------------------------- linear kind

def _linear_prepare(case, seed):
    g = _gen(seed)
    M, N, K = case["M"], case["N"], case["K"]
    w = _weight(g, N, K, 0.02, case)
    yt = torch.float32 if case["res"] else torch.bfloat16
    return SimpleNamespace(
        case=case, w=w, p=_params(case), X=_acts(g, (M, K)), dY=_normal(g, (M, N), 1e-3),
        res=_normal(g, (M, N), 1.0, yt) if case["res"] else None,
        Y=torch.empty((M, N), dtype=yt, device=DEV),
        dX=torch.empty((M, K), dtype=torch.bfloat16, device=DEV),
        ws=torch.empty(lib.catq_workspace_size(lib.WS_LINEAR_BWD, M, N, K), dtype=torch.uint8, device=DEV))


def _linear_run(s):
    M, N, K = s.case["M"], s.case["N"], s.case["K"]
    w = s.w
    lib.catq_fakeq_linear_fwd(s.X, w.Wf, s.Y, M, N, K, residual=s.res)
    lib.catq_fakeq_linear_bwd(s.dY, s.X, w.Wf, M, N, K, w.W, w.stats, *w.fac, s.p, *w.g, s.ws, dX=s.dX)
    return dict(Y=s.Y, dX=s.dX, g=w.g)


def _linear_exact(case, seed):
    s = _linear_prepare(case, seed)
    X, dY, Wf = s.X.double(), s.dY.double(), s.w.Wf.double()
    Y = X @ Wf.T
    if s.res is not None:
        Y += s.res.double()
    return dict(Y=Y, dX=dY @ Wf, g=list(_grads64(dY.T @ X, s.w, case)))


# ---------------------------------------------------------------- mlp kind

def _mlp_prepare(case, seed):
    g = _gen(seed)
    M, h, F = case["M"], case["h"], case["F"]
    gu, d = _weight(g, 2 * F, h, 0.02, case), _weight(g, h, F, 0.02, case)
    e = lambda *s, t=torch.bfloat16: torch.empty(s, dtype=t, device=DEV)  # noqa: E731
    ws = max(lib.catq_workspace_size(lib.WS_LINEAR_BWD, M, 2 * F, h),
             lib.catq_workspace_size(lib.WS_LINEAR_BWD, M, h, F))
    return SimpleNamespace(
        case=case, wg=gu, wd=d, p=_params(case), h1=_acts(g, (M, h)).float(), dy=_normal(g, (M, h), 1e-3),
        xn=e(M, h), rstd=e(M, t=torch.float32), gu=e(M, 2 * F), a=e(M, F), y=e(M, h, t=torch.float32),
        da=e(M, F), dgu=e(M, 2 * F), dxn=e(M, h), dh=e(M, h), ws=e(ws, t=torch.uint8))


def _mlp_run(s):
    M, h, F = s.case["M"], s.case["h"], s.case["F"]
    wg, wd = s.wg, s.wd
    lib.catq_aux_rmsnorm_fwd(s.h1, s.xn, s.rstd)
    lib.catq_fakeq_gateup_swiglu_fwd(s.xn, wg.Wf, s.gu, s.a, M, F, h)
    lib.catq_fakeq_linear_fwd(s.a, wd.Wf, s.y, M, h, F, residual=s.h1)
    lib.catq_fakeq_linear_bwd(s.dy, s.a, wd.Wf, M, h, F, wd.W, wd.stats, *wd.fac, s.p, *wd.g, s.ws)
    lib.catq_fakeq_down_swiglu_bwd(s.dy, wd.Wf, s.gu, s.dgu, M, h, F, da=s.da)
    lib.catq_fakeq_linear_bwd(s.dgu, s.xn, wg.Wf, M, 2 * F, h, wg.W, wg.stats, *wg.fac, s.p, *wg.g,
                              s.ws, dX=s.dxn)
    lib.catq_aux_rmsnorm_bwd(s.h1, s.rstd, s.dxn, s.dh, dres=s.dy)
    return dict(y=s.y, dh=s.dh, gg=wg.g, gd=wd.g)


def _mlp_exact(case, seed):
    s = _mlp_prepare(case, seed)
    Wg, Wd, x, dy = s.wg.Wf.double(), s.wd.Wf.double(), s.h1.double(), s.dy.double()
    xn, r = _norm64(x)
    gu = xn @ Wg.T
    a = _swiglu64(gu)
    dgu = _swiglu_bwd64(gu, dy @ Wd)
    return dict(y=x + a @ Wd.T, dh=dy + _norm_bwd64(x, r, dgu @ Wg),
                gg=list(_grads64(dgu.T @ xn, s.wg, case)), gd=list(_grads64(dy.T @ a, s.wd, case)))


# --------------------------------------------------------------- attn kind

def _attn_prepare(case, seed):
    g = _gen(seed)
    c = case
    M, Nq = c["batch"] * c["seq"], c["n_q"] * c["d"]
    N = Nq + 2 * c["n_kv"] * c["d"]
    desc = lib.attn_desc(c["batch"], c["seq"], c["n_q"], c["n_kv"], c["d"], c["qk_norm"], 1e6,
                         act_quant=c["a8"])
    e = lambda *s, t=torch.bfloat16: torch.empty(s, dtype=t, device=DEV)  # noqa: E731
    return SimpleNamespace(
        case=case, desc=desc, qkv=_normal(g, (M, N)), do=_normal(g, (M, Nq), 1e-3), o=e(M, Nq), dqkv=e(M, N),
        saved=e(lib.catq_attn_saved_bytes(desc), t=torch.uint8),
        ws=e(lib.catq_attn_bwd_workspace_bytes(desc), t=torch.uint8))


def _attn_run(s):
    lib.catq_aux_attention_fwd(s.desc, s.qkv, s.o, s.saved)
    lib.catq_aux_attention_bwd(s.desc, s.qkv, s.o, s.saved, s.do, s.dqkv, s.ws)
    return dict(o=s.o, dqkv=s.dqkv)


def _attn_exact(case, seed):
    if case["a8"]:
        return None   # as for the steps: 8-bit codes near a half
    s = _attn_prepare(case, seed)
    at = _Attn64(s.qkv.double(), case)
    return dict(o=at.out, dqkv=at.back(s.do.double()))


# ---------------------------------------------------------------- moe kind

def _moe_prepare(case, seed):
    g = _gen(seed)
    T, h, F, E, k = (case[n] for n in ("T", "h", "F", "E", "k"))
    R = T * k
    wg, wd = _weight(g, E * 2 * F, h, 0.02, case), _weight(g, E * h, F, 0.02, case)
    e = lambda *s, t=torch.bfloat16: torch.empty(s, dtype=t, device=DEV)  # noqa: E731
    ws = max(lib.catq_workspace_size(lib.WS_LINEAR_BWD, R, 2 * F, h, E),
             lib.catq_workspace_size(lib.WS_LINEAR_BWD, R, h, F, E))
    i32, f32 = torch.int32, torch.float32
    return SimpleNamespace(
        case=case, wg=wg, wd=wd, p=_params(case), x=_normal(g, (T, h)), dy=_normal(g, (T, h), 1e-3),
        res=_acts(g, (T, h)).float(), logits=torch.randn((T, E), generator=g, device=DEV),
        ids=e(T, k, t=i32), wts=e(T, k, t=f32), perm=e(T, k, t=i32), offs=e(E + 1, t=torch.int64),
        route_ws=e(lib.catq_aux_moe_route_workspace_bytes(T, E, k), t=torch.uint8),
        xg=e(R, h), gu=e(R, 2 * F), a=e(R, F), yg=e(R, h), y=e(T, h, t=f32), dyg=e(R, h),
        da=e(R, F), dgu=e(R, 2 * F), dxg=e(R, h), dx=e(T, h), ws=e(ws, t=torch.uint8))


def _moe_run(s):
    T, h, F, E, k = (s.case[n] for n in ("T", "h", "F", "E", "k"))
    R, wg, wd = T * k, s.wg, s.wd
    ex = dict(n_experts=E, row_offsets=s.offs)
    lib.catq_aux_moe_route(s.logits, k, s.ids, s.wts, s.perm, s.offs, s.route_ws)
    lib.catq_aux_moe_gather(s.x, s.perm, k, s.xg)
    lib.catq_fakeq_linear_fwd(s.xg, wg.Wf, s.gu, R, 2 * F, h, **ex)
    lib.catq_aux_swiglu_fwd(s.gu, s.a)
    lib.catq_fakeq_linear_fwd(s.a, wd.Wf, s.yg, R, h, F, **ex)
    lib.catq_aux_moe_combine(s.yg, s.perm, s.wts, s.res, s.y, k)
    lib.catq_aux_moe_combine_bwd(s.dy, s.perm, s.wts, s.dyg, k)
    lib.catq_fakeq_linear_bwd(s.dyg, s.a, wd.Wf, R, h, F, wd.W, wd.stats, *wd.fac, s.p, *wd.g, s.ws,
                              dX=s.da, **ex)
    lib.catq_aux_swiglu_bwd(s.gu, s.da, s.dgu)
    lib.catq_fakeq_linear_bwd(s.dgu, s.xg, wg.Wf, R, 2 * F, h, wg.W, wg.stats, *wg.fac, s.p, *wg.g,
                              s.ws, dX=s.dxg, **ex)
    lib.catq_aux_moe_scatter_add(s.dxg, s.perm, s.dx, k)
    return dict(ids=s.ids, wts=s.wts, perm=s.perm, offs=s.offs, y=s.y, dx=s.dx, gg=wg.g, gd=wd.g)


def _moe_exact(case, seed):
    s = _moe_prepare(case, seed)
    T, h, F, E, k = (case[n] for n in ("T", "h", "F", "E", "k"))
    top, ids = s.logits.double().topk(k, 1)
    wts = top.softmax(1)
    x, dy, y, dx = s.x.double(), s.dy.double(), s.res.double().clone(), torch.zeros((T, h), dtype=torch.float64, device=DEV)
    Gg = torch.zeros((E * 2 * F, h), dtype=torch.float64, device=DEV)
    Gd = torch.zeros((E * h, F), dtype=torch.float64, device=DEV)
    for e in range(E):
        t, j = (ids == e).nonzero(as_tuple=True)
        if not t.numel():
            continue
        rg, rd = slice(e * 2 * F, (e + 1) * 2 * F), slice(e * h, (e + 1) * h)
        Wg, Wd, w = s.wg.Wf[rg].double(), s.wd.Wf[rd].double(), wts[t, j][:, None]
        gu = x[t] @ Wg.T
        a = _swiglu64(gu)
        y.index_add_(0, t, w * (a @ Wd.T))
        dye = w * dy[t]
        dgu = _swiglu_bwd64(gu, dye @ Wd)
        Gd[rd], Gg[rg] = dye.T @ a, dgu.T @ x[t]
        dx.index_add_(0, t, dgu @ Wg)
    return dict(ids=None, wts=wts, perm=None, offs=None, y=y, dx=dx,
                gg=list(_grads64(Gg, s.wg, case)), gd=list(_grads64(Gd, s.wd, case)))


# ------------------------------------------------------------ weights kind

def _weights_prepare(case, seed):
    g = _gen(seed)
    rows, cols, gs = case["rows"], case["cols"], case["g"]
    n = rows * cols // gs
    W = _normal(g, (rows, cols), 0.02)
    f32 = dict(dtype=torch.float32, device=DEV)
    return SimpleNamespace(
        case=case, W=W, fac=_factors(g, n), soft=lib.lmst_params(gs, lib.SOFT, DELTA0, 15.0, 30.0),
        hard=lib.lmst_params(gs, lib.HARD, DELTA0, 1.0, 30.0), stats=torch.empty((n, 2), **f32),
        Wf=torch.empty_like(W), alpha=torch.empty(n, **f32),
        packed=torch.empty((rows, cols // 4), dtype=torch.uint8, device=DEV))


def _weights_run(s):
    lib.catq_modulate_ternarize(s.W, *s.fac, s.soft, s.stats, 0, W_fake=s.Wf)
    lib.catq_ternarize_pack(s.W, *s.fac, s.hard, s.stats, 1, s.packed, alpha_out=s.alpha)
    return dict(stats=s.stats, Wf=s.Wf, packed=s.packed, alpha=s.alpha)


def _weights_exact(case, seed):
    s = _weights_prepare(case, seed)
    g = case["g"]
    st = _stats(s.W, g)
    w = s.W.double().reshape(-1, g)
    mu0 = w.mean(1)
    return dict(stats=torch.stack([mu0, (w - mu0[:, None]).abs().mean(1)], 1),
                Wf=_lmst(s.W, st, s.fac, False, 15.0, g)[0].reshape(s.W.shape), packed=None,
                alpha=s.fac[1].double() * st[:, 1].double())


# ------------------------------------------------------------ ternary kind

def _layers(c):
    """(d_out, d_in) of q|k|v, o, gate|up and down; the o input is as wide as the model."""
    h = c["hidden"]
    return [(c["qkv"], h), (h, h), (2 * c["ffn"], h), (h, c["ffn"])]


def _ternary_prepare(case, seed):
    g = _gen(seed)
    M, out = case["M"], []
    yt = torch.float32 if case["out_f32"] else torch.bfloat16
    xs = {k: _acts(g, (M, k)) for k in sorted({case["hidden"], case["ffn"]})}
    for n, k in _layers(case):
        # half the codes zero, as ternarised Gaussian weights have
        c = (torch.randint(0, 4, (n, k // 4, 4), generator=g, device=DEV, dtype=torch.int16) + 1) // 2
        packed = (c[..., 0] | c[..., 1] << 2 | c[..., 2] << 4 | c[..., 3] << 6).to(torch.uint8)
        alpha = (torch.rand((n, k // 128), generator=g, device=DEV) * 0.6 - 0.3).exp() * 0.016
        out.append(SimpleNamespace(X=xs[k], packed=packed, alpha=alpha,
                                   Y=torch.empty((M, n), dtype=yt, device=DEV)))
        del c
    return SimpleNamespace(case=case, layers=out)


def _ternary_run(s):
    for t in s.layers:
        lib.catq_ternary_linear(t.X, t.packed, t.alpha, t.Y)
    return [t.Y for t in s.layers]


def _ternary_exact(case, seed):
    out = []
    for t in _ternary_prepare(case, seed).layers:
        X, ys = t.X.double(), []
        for p, a in zip(t.packed.split(4096), t.alpha.split(4096)):
            c = torch.stack([(p >> 2 * j) & 3 for j in range(4)], -1).to(torch.float64) - 1.0
            W = c.reshape(p.shape[0], -1, 128) * a.double()[..., None]
            ys.append(X @ W.reshape(p.shape[0], -1).T)
        out.append(torch.cat(ys, 1))
    return out


# ------------------------------------------------------------- entry points

_PREPARE = dict(f32=_f32_prepare, step=_step_prepare, linear=_linear_prepare, mlp=_mlp_prepare,
                attn=_attn_prepare, moe=_moe_prepare, weights=_weights_prepare,
                ternary=_ternary_prepare)
_RUN = dict(f32=_f32_run, step=_step_run, linear=_linear_run, mlp=_mlp_run, attn=_attn_run,
            moe=_moe_run, weights=_weights_run, ternary=_ternary_run)
_EXACT = dict(f32=_f32_exact, step=_step_exact, linear=_linear_exact, mlp=_mlp_exact,
              attn=_attn_exact, moe=_moe_exact, weights=_weights_exact, ternary=_ternary_exact)


def prepare(case, seed):
    return _PREPARE[case["kind"]](case, seed)


def run(state):
    return _RUN[state.case["kind"]](state)


def exact(case, seed):
    return _EXACT[case["kind"]](case, seed)


def _attn_work(c):
    """Causal attention, forward (two products) and backward (five)."""
    pairs = c["batch"] * c["n_q"] * c["seq"] * (c["seq"] + 1) / 2
    rows = c["batch"] * c["seq"] * c["d"] * 2
    return dict(flops=14.0 * pairs * c["d"], bytes=float(rows * (4 * c["n_q"] + 4 * c["n_kv"])))


def work(case):
    c, kind = case, case["kind"]
    if kind == "f32":
        M, N, K = c["M"], c["N"], c["K"]
        return dict(flops=6.0 * M * N * K, bytes=4.0 * (2 * N * K + 2 * M * N + 2 * M * K))
    if kind == "step":
        M, h = c["batch"] * c["seq"], c["hidden"]
        qkv = (c["n_q"] + 2 * c["n_kv"]) * c["d"] * h
        P = qkv + c["n_q"] * c["d"] * h + 3 * h * c["ffn"]
        flops = 6.0 * M * P - (0 if c["input_grad"] else 2.0 * M * qkv)
        return dict(flops=flops + _attn_work(c)["flops"],
                    bytes=2.0 * P + P / 128 * 32.0 + M * h * (10.0 + 2 * c["input_grad"]))
    if kind == "linear":
        M, N, K = c["M"], c["N"], c["K"]
        return dict(flops=6.0 * M * N * K,
                    bytes=4.0 * N * K + N * K / 128 * 32.0 + 4.0 * M * K + (10.0 if c["res"] else 4.0) * M * N)
    if kind == "mlp":
        M, h, F = c["M"], c["h"], c["F"]
        return dict(flops=18.0 * M * h * F, bytes=12.0 * h * F + 3 * h * F / 128 * 32.0 + 12.0 * M * h)
    if kind == "attn":
        return _attn_work(c)
    if kind == "moe":
        T, h, F, E, k = (c[n] for n in ("T", "h", "F", "E", "k"))
        P = 3.0 * E * h * F
        return dict(flops=18.0 * T * k * h * F, bytes=4.0 * P + P / 128 * 32.0 + 14.0 * T * h + 4.0 * T * E)
    if kind == "weights":
        P = c["rows"] * c["cols"]
        return dict(flops=0.0, bytes=4.25 * P + P / c["g"] * 24.0)
    out = 4 if c["out_f32"] else 2
    P = float(sum(n * k for n, k in _layers(c)))
    rows = float(sum(n for n, _ in _layers(c)))
    return dict(flops=2.0 * c["M"] * P,
                bytes=P / 4 + P / 32 + c["M"] * (2.0 * (c["hidden"] + c["ffn"]) + out * rows))


def tolerance(case):
    """About four times what was measured against ``exact``
    (relative 2-norm; largest difference), which is what the data types give:
    fp32 sums 1e-6; one bf16 rounding 1.7e-3; chains of bf16 activations
    3e-3 to 5e-3.  Whole numbers (codes, routing) are the same."""
    kind = case["kind"]
    if kind == "f32" or case.get("out_f32"):
        return dict(rel=4e-6, max=4e-5)
    if kind in ("linear", "weights", "ternary"):
        return dict(rel=7e-3, max=1.6e-2)
    if case.get("a8"):
        return dict(rel=3e-2, max=0.4)   # an 8-bit code near a half moves by a whole step
    if kind == "step":
        return dict(rel=1.9e-2, max=0.2)
    return dict(rel=1.6e-2, max=0.3 if kind == "attn" else 0.2)
