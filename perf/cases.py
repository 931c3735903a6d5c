"""The work this framework is measured on: the layers of a GPT training step
through the kernel entry points (atom_kernels.h), and whole steps through
Session.

A layer case is one training pass of that layer, forward and backward, with
the calls, layouts and types of the training step: bf16 operands, fp32
residual stream, statistics and parameter-gradient sums.  Widths and token
counts are those of the GPT-3 configurations (Small 768 / 12 heads of 64,
batch 8 x 2048 tokens; XL 2048 / 16 heads of 128, 4 x 2048; 6.7B 4096 / 32
heads, 2 x 2048; 13B 5120 / 40 heads, 1 x 2048) and, for the short ones, one
small batch of sequences that are no multiple of a tile, as in fine-tuning.

Operations (field "op"):
  attn   causal attention, forward and backward (atom_k_attn_fwd, atom_k_attn_bwd)
  proj   a block's attention projections: qkv = a W^T + b and
         x1 = x + o W_o^T + b_o, then both layers' data, weight and bias gradients
  mlp    a block's MLP: GELU(c W_fc^T + b_fc), then the residual projection,
         and the data, weight and bias gradients of both
  norm   LayerNorm forward, and backward into the residual gradient
  head   LM head: fp32 logits in chunks of 2048 tokens, softmax cross-entropy
         with its gradient, data and weight gradient of the head
  step   training steps through Session: whole model, gradients on the host
"""
from __future__ import annotations

import math

import numpy as np
import torch

import synthetic
from paper_2403_10504_amd import Session
from paper_2403_10504_amd import atom as A

BF16 = torch.bfloat16
HEAD_CHUNK = 2048        # tokens per chunk of fp32 logits, as in the step
WS_BYTES = 64 << 20      # split-k workspace, the size the step keeps


def listed():
    return [
        # attention of one 6.7B block: the step's own batch, long heads
        dict(name="attn_6.7b", op="attn", B=2, T=2048, H=32, dh=128),
        # attention of one GPT-3 Small block: many sequences, narrow heads
        dict(name="attn_small", op="attn", B=8, T=2048, H=12, dh=64),
        # attention at XL width over a few short ragged sequences (fine-tuning)
        dict(name="attn_short", op="attn", B=3, T=333, H=16, dh=128),
        # MLP of one 13B block: one sequence, the widest layer
        dict(name="mlp_13b", op="mlp", N=2048, d=5120, f=20480),
        # MLP of one GPT-3 Small block: many tokens, narrow layer
        dict(name="mlp_small", op="mlp", N=16384, d=768, f=3072),
        # MLP of one XL block on a single ragged sequence of 1000 tokens
        dict(name="mlp_short", op="mlp", N=1000, d=2048, f=8192),
        # attention projections of one 6.7B block at its own batch
        dict(name="proj_6.7b", op="proj", N=4096, d=4096),
        # attention projections of one GPT-3 Small block on one short sequence
        dict(name="proj_short", op="proj", N=520, d=768),
        # LayerNorm of one 13B block
        dict(name="norm_13b", op="norm", N=2048, d=5120),
        # LM head of GPT-3 Small at its own batch: the vocabulary dominates
        dict(name="head_small", op="head", N=16384, d=768, V=50257),
        # one step of the tiny fp32 decoder, every group swapped through two
        # slots: the smallest call, host and launches dominate
        dict(name="step_tiny", op="step", L=2, d=256, H=4, f=1024, V=1024, T=128, B=2, C=1, dtype="f32", steps=1,
             swap=True, rows=False),
        # two pipelined steps at GPT-3 Small's width, resident (two blocks, full vocabulary)
        dict(name="step_small", op="step", L=2, d=768, H=12, f=3072, V=50257, T=2048, B=8, C=1, dtype="bf16", steps=2,
             swap=False, rows=False),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["attn", "attn", "attn", "mlp", "mlp", "mlp", "proj", "proj", "norm", "head", "step"])
    if op == "attn":
        dh = rng.choice([64, 128])
        H = _log(rng, 4, 40)
        T = _log(rng, 64, 2048)
        most = max(1, int(2 * 32 * 128 * 2048 * 2048 // (H * dh * T * T)))
        return dict(op=op, B=_log(rng, 1, min(32, most)), T=T, H=H, dh=dh)
    if op == "norm":
        return dict(op=op, N=_log(rng, 64, 16384), d=64 * _log(rng, 4, 80))
    if op == "step":
        d = 64 * rng.randint(2, 8)
        return dict(op=op, L=rng.randint(1, 2), d=d, H=d // 64, f=8 * rng.randint(d // 4, d // 2),
                    V=_log(rng, 500, 8000), T=8 * _log(rng, 8, 48), B=rng.randint(1, 4), C=rng.randint(1, 2),
                    dtype=rng.choice(["bf16", "bf16", "f32"]), steps=rng.randint(1, 2), swap=rng.random() < 0.5,
                    rows=rng.random() < 0.3)
    # token counts are multiples of 8, as the weight gradients' contraction needs
    if op == "head":
        V = _log(rng, 1000, 50257)
        d = 64 * _log(rng, 4, 32)
        most = 2048 * 5120 * 20480 // (V * d)
        return dict(op=op, N=8 * _log(rng, 8, max(8, min(16384, most) // 8)), d=d, V=V)
    d = 64 * _log(rng, 4, 80)
    if op == "proj":
        return dict(op=op, N=8 * _log(rng, 8, min(16384, 2048 * 5120 * 20480 // (2 * d * d)) // 8), d=d)
    return dict(op=op, N=8 * _log(rng, 8, min(16384, 2048 * 5120 * 20480 // (4 * d * d)) // 8), d=d, f=4 * d)


# ------------------------------------------------------------------ inputs
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _randn(g, shape, std=1.0, dtype=BF16):
    return (torch.randn(shape, device="cuda", generator=g) * std).to(dtype)


def _empty(shape, dtype=BF16):
    return torch.empty(shape, device="cuda", dtype=dtype)


def _inputs(case, seed):
    """The tensors a layer reads, from the seed alone."""
    g, op = _gen(seed), case["op"]
    if op == "attn":
        n, d = case["B"] * case["T"], case["H"] * case["dh"]
        return dict(qkv=_randn(g, (n, 3 * d)), do=_randn(g, (n, d), 1e-2))
    N, d = case["N"], case["d"]
    if op == "norm":
        return dict(x=_randn(g, (N, d), 2.0, torch.float32) + 0.3, gamma=1 + _randn(g, (d,), 0.1),
                    beta=_randn(g, (d,), 0.1), dy=_randn(g, (N, d), 1e-2),
                    dres=_randn(g, (N, d), 1e-2, torch.float32))
    if op == "proj":
        return dict(a=_randn(g, (N, d)), w_qkv=_randn(g, (3 * d, d), 0.02), b_qkv=_randn(g, (3 * d,), 0.02),
                    o=_randn(g, (N, d), 0.5), w_o=_randn(g, (d, d), 0.02), b_o=_randn(g, (d,), 0.02),
                    x=_randn(g, (N, d), 1.0, torch.float32), dx=_randn(g, (N, d), 1e-2, torch.float32),
                    dqkv=_randn(g, (N, 3 * d), 1e-2))
    if op == "mlp":
        f = case["f"]
        return dict(c=_randn(g, (N, d)), w_fc=_randn(g, (f, d), 0.02), b_fc=_randn(g, (f,), 0.02),
                    w_pr=_randn(g, (d, f), 0.02), b_pr=_randn(g, (d,), 0.02),
                    x1=_randn(g, (N, d), 1.0, torch.float32), dx=_randn(g, (N, d), 1e-2, torch.float32))
    V = case["V"]
    Vp = (V + 127) // 128 * 128
    w = _randn(g, (Vp, d), 0.02)
    w[V:] = 0
    return dict(y=_randn(g, (N, d)), w=w,
                tgt=torch.randint(0, V, (N,), device="cuda", generator=g, dtype=torch.int32))


def _step_config(case):
    return synthetic.Config("measured", case["L"], case["d"], case["H"], case["f"], case["V"], case["T"], case["B"],
                            case["C"], case["dtype"], 0)


def _step_inputs(case, seed):
    """Weights (working-dtype values, on the GPU, list over nodes of {name: tensor}) and host tokens."""
    cfg, g = _step_config(case), _gen(seed)
    dt = BF16 if case["dtype"] == "bf16" else torch.float32
    weights = []
    for node in range(cfg.n_nodes):
        p = {}
        for name, shape, init in synthetic.param_specs(cfg, node):
            if init == "normal":
                p[name] = _randn(g, shape, synthetic.INIT_STD, dt)
            else:
                p[name] = torch.full(shape, 1.0 if init == "one" else 0.0, device="cuda", dtype=dt)
        weights.append(p)
    tok = np.random.default_rng(seed).integers(0, cfg.vocab, (case["steps"], cfg.accum, cfg.batch, cfg.seq_len + 1),
                                               dtype=np.int32)
    return cfg, weights, tok


def _host(view, dtype):
    """A host tensor over one of the library's host buffers (bf16 ones come as 16-bit patterns)."""
    t = torch.from_numpy(view.view(np.int16) if dtype == "bf16" else view)
    return t.view(BF16) if dtype == "bf16" else t


def _prepare_step(case, seed):
    cfg, weights, tok = _step_inputs(case, seed)
    plan = None
    if case["swap"]:
        n = cfg.n_nodes
        plan = A.atom_plan_fixed(A.make_config(cfg), list(range(n)), 2)
    s = Session(cfg, plan=plan)
    for node, p in enumerate(weights):
        for name, w in p.items():
            _host(s.host_view(node, name), case["dtype"])[: w.shape[0]].copy_(w)
    if case["rows"]:
        s.set_embedding_rows(True)
    elif not case["swap"]:
        s.set_retention(True)  # a resident model keeps its weights across the steps of a call
    return dict(case=case, session=s, tok=tok)


def prepare(case, seed):
    if case["op"] == "step":
        return _prepare_step(case, seed)
    st = dict(case=case, **_inputs(case, seed))
    f32, op = torch.float32, case["op"]
    if op == "attn":
        n, d = case["B"] * case["T"], case["H"] * case["dh"]
        st.update(o=_empty((n, d)), lse=_empty((case["B"], case["H"], case["T"]), f32),
                  delta=_empty((case["B"], case["H"], case["T"]), f32), dqkv=_empty((n, 3 * d)))
        return st
    N, d = case["N"], case["d"]
    if op == "norm":
        st.update(yn=_empty((N, d)), mean=_empty((N,), f32), rstd=_empty((N,), f32), dres_out=_empty((N, d), f32),
                  dres_lp=_empty((N, d)), dgamma=_empty((d,), f32), dbeta=_empty((d,), f32),
                  part=_empty((A.atom_k_layernorm_bwd_part_floats(N, d),), f32))
        return st
    st["ws"] = _empty((WS_BYTES // 4,), f32)
    if op == "head":
        Vp = st["w"].shape[0]
        st.update(logits=_empty((min(N, HEAD_CHUNK), Vp), f32), dz=_empty((N, Vp)), loss=_empty((N,), f32),
                  dy=_empty((N, d)), dw=_empty((Vp, d)))
        return st
    wide = 3 * d if op == "proj" else case["f"]
    st.update(dx_lp=st["dx"].to(BF16), part=_empty((A.atom_k_colsum_part_floats(N, wide),), f32))
    if op == "proj":
        st.update(qkv=_empty((N, 3 * d)), x1=_empty((N, d), f32), do=_empty((N, d)), da=_empty((N, d)),
                  dw_qkv=_empty((3 * d, d)), db_qkv=_empty((3 * d,), f32), dw_o=_empty((d, d)), db_o=_empty((d,), f32))
    else:
        f = case["f"]
        st.update(u=_empty((N, f)), g=_empty((N, f)), x2=_empty((N, d), f32), du=_empty((N, f)), dc=_empty((N, d)),
                  dw_fc=_empty((f, d)), db_fc=_empty((f,), f32), dw_pr=_empty((d, f)), db_pr=_empty((d,), f32))
    return st


# --------------------------------------------------------------------- runs
def _gemm(st, s, akc, bkc, epi, M, N, K, a, b, c, bias=None, resid=None, aux=None):
    p = lambda t: None if t is None else t.data_ptr()  # noqa: E731
    A.atom_k_gemm(A.ATOM_BF16, akc, bkc, epi, M, N, K, a.data_ptr(), a.stride(0), b.data_ptr(), b.stride(0),
                  c.data_ptr(), c.stride(0), p(bias), p(resid), p(aux), 0 if aux is None else aux.stride(0), s,
                  p(st["ws"]), WS_BYTES)


def _colsum(st, s, dt, x, out):
    A.atom_k_colsum(dt, x.data_ptr(), x.shape[0], x.shape[1], out.data_ptr(), st["part"].data_ptr(), s)


def _run_attn(st, s):
    c = st["case"]
    dims = (c["B"], c["T"], c["H"], c["dh"])
    A.atom_k_attn_fwd(A.ATOM_BF16, st["qkv"].data_ptr(), st["o"].data_ptr(), st["lse"].data_ptr(), *dims, s)
    A.atom_k_attn_bwd(A.ATOM_BF16, st["qkv"].data_ptr(), st["o"].data_ptr(), st["do"].data_ptr(), st["lse"].data_ptr(),
                      st["delta"].data_ptr(), st["dqkv"].data_ptr(), *dims, s)
    return dict(o=st["o"], lse=st["lse"], dqkv=st["dqkv"])


def _run_norm(st, s):
    N, d = st["x"].shape
    A.atom_k_layernorm_fwd(A.ATOM_BF16, st["x"].data_ptr(), st["gamma"].data_ptr(), st["beta"].data_ptr(),
                           st["yn"].data_ptr(), st["mean"].data_ptr(), st["rstd"].data_ptr(), N, d, s)
    # dres accumulates in place: each pass starts from the incoming gradient
    A.atom_k_copy(st["dres"].data_ptr(), st["dres_out"].data_ptr(), N * d * 4, s)
    A.atom_k_layernorm_bwd(A.ATOM_BF16, st["dy"].data_ptr(), st["x"].data_ptr(), st["mean"].data_ptr(),
                           st["rstd"].data_ptr(), st["gamma"].data_ptr(), st["dres_out"].data_ptr(),
                           st["dres_lp"].data_ptr(), 1, st["dgamma"].data_ptr(), st["dbeta"].data_ptr(),
                           st["part"].data_ptr(), N, d, s)
    return {k: st[k] for k in ("yn", "mean", "rstd", "dres_out", "dres_lp", "dgamma", "dbeta")}


def _run_proj(st, s):
    N, d = st["a"].shape
    _gemm(st, s, 1, 1, A.ATOM_EPI_BIAS, N, 3 * d, d, st["a"], st["w_qkv"], st["qkv"], st["b_qkv"])
    _gemm(st, s, 1, 1, A.ATOM_EPI_BIAS_RESID, N, d, d, st["o"], st["w_o"], st["x1"], st["b_o"], st["x"])
    _colsum(st, s, A.ATOM_F32, st["dx"], st["db_o"])
    _gemm(st, s, 0, 0, A.ATOM_EPI_STORE, d, d, N, st["dx_lp"], st["o"], st["dw_o"])
    _gemm(st, s, 1, 0, A.ATOM_EPI_STORE, N, d, d, st["dx_lp"], st["w_o"], st["do"])
    _colsum(st, s, A.ATOM_BF16, st["dqkv"], st["db_qkv"])
    _gemm(st, s, 0, 0, A.ATOM_EPI_STORE, 3 * d, d, N, st["dqkv"], st["a"], st["dw_qkv"])
    _gemm(st, s, 1, 0, A.ATOM_EPI_STORE, N, d, 3 * d, st["dqkv"], st["w_qkv"], st["da"])
    return {k: st[k] for k in ("qkv", "x1", "db_o", "dw_o", "do", "db_qkv", "dw_qkv", "da")}


def _run_mlp(st, s):
    N, d = st["c"].shape
    f = st["u"].shape[1]
    _gemm(st, s, 1, 1, A.ATOM_EPI_BIAS_GELU, N, f, d, st["c"], st["w_fc"], st["g"], st["b_fc"], aux=st["u"])
    _gemm(st, s, 1, 1, A.ATOM_EPI_BIAS_RESID, N, d, f, st["g"], st["w_pr"], st["x2"], st["b_pr"], st["x1"])
    _colsum(st, s, A.ATOM_F32, st["dx"], st["db_pr"])
    _gemm(st, s, 0, 0, A.ATOM_EPI_STORE, d, f, N, st["dx_lp"], st["g"], st["dw_pr"])
    _gemm(st, s, 1, 0, A.ATOM_EPI_GELU_BWD, N, f, d, st["dx_lp"], st["w_pr"], st["du"], aux=st["u"])
    _colsum(st, s, A.ATOM_BF16, st["du"], st["db_fc"])
    _gemm(st, s, 0, 0, A.ATOM_EPI_STORE, f, d, N, st["du"], st["c"], st["dw_fc"])
    _gemm(st, s, 1, 0, A.ATOM_EPI_STORE, N, d, f, st["du"], st["w_fc"], st["dc"])
    return {k: st[k] for k in ("g", "x2", "db_pr", "dw_pr", "du", "db_fc", "dw_fc", "dc")}


def _run_head(st, s):
    N, d = st["y"].shape
    Vp, V = st["w"].shape[0], st["case"]["V"]
    for r0 in range(0, N, HEAD_CHUNK):
        n = min(HEAD_CHUNK, N - r0)
        _gemm(st, s, 1, 1, A.ATOM_EPI_STORE_F32, n, Vp, d, st["y"][r0:], st["w"], st["logits"])
        A.atom_k_xent(A.ATOM_BF16, st["logits"].data_ptr(), Vp, st["tgt"][r0:].data_ptr(), st["dz"][r0:].data_ptr(), Vp,
                      st["loss"][r0:].data_ptr(), n, V, 1.0 / N, s)
    _gemm(st, s, 1, 0, A.ATOM_EPI_STORE, N, d, Vp, st["dz"], st["w"], st["dy"])
    _gemm(st, s, 0, 0, A.ATOM_EPI_STORE, Vp, d, N, st["dz"], st["y"], st["dw"])
    return {k: st[k] for k in ("loss", "dz", "dy", "dw")}


def _run_step(st):
    s, case = st["session"], st["case"]
    if case["steps"] == 1:
        losses = [s.step(st["tok"][0])]
    else:
        losses = [float(v) for v in s.steps(st["tok"])]
    grads = {}
    for node in range(s.n_nodes):
        for name, rows, _, _, _ in s.layout[node]:
            v = _host(s.host_view(node, name, A.GRAD_LAST), case["dtype"])
            v.session = s  # the library's buffer lives as long as its session
            grads["%d_%s" % (node, name)] = v
    return dict(loss=torch.tensor(losses, dtype=torch.float32), grads=grads)


_RUNS = dict(attn=_run_attn, norm=_run_norm, proj=_run_proj, mlp=_run_mlp, head=_run_head)


def run(state):
    if state["case"]["op"] == "step":
        return _run_step(state)
    return _RUNS[state["case"]["op"]](state, torch.cuda.current_stream().cuda_stream)


# --------------------------------------------------------------------- work
def _attn_flops(B, T, H, dh):
    # causal: forward 2 products, backward 5, of 2 T (T + 1) / 2 dh each
    return 7 * B * H * T * (T + 1) * dh


def work(case):
    op = case["op"]
    if op == "attn":
        n, d = case["B"] * case["T"], case["H"] * case["dh"]
        # forward reads qkv and writes o, lse; backward reads qkv, o, do, lse and writes dqkv
        return dict(bytes=2 * (n * d * (3 + 1 + 3 + 1 + 1 + 3)) + 8 * n * case["H"], flops=_attn_flops(
            case["B"], case["T"], case["H"], case["dh"]))
    if op == "step":
        N, d, f, L = case["B"] * case["T"], case["d"], case["f"], case["L"]
        e = 2 if case["dtype"] == "bf16" else 4
        n_par = case["V"] * d * 2 + case["T"] * d + L * (4 * d * d + 2 * d * f)
        micro = case["C"] * case["steps"]
        flops = micro * (6 * N * (L * (4 * d * d + 2 * d * f) + case["V"] * d) + L * _attn_flops(
            case["B"], case["T"], case["H"], d // case["H"]))
        # weights in once, gradients out every step, block inputs written and read, fp32
        return dict(bytes=n_par * e * (1 + case["steps"]) + micro * 8 * (L + 1) * N * d, flops=flops)
    N, d = case["N"], case["d"]
    if op == "norm":
        # forward: x, y, statistics; backward: dy, x, statistics, dres in and out, its bf16 copy
        return dict(bytes=N * d * (4 + 2 + 2 + 4 + 4 + 4 + 2) + 16 * N + 12 * d, flops=16 * N * d)
    if op == "head":
        V = case["V"]
        return dict(bytes=2 * (2 * N * d + 2 * V * d) + 2 * N * V + 8 * N, flops=6 * N * V * d)
    if op == "proj":
        return dict(bytes=2 * (2 * 4 * d * d + N * d * (2 + 3 + 1 + 3 + 1 + 1)) + 4 * N * d * 3, flops=6 * N * 4 * d * d)
    f = case["f"]
    return dict(bytes=2 * (4 * d * f + N * d * 2 + N * d + 3 * N * f) + 4 * N * d * 3, flops=6 * N * 2 * d * f)


def tolerance(case):
    # about four times the largest error against exact(): one bf16 rounding
    # (1.7e-3) where operands are exact, more where an intermediate is rounded
    # too (attention 2.4e-3, MLP 3.2e-3), and 6e-3 through a whole bf16 model;
    # 1e-6 for the fp32 step, stated with room for other summation orders
    if case["op"] == "step":
        return {"rel": 1e-5} if case["dtype"] == "f32" else {"rel": 2e-2}
    return {"rel": {"attn": 1e-2, "norm": 7e-3, "proj": 7e-3, "mlp": 1.2e-2, "head": 7e-3}[case["op"]]}


# -------------------------------------------------------------------- exact
def _gelu(u):
    return 0.5 * u * (1 + torch.tanh(0.7978845608028654 * (u + 0.044715 * u ** 3)))


def _layer_norm(x, gamma, beta):
    mean = x.mean(-1, keepdim=True)
    rstd = (((x - mean) ** 2).mean(-1, keepdim=True) + 1e-5).rsqrt()
    return (x - mean) * rstd * gamma + beta, mean.squeeze(-1), rstd.squeeze(-1)


def _attention(qkv, B, T, H, dh):
    x = qkv.view(B, T, 3, H, dh).permute(2, 0, 3, 1, 4).contiguous()
    s = torch.matmul(x[0], x[1].transpose(-1, -2).contiguous()) / math.sqrt(dh)
    s = s.masked_fill(torch.ones(T, T, device=s.device, dtype=torch.bool).triu(1), float("-inf"))
    lse = torch.logsumexp(s, -1)
    o = torch.matmul(torch.exp(s - lse.unsqueeze(-1)), x[2])
    return o.permute(0, 2, 1, 3).reshape(B * T, H * dh), lse


def _model_loss(case, w, tok):
    """Mean cross-entropy of one micro-batch (tok [B][T + 1])."""
    B, T, H, d = case["B"], case["T"], case["H"], case["d"]
    t = torch.from_numpy(tok).long().cuda()
    x = (w[0]["wte"][t[:, :T]] + w[0]["wpe"]).view(B * T, d)
    for p in w[1:-1]:
        a = _layer_norm(x, p["ln1_g"], p["ln1_b"])[0]
        o, _ = _attention(a @ p["w_qkv"].T + p["b_qkv"], B, T, H, d // H)
        x = x + o @ p["w_o"].T + p["b_o"]
        c = _layer_norm(x, p["ln2_g"], p["ln2_b"])[0]
        x = x + _gelu(c @ p["w_fc"].T + p["b_fc"]) @ p["w_pr"].T + p["b_pr"]
    z = _layer_norm(x, w[-1]["lnf_g"], w[-1]["lnf_b"])[0] @ w[-1]["w_head"].T
    return (torch.logsumexp(z, -1) - z.gather(1, t[:, 1:].reshape(-1, 1)).squeeze(1)).mean()


def _exact_step(case, seed):
    cfg, weights, tok = _step_inputs(case, seed)
    w = [{k: v.double().requires_grad_() for k, v in p.items()} for p in weights]
    losses = []
    for k in range(case["steps"]):
        last = k == case["steps"] - 1
        total = 0.0
        for micro in range(case["C"]):
            with torch.set_grad_enabled(last):
                loss = _model_loss(case, w, tok[k, micro]) / case["C"]
            if last:
                loss.backward()
            total += loss.item()
        losses.append(total)
    grads = {}
    for node, p in enumerate(w):
        for name, v in p.items():
            g = v.grad
            if name == "w_head":
                pad = (cfg.vocab + 127) // 128 * 128 - cfg.vocab
                g = torch.cat([g, g.new_zeros(pad, cfg.d_model)])
            grads["%d_%s" % (node, name)] = g.cpu()
    return dict(loss=torch.tensor(losses, dtype=torch.float64), grads=grads)


def exact(case, seed):
    if case["op"] == "step":
        return _exact_step(case, seed)
    x = {k: v.double() if v.is_floating_point() else v for k, v in _inputs(case, seed).items()}
    op = case["op"]
    if op == "attn":
        n, d = case["B"] * case["T"], case["H"] * case["dh"]
        o = torch.empty(case["B"], case["T"], d, device="cuda", dtype=torch.float64)
        lse, dqkv = [], []
        for b in range(case["B"]):
            q = x["qkv"].view(case["B"], case["T"], 3 * d)[b].clone().requires_grad_()
            ob, lb = _attention(q, 1, case["T"], case["H"], case["dh"])
            ob.backward(x["do"].view(case["B"], case["T"], d)[b])
            o[b] = ob.detach()
            lse.append(lb.detach())
            dqkv.append(q.grad)
        return dict(o=o.view(n, d), lse=torch.cat(lse), dqkv=torch.cat(dqkv))
    if op == "norm":
        leaf = {k: x[k].requires_grad_() for k in ("x", "gamma", "beta")}
        y, mean, rstd = _layer_norm(leaf["x"], leaf["gamma"], leaf["beta"])
        y.backward(x["dy"])
        dres = x["dres"] + leaf["x"].grad
        return dict(yn=y.detach(), mean=mean.detach(), rstd=rstd.detach(), dres_out=dres, dres_lp=dres,
                    dgamma=leaf["gamma"].grad, dbeta=leaf["beta"].grad)
    if op == "proj":
        lp = x["dx"].to(BF16).double()  # the backward's operand is the bf16 copy
        return dict(qkv=x["a"] @ x["w_qkv"].T + x["b_qkv"], x1=x["x"] + x["o"] @ x["w_o"].T + x["b_o"],
                    db_o=x["dx"].sum(0), dw_o=lp.T @ x["o"], do=lp @ x["w_o"], db_qkv=x["dqkv"].sum(0),
                    dw_qkv=x["dqkv"].T @ x["a"], da=x["dqkv"] @ x["w_qkv"])
    if op == "mlp":
        lp = x["dx"].to(BF16).double()
        u = (x["c"] @ x["w_fc"].T + x["b_fc"]).requires_grad_()
        g = _gelu(u)
        g.backward(lp @ x["w_pr"])
        g, du = g.detach(), u.grad
        return dict(g=g, x2=x["x1"] + g @ x["w_pr"].T + x["b_pr"], db_pr=x["dx"].sum(0), dw_pr=lp.T @ g, du=du,
                    db_fc=du.sum(0), dw_fc=du.T @ x["c"], dc=du @ x["w_fc"])
    N, V = case["N"], case["V"]
    z = x["y"] @ x["w"][:V].T
    lse = torch.logsumexp(z, -1)
    t = x["tgt"].long().unsqueeze(1)
    loss = lse - z.gather(1, t).squeeze(1)
    p = torch.exp(z - lse.unsqueeze(1))
    p.scatter_add_(1, t, torch.full_like(loss, -1.0).unsqueeze(1))
    p /= N
    dz = torch.cat([p, p.new_zeros(N, x["w"].shape[0] - V)], 1)
    return dict(loss=loss, dz=dz, dy=dz @ x["w"], dw=dz.T @ x["y"])
