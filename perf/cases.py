"""Performance cases: what a program that trains decoders with this library has it do, at the sizes of the library's
own workloads, tests and benchmark.

A case is a plain dict.  Its "kind" names the piece of a training step it runs:

  linear     one linear layer, forward and backward (y, dx, dW), as the shard executor calls its products
  attention  one causal self-attention layer, forward and backward (bf16 operands)
  norm       one LayerNorm, forward and backward with the residual gradient added
  head       LM head: logits, cross-entropy, d(loss)/dz and d(loss)/dW
  adam       the optimizer step of one shard
  manual     a whole training step in fp32, shard by shard through the low-level calls (logits, loss, gradients, state)
  sched      a whole scheduled training step of two spilled bf16 models with micro-batches (state back in host memory)

Everything goes through the public entry points (paper_2110_08633_amd.hydra and .runtime).
"""
import math
import weakref

import torch

from paper_2110_08633_amd import hydra as H
from paper_2110_08633_amd import runtime as R

LR, BETA1, BETA2, EPS = 1e-4, 0.9, 0.999, 1e-8


def listed():
    return [
        # The smallest products: one short sample (an odd number of tokens) through the QKV projection of the smallest
        # GPT-2.  Launches and latency count.
        dict(name="linear_short", kind="linear", dtype="bf16", M=201, K=768, N=2304, acc=False),
        # MLP down projection of GPT-2 small at the benchmark's 4 x 512 tokens, a later micro-batch: dW is added to.
        dict(name="linear_gpt2s", kind="linear", dtype="bf16", M=2048, K=3072, N=768, acc=True),
        # MLP up projection of GPT-2 XL (width 1600 = 25 heads) on a sample whose length fills no tile.
        dict(name="linear_xl_ragged", kind="linear", dtype="bf16", M=1000, K=1600, N=6400, acc=False),
        # MLP up projection of the 6 B model at its 1024 tokens: the largest product of a block.
        dict(name="linear_6b", kind="linear", dtype="bf16", M=1024, K=4096, N=16384, acc=False),
        # The fp32 path (parity runs, models trained without reduced precision), GPT-2 small width.
        dict(name="linear_f32", kind="linear", dtype="f32", M=1000, K=768, N=3072, acc=False),
        # Attention of GPT-2 small at the benchmark's batch.
        dict(name="attention_gpt2s", kind="attention", B=4, H=12, T=512, dh=64),
        # Long sequences at the 6 B model's head width.
        dict(name="attention_long", kind="attention", B=4, H=16, T=2048, dh=128),
        # LayerNorm at the XL width, two of its samples in two micro-batches' worth of rows.
        dict(name="norm_xl", kind="norm", dtype="bf16", M=4096, d=1600),
        # LM head of GPT-2 small: the vocabulary is odd.
        dict(name="head_gpt2s", kind="head", M=2048, d=768, V=50257, T=512),
        # Adam on a four-block shard of GPT-2 medium.
        dict(name="adam_gpt2m", kind="adam", n=50384896, shadow=True),
        # The test suite's tiny fp32 decoder, whole step: dozens of small launches, copies and waits.
        dict(name="manual_tiny", kind="manual", L=2, d=128, H=4, F=512, V=512, T=64, B=2, k=1),
        # Two models of GPT-2 small width, two shards each, spilled, eight micro-batches per visit (where the
        # benchmark's transfers and compute are about equal).
        dict(name="sched_two_models", kind="sched", L=2, d=768, H=12, F=3072, V=8192, T=512, B=4, k=1, n_micro=8),
    ]


def _logu(rng, lo, hi, mult=1):
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(lo, min(hi, int(round(v / mult)) * mult))


def draw(rng):
    kind = rng.choice(["linear", "linear", "linear", "linear", "attention", "attention", "norm", "head", "adam",
                       "manual", "sched"])
    if kind == "linear":
        dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
        top = 1024 * 4096 * 16384 if dtype == "bf16" else 1000 * 768 * 3072
        while True:
            K, N = (_logu(rng, 128, 16384, 8) for _ in range(2))  # widths are multiples of 8, token counts are not
            M = _logu(rng, 64, 8192)
            if M * K * N <= top:
                return dict(kind=kind, dtype=dtype, M=M, K=K, N=N, acc=rng.random() < 0.5)
    if kind == "attention":
        while True:
            c = dict(kind=kind, B=rng.randint(1, 8), H=rng.choice([4, 12, 16, 25, 32]), T=_logu(rng, 64, 2048, 8),
                     dh=rng.choice([64, 128]))
            if c["B"] * c["H"] * c["dh"] * c["T"] ** 2 <= 4 * 16 * 128 * 2048 ** 2:
                return c
    if kind == "norm":
        while True:
            M, d = _logu(rng, 64, 16384), _logu(rng, 128, 2048, 8)
            if M * d <= 4096 * 1600:
                return dict(kind=kind, dtype=rng.choice(["bf16", "bf16", "f32"]), M=M, d=d)
    if kind == "head":
        while True:
            T = _logu(rng, 64, 1024, 8)
            M, d, V = T * rng.randint(1, 4), _logu(rng, 256, 1600, 8), _logu(rng, 1000, 50400)
            if M * d * V <= 2048 * 768 * 50257 and M * V <= 2048 * 50257:
                return dict(kind=kind, M=M, d=d, V=V, T=T)
    if kind == "adam":
        return dict(kind=kind, n=_logu(rng, 10000, 50384896), shadow=rng.random() < 0.7)
    if kind == "manual":
        k = rng.randint(1, 2)
        heads = rng.choice([2, 4, 8])
        d = heads * rng.choice([16, 32])
        return dict(kind=kind, L=2, d=d, H=heads, F=4 * d, V=rng.randint(200, 512), T=8 * rng.randint(3, 8),
                    B=rng.randint(1, 2), k=k)
    heads = rng.choice([6, 8, 12])
    d = heads * 64
    return dict(kind=kind, L=2, d=d, H=heads, F=4 * d, V=rng.randint(2000, 8192), T=8 * rng.randint(16, 64),
                B=rng.randint(1, 4), k=rng.randint(1, 2), n_micro=rng.randint(1, 8))


# ---------------------------------------------------------------------------------------------------------- inputs

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _randn(g, *shape, std=1.0, mean=0.0):
    return torch.randn(*shape, generator=g, device="cuda") * std + mean


def _inputs(case, seed):
    g, k = _gen(seed), case["kind"]
    if k == "linear":
        M, K, N = case["M"], case["K"], case["N"]
        act = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
        i = dict(x=_randn(g, M, K).to(act), w=_randn(g, K, N, std=0.02).to(act), b=_randn(g, N, std=0.02),
                 dy=_randn(g, M, N, std=1e-2).to(act))
        if case["acc"]:
            i["prev"] = _randn(g, K, N, std=0.1)
        return i
    if k == "attention":
        rows, d = case["B"] * case["T"], case["H"] * case["dh"]
        return dict(qkv=_randn(g, rows, 3 * d).bfloat16(), d_o=_randn(g, rows, d, std=1e-2).bfloat16())
    if k == "norm":
        M, d = case["M"], case["d"]
        return dict(x=_randn(g, M, d, std=2.0, mean=0.5), gamma=_randn(g, d, std=0.1, mean=1.0), beta=_randn(g, d, std=0.1),
                    dy=_randn(g, M, d, std=1e-2), dres=_randn(g, M, d, std=1e-2))
    if k == "head":
        M, d, V = case["M"], case["d"], case["V"]
        tgt = torch.randint(0, V, (M,), generator=g, device="cuda", dtype=torch.int32)
        tgt[case["T"] - 1::case["T"]] = -1  # the last position of a sample predicts nothing
        return dict(z=_randn(g, M, d).bfloat16(), w=_randn(g, V, d, std=0.02).bfloat16(), tgt=tgt)
    if k == "adam":
        n = case["n"]
        return dict(w=_randn(g, n, std=0.02), m=_randn(g, n, std=1e-3), v=_randn(g, n, std=1e-3) ** 2,
                    g=_randn(g, n, std=1e-2))
    models = []
    for _ in range(2 if k == "sched" else 1):
        lay, total = _layout(case)
        flat = _randn(g, total, std=0.02)
        for name, (off, shape) in lay.items():
            if name.endswith("_g"):
                flat[off:off + shape[0]] += 1.0
        rows = case.get("n_micro", 1) * case["B"]
        tok = torch.randint(0, case["V"], (rows, case["T"]), generator=g, device="cuda", dtype=torch.int32)
        tgt = torch.cat([tok[:, 1:], torch.full_like(tok[:, :1], -1)], 1)
        models.append((flat, tok, tgt))
    return models


def _layout(case):
    """name -> (offset, shape) of the canonical flat parameter layout, and its length."""
    L, d, F, V, T = (case[k] for k in ("L", "d", "F", "V", "T"))
    shapes = [("wte", (V, d)), ("wpe", (T, d))]
    for i in range(L):
        shapes += [(f"h{i}.{n}", s) for n, s in (
            ("ln1_g", (d,)), ("ln1_b", (d,)), ("w_qkv", (d, 3 * d)), ("b_qkv", (3 * d,)), ("w_o", (d, d)), ("b_o", (d,)),
            ("ln2_g", (d,)), ("ln2_b", (d,)), ("w_fc", (d, F)), ("b_fc", (F,)), ("w_proj", (F, d)), ("b_proj", (d,)))]
    shapes += [("lnf_g", (d,)), ("lnf_b", (d,)), ("w_lm", (d, V))]
    out, off = {}, 0
    for name, s in shapes:
        out[name] = (off, s)
        off += math.prod(s)
    return out, off


class _State:
    """What a program holds between the calls."""


def _pinned(src):
    """Page-locked copy of a float32 tensor (or zeros of a length) as a numpy array that owns its memory."""
    n = src if isinstance(src, int) else src.numel()
    t = torch.empty(n, dtype=torch.float32, pin_memory=True)
    if isinstance(src, int):
        t.zero_()
    else:
        t.copy_(src)
    return t.numpy()


def prepare(case, seed):
    s, k = _State(), case["kind"]
    i = _inputs(case, seed)
    s.case, s.i = case, i
    if k == "linear":
        M, K, N = case["M"], case["K"], case["N"]
        s.dt = 1 if case["dtype"] == "bf16" else 0
        if s.dt:
            s.wt = i["w"].t().contiguous()  # the transposed working copy that forward products multiply by
        s.y = torch.empty(M, N, dtype=i["x"].dtype, device="cuda")
        s.dx, s.dw = torch.empty(M, K, device="cuda"), torch.empty(K, N, device="cuda")
    elif k == "attention":
        rows, d = case["B"] * case["T"], case["H"] * case["dh"]
        s.o = torch.empty(rows, d, dtype=torch.bfloat16, device="cuda")
        s.lse, s.dsum = (torch.empty(case["B"] * case["H"] * case["T"], device="cuda") for _ in range(2))
        s.dqkv = torch.empty(rows, 3 * d, dtype=torch.bfloat16, device="cuda")
    elif k == "norm":
        M, d = case["M"], case["d"]
        s.y = torch.empty(M, d, dtype=torch.bfloat16 if case["dtype"] == "bf16" else torch.float32, device="cuda")
        s.mean, s.rstd = torch.empty(M, device="cuda"), torch.empty(M, device="cuda")
        s.dx, s.dxh = torch.empty(M, d, device="cuda"), torch.empty(M, d, dtype=torch.bfloat16, device="cuda")
        s.cols = [torch.empty(d, device="cuda") for _ in range(3)]
        s.scratch = torch.empty(3 * d * ((M + 7) // 8), device="cuda")
    elif k == "head":
        M, d, V = case["M"], case["d"], case["V"]
        s.ld = (V + 63) // 64 * 64
        s.inv_n = 1.0 / int((i["tgt"] >= 0).sum())
        s.logits = torch.zeros(M, s.ld, device="cuda")
        s.dlogits = torch.empty(M, s.ld, dtype=torch.bfloat16, device="cuda")
        s.row, s.dz, s.dw = torch.empty(M, device="cuda"), torch.empty(M, d, device="cuda"), torch.empty(d, V, device="cuda")
    elif k == "adam":
        s.shadow = torch.empty(case["n"], dtype=torch.bfloat16, device="cuda") if case["shadow"] else None
        s.t = 0
    else:
        cfg = {n: case[n] for n in ("L", "d", "H", "F", "V", "T", "B", "k")}
        cfg.update(dtype="bf16" if k == "sched" else "f32", n_micro=case.get("n_micro", 1))
        lanes, slots = (2, 6) if k == "sched" else (1, 2)
        s.sess = R.Session(R.arena_bytes_for([cfg] * len(i), slots, lanes=lanes), max_slots=slots, lanes=lanes)
        weakref.finalize(s, s.sess.close)
        s.recs = []
        for flat, _, _ in i:
            host = (_pinned(flat), _pinned(flat.numel()), _pinned(flat.numel()))
            s.recs.append(s.sess.add_model(cfg, None, LR, host=host))
            assert s.recs[-1]["layout"].n_params == flat.numel()
        s.tok = [t.cpu().numpy() for _, t, _ in i]
        s.tgt = [t.cpu().numpy() for _, _, t in i]
        if k == "sched":
            S = s.recs[0]["S"]
            block, ends = cfg["k"] * 12 * cfg["d"] ** 2, cfg["d"] * cfg["V"]
            fwd = [1] + [block] * S + [ends]  # cost table: multiply-adds per token
            s.costs = [fwd + [3 * c for c in fwd]] * len(i)
    torch.cuda.synchronize()
    return s


def run(s):
    case, i, k = s.case, s.i, s.case["kind"]
    if k == "linear":
        M, K, N = case["M"], case["K"], case["N"]
        x, w, dy = i["x"], i["w"], i["dy"]
        if s.dt:
            H.hydra_op_gemm(1, 0, 0, M, N, K, 1.0, x, K, s.wt, K, i["b"], None, None, s.y, N)
        else:
            H.hydra_op_gemm(0, 0, 1, M, N, K, 1.0, x, K, w, N, i["b"], None, None, s.y, N)
        H.hydra_op_gemm(s.dt, 0, 0, M, K, N, 1.0, dy, N, w, N, None, None, s.dx, None, K)
        H.hydra_op_gemm(s.dt, 1, 1, K, N, M, 1.0, x, K, dy, N, None, i.get("prev"), s.dw, None, N)
        return dict(y=s.y, dx=s.dx, dw=s.dw)
    if k == "attention":
        dims = (case["B"], case["H"], case["T"], case["dh"])
        H.hydra_op_attention_fwd(i["qkv"], s.o, s.lse, *dims)
        H.hydra_op_attention_bwd(i["qkv"], s.o, i["d_o"], s.lse, s.dsum, s.dqkv, *dims)
        return dict(o=s.o, lse=s.lse, dqkv=s.dqkv)
    if k == "norm":
        M, d = case["M"], case["d"]
        H.hydra_op_layernorm_fwd(1 if case["dtype"] == "bf16" else 0, i["x"], i["gamma"], i["beta"], s.y, s.mean, s.rstd,
                                 M, d)
        H.hydra_op_layernorm_bwd(i["dy"], i["x"], s.mean, s.rstd, i["gamma"], i["dres"], s.dx, s.dxh, *s.cols, s.scratch,
                                 M, d)
        return dict(y=s.y, mean=s.mean, rstd=s.rstd, dx=s.dx, dx_bf16=s.dxh, dgamma=s.cols[0], dbeta=s.cols[1],
                    dx_colsum=s.cols[2])
    if k == "head":
        M, d, V, ld = case["M"], case["d"], case["V"], s.ld
        H.hydra_op_gemm(1, 0, 0, M, V, d, 1.0, i["z"], d, i["w"], d, None, None, s.logits, None, ld)
        H.hydra_op_cross_entropy(1, s.logits, i["tgt"], s.row, s.dlogits, M, V, ld, s.inv_n)
        H.hydra_op_gemm(1, 1, 1, d, V, M, 1.0, i["z"], d, s.dlogits, ld, None, None, s.dw, None, V)
        H.hydra_op_gemm(1, 0, 1, M, d, V, 1.0, s.dlogits, ld, i["w"], d, None, None, s.dz, None, d)
        return dict(logits=s.logits, row_loss=s.row, dlogits=s.dlogits, dz=s.dz, dw=s.dw)
    if k == "adam":
        s.t += 1
        H.hydra_op_adam(i["w"], i["m"], i["v"], i["g"], s.shadow, case["n"], LR, BETA1, BETA2, EPS, s.t)
        out = dict(w=i["w"], m=i["m"], v=i["v"])
        if s.shadow is not None:
            out["shadow"] = s.shadow
        return out
    if k == "manual":
        rec = s.recs[0]
        got = s.sess.train_step_manual(rec, s.tok[0], s.tgt[0])
        H.hydra_sync(s.sess.ctx)
        out = dict(logits=got["logits"], loss=got["loss"], w=rec["master"], m=rec["m"], v=rec["v"])
        out.update({"grad." + n: a for n, a in got["grads"].items()})
        return out
    sched = H.hydra_sched_create(s.sess.ctx, [r["id"] for r in s.recs], [1] * len(s.recs), s.costs)
    H.hydra_sched_run(sched, s.tok, s.tgt, s.sess.ctx)
    s.sess.flush()
    out = {}
    for n, rec in enumerate(s.recs):
        out.update({f"loss{n}": H.hydra_get_loss(s.sess.ctx, rec["id"]), f"w{n}": rec["master"], f"m{n}": rec["m"],
                    f"v{n}": rec["v"]})
    H.hydra_sched_destroy(sched)
    return out


def work(case):
    k = case["kind"]
    if k == "linear":
        M, K, N = case["M"], case["K"], case["N"]
        e = 2 if case["dtype"] == "bf16" else 4
        return dict(bytes=e * (M * K + K * N + 2 * M * N) + 4 * (N + M * K + K * N * (2 if case["acc"] else 1)),
                    flops=6 * M * N * K)
    if k == "attention":
        rows, d = case["B"] * case["T"], case["H"] * case["dh"]
        # qkv, d_o in; o, dqkv, lse out; two causal products forward, five backward
        return dict(bytes=18 * rows * d + 4 * rows * case["H"], flops=7 * rows * d * (case["T"] + 1))
    if k == "norm":
        M, d = case["M"], case["d"]
        return dict(bytes=M * d * (18 + (2 if case["dtype"] == "bf16" else 4)) + 8 * M + 20 * d, flops=25 * M * d)
    if k == "head":
        M, d, V = case["M"], case["d"], case["V"]
        return dict(bytes=2 * (M * d + V * d) + 4 * M + 6 * M * V + 4 * (M + M * d + d * V), flops=6 * M * V * d + 8 * M * V)
    if k == "adam":
        return dict(bytes=case["n"] * (30 if case["shadow"] else 28), flops=15 * case["n"])
    _, n = _layout(case)
    models = 2 if k == "sched" else 1
    rows = case.get("n_micro", 1) * case["B"] * case["T"]
    dense = 12 * case["d"] ** 2 * case["L"] + case["d"] * case["V"]
    grads = 4 * n + 4 * rows * case["V"] if k == "manual" else 0
    return dict(bytes=models * (24 * n + 8 * rows + grads),
                flops=models * rows * (6 * dense + 7 * case["L"] * case["d"] * (case["T"] + 1)))


def tolerance(case):
    """About four times the error measured against exact(); bf16 results carry 1.7e-3 from their own rounding."""
    k = case["kind"]
    if k == "linear":
        return {"rel": 7e-3} if case["dtype"] == "bf16" else {"rel": 5e-6}
    if k == "attention":
        return {"rel": 1e-2}
    if k == "norm":
        return {"rel": 7e-3}
    if k == "head":
        return {"rel": 8e-3}
    if k == "adam":
        return {"rel": 7e-3} if case["shadow"] else {"rel": 1e-6}
    if k == "manual":
        return {"rel": 1e-5}
    return {"rel": 3e-2}  # bf16 through a whole model; second moments hold the square of the gradient


# ------------------------------------------------------------------------------------------------- 64-bit results

def _attention64(q, k, v):
    """q, k, v [B, H, T, dh] -> output and log-sum-exp."""
    T = q.shape[2]
    s = (q @ k.transpose(2, 3).contiguous()) / math.sqrt(q.shape[3])
    s = s.masked_fill(torch.ones(T, T, dtype=torch.bool, device=s.device).triu(1), -math.inf)
    lse = torch.logsumexp(s, -1)
    return torch.exp(s - lse[..., None]) @ v, lse


def _heads(x, B, T, H):
    return x.reshape(B, T, H, -1).transpose(1, 2)


def _norm64(x, g, b):
    mu = x.mean(-1, keepdim=True)
    rs = 1.0 / torch.sqrt(((x - mu) ** 2).mean(-1, keepdim=True) + 1e-5)
    return (x - mu) * rs * g + b, mu, rs


def _loss64(case, W, tok, tgt):
    """Loss of one minibatch (mean over its valid targets) and the logits of its last micro-batch."""
    B, T, Hn, d = tok.shape[0], case["T"], case["H"], case["d"]
    x = W["wte"][tok.long()].reshape(-1, d) + W["wpe"].repeat(B, 1)
    for n in range(case["L"]):
        P = {k[len(f"h{n}."):]: v for k, v in W.items() if k.startswith(f"h{n}.")}
        a, _, _ = _norm64(x, P["ln1_g"], P["ln1_b"])
        q, k, v = ((a @ P["w_qkv"] + P["b_qkv"])[:, j * d:(j + 1) * d] for j in range(3))
        o, _ = _attention64(*(_heads(t, B, T, Hn) for t in (q, k, v)))
        x = x + o.transpose(1, 2).reshape(-1, d) @ P["w_o"] + P["b_o"]
        c, _, _ = _norm64(x, P["ln2_g"], P["ln2_b"])
        u = c @ P["w_fc"] + P["b_fc"]
        u = 0.5 * u * (1.0 + torch.tanh(math.sqrt(2.0 / math.pi) * (u + 0.044715 * u ** 3)))
        x = x + u @ P["w_proj"] + P["b_proj"]
    z, _, _ = _norm64(x, W["lnf_g"], W["lnf_b"])
    logits = z @ W["w_lm"]
    t = tgt.reshape(-1).long()
    keep = t >= 0
    lp = torch.log_softmax(logits, -1)
    nll = -lp.gather(1, t.clamp(min=0)[:, None])[:, 0]
    return (nll * keep).sum() / keep.sum(), logits[-case["B"] * T:]


def exact(case, seed):
    k = case["kind"]
    i = _inputs(case, seed)
    if k == "linear":
        x, w, dy = (i[n].double() for n in ("x", "w", "dy"))
        dw = x.t() @ dy
        if case["acc"]:
            dw += i["prev"].double()
        return dict(y=x @ w + i["b"].double(), dx=dy @ w.t(), dw=dw)
    if k == "attention":
        B, Hn, T = case["B"], case["H"], case["T"]
        d = Hn * case["dh"]
        qkv, d_o = i["qkv"].double(), i["d_o"].double()
        o, lse = torch.empty(B * T, d, dtype=torch.float64, device="cuda"), []
        dqkv = torch.empty_like(qkv)
        for b in range(B):  # a sample at a time: the score matrices in 64 bits are large
            rows = slice(b * T, (b + 1) * T)
            x = qkv[rows].clone().requires_grad_()
            ob, lb = _attention64(*(_heads(x[:, j * d:(j + 1) * d], 1, T, Hn) for j in range(3)))
            ob = ob.transpose(1, 2).reshape(T, d)
            ob.backward(d_o[rows])
            o[rows], dqkv[rows] = ob.detach(), x.grad
            lse.append(lb.detach().reshape(-1))
        return dict(o=o, lse=torch.cat(lse), dqkv=dqkv)
    if k == "norm":
        x, gm, bt = (i[n].double().requires_grad_() for n in ("x", "gamma", "beta"))
        y, mu, rs = _norm64(x, gm, bt)
        y.backward(i["dy"].double())
        dx = x.grad + i["dres"].double()
        return dict(y=y.detach(), mean=mu.detach()[:, 0], rstd=rs.detach()[:, 0], dx=dx, dx_bf16=dx, dgamma=gm.grad,
                    dbeta=bt.grad, dx_colsum=dx.sum(0))
    if k == "head":
        M, V = case["M"], case["V"]
        z, w, t = i["z"].double(), i["w"].double(), i["tgt"].long()
        keep = t >= 0
        l = z @ w.t()
        ls = torch.logsumexp(l, -1)
        at = t.clamp(min=0)[:, None]
        row = (ls - l.gather(1, at)[:, 0]) * keep
        p = torch.exp(l - ls[:, None])
        p.scatter_add_(1, at, torch.full((M, 1), -1.0, dtype=torch.float64, device="cuda"))
        p *= (keep / keep.sum())[:, None]
        pad = (0, (V + 63) // 64 * 64 - V)
        return dict(logits=torch.nn.functional.pad(l, pad), row_loss=row, dlogits=torch.nn.functional.pad(p, pad),
                    dz=p @ w, dw=z.t() @ p)
    if k == "adam":
        w, m, v, g = (i[n].double() for n in ("w", "m", "v", "g"))
        w, m, v = _adam64(w, m, v, g)
        out = dict(w=w, m=m, v=v)
        if case["shadow"]:
            out["shadow"] = w
        return out
    out = {}
    for n, (flat, tok, tgt) in enumerate(i):
        flat = flat.double()
        lay, _ = _layout(case)
        leaf = flat.clone().requires_grad_()
        W = {name: leaf[off:off + math.prod(s)].reshape(s) for name, (off, s) in lay.items()}
        loss, logits = _loss64(case, W, tok, tgt)
        loss.backward()
        g = leaf.grad
        w, m, v = (a.cpu().numpy() for a in _adam64(flat, torch.zeros_like(flat), torch.zeros_like(flat), g))
        if k == "manual":
            out = dict(logits=logits.detach().cpu().numpy(), loss=float(loss.detach()), w=w, m=m, v=v)
            out.update({"grad." + name: g[off:off + math.prod(s)].reshape(s).cpu().numpy()
                        for name, (off, s) in lay.items()})
        else:
            out.update({f"loss{n}": float(loss.detach()), f"w{n}": w, f"m{n}": m, f"v{n}": v})
    return out


def _adam64(w, m, v, g):
    """The first step (t = 1)."""
    m = BETA1 * m + (1 - BETA1) * g
    v = BETA2 * v + (1 - BETA2) * g * g
    return w - LR * (m / (1 - BETA1)) / (torch.sqrt(v / (1 - BETA2)) + EPS), m, v
