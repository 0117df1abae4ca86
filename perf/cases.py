"""The calls that a program makes of this library, as cases to be timed and compared.

Each case names one public entry point and the sizes, data type and options of the call:

    forward     qdelta.chunk_fwd            prefill: outputs and the final state
    segmented   qdelta.chunk_fwd_segmented  one long sequence over few heads, segment count left to the library
    train       qdelta.chunk_fwd + chunk_bwd, workspaces kept by the caller
    autograd    layer.qdelta_chunk forward and backward
    layer       layer.QDeltaLayer forward and backward, projections included
    decode      qdelta.recurrent_step       one token per sequence, state updated in place
    recurrent   qdelta.recurrent_fwd        a few tokens per continuing sequence
    rec_train   qdelta.recurrent_fwd + recurrent_bwd

q and k are unit vectors per head, v and the output gradients standard normal, beta and lambda
sigmoid(N(0, 1)); log alpha is logsigmoid(N(0, 1)) ("fast" decay), logsigmoid(N(4, 1)) ("slow") or absent.
"""
import math
import random

import torch
import torch.nn.functional as F

from paper_2606_08804_amd import layer as qlayer
from paper_2606_08804_amd import qdelta

CHUNK = 64      # of the reference below; the result does not depend on it


def _case(op, batch, tokens, heads, dk, dv, dtype="bf16", decay="fast", lam="token", state=True, packed=False,
          d_model=0, name=None):
    """lam: "token" (per token and head) or a number; packed: `tokens` in all, in `batch` sequences."""
    c = dict(op=op, batch=batch, tokens=tokens, heads=heads, dk=dk, dv=dv, dtype=dtype, decay=decay, lam=lam,
             state=state, packed=packed, d_model=d_model)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest layer of the tests and the benchmark: launches and latency
        _case("forward", 1, 256, 2, 64, 64, "f32", state=False, name="forward_tiny_f32"),
        # prefill of a batch of prompts, the benchmark's forward shape
        _case("forward", 8, 2048, 8, 128, 128, name="forward_bf16"),
        # prefill of ragged prompts in one packed batch, the gated delta rule's ablation (constant lambda, no decay)
        _case("forward", 9, 6007, 8, 64, 128, decay="none", lam=0.5, state=False, packed=True,
              name="forward_packed_const_lam"),
        # one long document over few heads
        _case("segmented", 1, 65536, 16, 128, 128, name="long_bf16"),
        # the training step that the benchmark reports
        _case("train", 4, 4096, 16, 128, 128, name="train_bf16"),
        # training in fp32 on sequences that no tile divides, decay that lasts over many chunks
        _case("autograd", 2, 1003, 6, 64, 128, "f32", decay="slow", name="train_ragged_f32"),
        # training on a packed batch of documents, wide value heads
        _case("autograd", 24, 32768, 32, 128, 256, state=False, packed=True, name="train_packed_bf16"),
        # the token mixer of a block with its projections and gates
        _case("layer", 4, 4096, 16, 128, 128, state=False, d_model=2048, name="layer_bf16"),
        # one decode step of a serving batch
        _case("decode", 64, 1, 16, 128, 128, name="decode_batch"),
        # one decode step of a single request
        _case("decode", 1, 1, 16, 128, 128, name="decode_single"),
        # a few new tokens of continuing sequences (a chat turn, speculated tokens)
        _case("recurrent", 64, 16, 16, 128, 128, name="recurrent_bf16"),
        # ... and their gradients
        _case("rec_train", 64, 16, 16, 128, 128, name="recurrent_train_bf16"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["forward", "forward", "segmented", "train", "autograd", "autograd", "layer", "decode",
                     "recurrent", "rec_train"])
    heads = rng.choice([1, 2, 3, 4, 6, 8, 12, 16, 24, 32])
    dk, dv = rng.choice([64, 128, 128]), rng.choice([64, 128, 128, 256])
    dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
    if dtype == "f32" and op not in ("decode", "recurrent", "rec_train"):
        dk = 64                                 # the chunk kernels' fp32 head size
    decay = rng.choice(["fast", "fast", "slow", "none"])
    # a constant lambda's own gradient is one number, a sum with cancellation: no case of 16-bit training returns it
    lam = "token" if op == "train" else rng.choice(["token", "token", "token", 0.0, 0.2, 0.8, 1.0])
    state = rng.random() < 0.5
    packed = False
    d_model = 0
    if op in ("forward", "train", "autograd"):
        packed = rng.random() < 0.4
        # at most the packed training case's token-heads, counted by their values
        most = 32768 * 32 * 256 // (heads * dv)
        tokens = _log_int(rng, 100, min(40000, most))
        if packed:
            batch = rng.randint(1, max(1, min(40, tokens // 40)))
        else:
            batch = min(rng.choice([1, 2, 3, 4, 8]), tokens // 60)
            tokens = max(1, tokens // batch)
    elif op == "segmented":
        heads = rng.choice([1, 2, 4, 8, 16])
        dv = min(dv, 128)
        batch, tokens = 1, _log_int(rng, 4000, 65536)
    elif op == "layer":
        heads = rng.choice([2, 4, 8, 16])
        d_model = rng.choice([256, 512, 1024, 2048])
        dtype, state = "bf16", False
        dv = min(dv, 128)
        batch, tokens = rng.randint(1, 4), _log_int(rng, 100, 4096)
    elif op == "decode":
        batch, tokens = _log_int(rng, 1, 128), 1
    else:
        packed = rng.random() < 0.3
        batch, tokens = _log_int(rng, 1, 64), _log_int(rng, 1, 64)
        heads = min(heads, 16)
        if packed:
            tokens *= batch
    return _case(op, batch, tokens, heads, dk, dv, dtype, decay, lam, state, packed, d_model)


# ------------------------------------------------------------------ inputs
def _lengths(case):
    """Sequence lengths of a packed batch: a spread of short and long documents that depends on the sizes alone."""
    n, total = case["batch"], case["tokens"]
    r = random.Random(1000003 * n + total)
    w = [math.exp(r.gauss(0.0, 1.0)) for _ in range(n)]
    cuts = [0]
    for i in range(n):
        cuts.append(min(total, max(cuts[-1] + (total >= n), round(total * sum(w[:i + 1]) / sum(w)))))
    cuts[-1] = total
    return [b - a for a, b in zip(cuts, cuts[1:])]


def _inputs(case, seed):
    """The tensors of one call, from the seed alone; activations [B, T, H, D] ([1, sum T, H, D] packed)."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    B, T, H, dk, dv = (case[k] for k in ("batch", "tokens", "heads", "dk", "dv"))
    td = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    n_seqs = B
    if case["packed"]:
        B = 1

    def normal(*shape):
        return torch.randn(shape, device="cuda", generator=g)

    x = dict(q=F.normalize(normal(B, T, H, dk), dim=-1).to(td), k=F.normalize(normal(B, T, H, dk), dim=-1).to(td),
             v=normal(B, T, H, dv).to(td), beta=torch.sigmoid(normal(B, T, H)))
    x["lam"] = torch.sigmoid(normal(B, T, H)) if case["lam"] == "token" else float(case["lam"])
    x["log_alpha"] = None
    if case["decay"] != "none":
        x["log_alpha"] = F.logsigmoid(normal(B, T, H) + (4.0 if case["decay"] == "slow" else 0.0))
    x["initial_state"] = 0.02 * normal(n_seqs, H, dv, dk) if case["state"] else None
    x["d_o"] = normal(B, T, H, dv).to(td)
    x["cu_seqlens"] = None
    if case["packed"]:
        lens = _lengths(case)
        x["cu_seqlens"] = torch.tensor([sum(lens[:i]) for i in range(len(lens) + 1)], dtype=torch.int32, device="cuda")
    return x


def _layer_inputs(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    m = qlayer.QDeltaLayer(case["d_model"], case["heads"], case["dk"], case["dv"], use_decay=case["decay"] != "none",
                           fixed_lambda=None if case["lam"] == "token" else case["lam"]).cuda()
    with torch.no_grad():
        for lin in (m.w_qkv, m.w_gates, m.w_out):
            lin.weight.copy_(torch.randn(lin.weight.shape, device="cuda", generator=g) / math.sqrt(lin.in_features))
    m = m.to(torch.bfloat16)
    shape = (case["batch"], case["tokens"], case["d_model"])
    h = torch.randn(shape, device="cuda", generator=g).to(torch.bfloat16).requires_grad_()
    dy = torch.randn(shape, device="cuda", generator=g).to(torch.bfloat16)
    return m, h, dy


ARGS = ("q", "k", "v", "beta", "lam", "log_alpha", "initial_state")


def prepare(case, seed):
    op = case["op"]
    if op == "layer":
        m, h, dy = _layer_inputs(case, seed)
        return dict(op=op, m=m, h=h, dy=dy)
    x = _inputs(case, seed)
    s = dict(op=op, x=x, args=tuple(x[a] for a in ARGS), cu=x["cu_seqlens"])
    B, T, H, dk, dv = (case[k] for k in ("batch", "tokens", "heads", "dk", "dv"))
    if op == "train":
        n_seqs = B if case["packed"] else 0
        dt = qdelta.QDELTA_BF16 if case["dtype"] == "bf16" else qdelta.QDELTA_F32
        for key, is_bwd in (("wsf", False), ("wsb", True)):
            n = qdelta.workspace_bytes(1 if case["packed"] else B, T, H, dk, dv, dt, n_seqs, is_bwd)
            s[key] = torch.empty(n, dtype=torch.uint8, device="cuda")
    elif op == "autograd":
        s["leaves"] = [t.requires_grad_() for t in s["args"] if isinstance(t, torch.Tensor)]
    elif op == "decode":
        # [N, H, D] tensors of one token and the running state
        for name in ("q", "k", "v", "beta", "lam", "log_alpha"):
            if isinstance(x[name], torch.Tensor):
                x[name] = x[name][:, 0].contiguous()
        s["args"] = tuple(x[a] for a in ARGS[:-1])
        s["state"] = x["initial_state"] if x["initial_state"] is not None else torch.zeros((B, H, dv, dk), device="cuda")
        s["out"] = torch.empty((B, H, dv), dtype=x["q"].dtype, device="cuda")
    return s


def run(s):
    op = s["op"]
    if op == "forward":
        o, final, _ = qdelta.chunk_fwd(*s["args"], cu_seqlens=s["cu"])
        return {"o": o, "final_state": final}
    if op == "segmented":
        o, final, _ = qdelta.chunk_fwd_segmented(*s["args"])
        return {"o": o, "final_state": final}
    if op == "train":
        o, final, saved = qdelta.chunk_fwd(*s["args"], cu_seqlens=s["cu"], save_states=True, workspace=s["wsf"])
        g = qdelta.chunk_bwd(*s["args"], saved, s["x"]["d_o"], cu_seqlens=s["cu"], workspace=s["wsb"])
        return {"o": o, "final_state": final, "grads": g}
    if op == "autograd":
        x = s["x"]
        for t in s["leaves"]:
            t.grad = None
        o, final = qlayer.qdelta_chunk(*s["args"], cu_seqlens=s["cu"])
        o.backward(x["d_o"])
        return {"o": o, "final_state": final,
                "grads": {a: x[a].grad for a in ARGS if isinstance(x[a], torch.Tensor)}}
    if op == "layer":
        m, h = s["m"], s["h"]
        m.zero_grad(set_to_none=True)
        h.grad = None
        y = m(h)
        y.backward(s["dy"])
        # the lambda bias is one number, a sum with cancellation: it goes with the gate weights' gradients
        gates = [m.w_gates.weight.grad.reshape(-1)]
        if m.fixed_lambda is None:
            gates.append(m.lambda_bias.grad.reshape(1))
        return {"y": y, "dh": h.grad, "qkv": m.w_qkv.weight.grad, "gates": torch.cat(gates), "out": m.w_out.weight.grad}
    if op == "decode":
        o = qdelta.recurrent_step(*s["args"], s["state"], out=s["out"])
        return {"o": o, "state": s["state"]}
    o, final = qdelta.recurrent_fwd(*s["args"], cu_seqlens=s["cu"])
    if op == "recurrent":
        return {"o": o, "final_state": final}
    g = qdelta.recurrent_bwd(*s["args"], s["x"]["d_o"], cu_seqlens=s["cu"])
    return {"o": o, "final_state": final, "grads": g}


# ------------------------------------------------------------------ work and tolerance
def work(case):
    """Inputs read once and outputs written once (entry states, workspaces and saved contexts do not count); the
    recurrence's own operations: three Dk x Dv products forward, seven more (adjoint and gradients) backward."""
    B, T, H, dk, dv = (case[k] for k in ("batch", "tokens", "heads", "dk", "dv"))
    e = 2 if case["dtype"] == "bf16" else 4
    op = case["op"]
    tokens = T if case["packed"] else B * T
    train = op in ("train", "autograd", "rec_train", "layer")
    gates = 4 * (1 + (case["lam"] == "token") + (case["decay"] != "none"))
    per = (2 * dk + dv) * e + gates + dv * e                        # q, k, v, gates -> o
    flops = 6 * dk * dv
    if train:
        per += (2 * dk + dv) * e * 2 + dv * e + 2 * gates           # q, k, v, gates, dO -> their gradients
        flops += 14 * dk * dv
    states = 1 + bool(case["state"]) + (train and bool(case["state"]))
    if op == "decode":
        states = 2
    w = {"bytes": tokens * H * per + B * H * dk * dv * 4 * states, "flops": tokens * H * flops}
    if op == "layer":
        d = case["d_model"]
        n_gates = 1 + (case["lam"] == "token") + (case["decay"] != "none")
        weights = d * H * (2 * dk + dv + n_gates + dv)
        # h, dy, weights -> y, dh, weight gradients; q, k, v and their gradients stay inside
        w["bytes"] = 2 * (4 * tokens * d + 3 * weights)
        w["flops"] += 3 * 2 * tokens * weights
    return w


def tolerance(case):
    """About four times the error measured against exact() (per output at most: fp32 9e-7; bf16 results of fp32 state
    arithmetic 1.7e-3; bf16 chunk operands 3.7e-3, 6e-3 without decay; the layer 5.5e-3)."""
    if case["dtype"] == "f32":
        return {"rel": 1e-5}
    if case["op"] in ("decode", "recurrent", "rec_train"):
        return {"rel": 7e-3}
    if case["op"] == "layer" or case["decay"] == "none":
        return {"rel": 2.4e-2}
    return {"rel": 1.5e-2}


# ------------------------------------------------------------------ reference in 64 bits
def _reference(q, k, v, beta, lam, log_alpha, S0):
    """The recurrence S_t = a_t S_{t-1} (I - b_t x_t k_t^T) + b_t v_t k_t^T, o_t = S_t q_t, x = k + lambda q, in float64
    over [N, T, H, D], by the WY form of chunks (exact in real arithmetic).  Returns o and the final state."""
    N, T, H, dk = q.shape
    dv = v.shape[-1]
    nc = max(1, -(-T // CHUNK))
    pad = nc * CHUNK - T

    def units(x):       # [N, T, H, D] -> [N H, chunks, C, D]; the zero rows past the end change nothing
        x = F.pad(x.transpose(1, 2), (0, 0, 0, pad))
        return x.reshape(N * H, nc, CHUNK, x.shape[-1])

    def units_gate(x):  # [N, T, H] -> [N H, chunks, C]
        return F.pad(x.transpose(1, 2), (0, pad)).reshape(N * H, nc, CHUNK)

    if log_alpha is None:
        log_alpha = torch.zeros_like(beta)
    Q, K, V = units(q), units(k), units(v)
    be, lm, b = units_gate(beta), units_gate(lam), units_gate(log_alpha).cumsum(-1)
    low = torch.ones(CHUNK, CHUNK, dtype=torch.bool, device=q.device).tril()
    gam = torch.where(low, b[..., :, None] - b[..., None, :], torch.full((), -math.inf, dtype=b.dtype, device=b.device)).exp()
    X = K + lm[..., None] * Q
    A = (be[..., None] * gam * (X @ K.transpose(-1, -2).contiguous())).tril(-1)
    eye = torch.eye(CHUNK, dtype=b.dtype, device=b.device)
    Tm = torch.linalg.solve_triangular(eye + A, torch.diag_embed(be), upper=False, unitriangular=True)
    g = b.exp()
    U, W = Tm @ V, Tm @ (g[..., None] * X)
    Pm = gam * (Q @ K.transpose(-1, -2).contiguous())
    Qg, gC = g[..., None] * Q, g[..., -1]
    Kb = (b[..., -1:] - b).exp()[..., None] * K
    S = S0.reshape(N * H, dv, dk).transpose(1, 2) if S0 is not None else torch.zeros(N * H, dk, dv, dtype=b.dtype, device=b.device)
    outs = []
    for c in range(nc):         # S here is [Dk, Dv]
        D = U[:, c] - W[:, c] @ S
        outs.append(Qg[:, c] @ S + Pm[:, c] @ D)
        S = gC[:, c, None, None] * S + Kb[:, c].transpose(1, 2) @ D
    o = torch.stack(outs, 1).reshape(N, H, nc * CHUNK, dv)[:, :, :T].transpose(1, 2)
    return o, S.transpose(1, 2).reshape(N, H, dv, dk)


def exact(case, seed):
    op = case["op"]
    if op == "layer":
        return _exact_layer(case, seed)
    x = _inputs(case, seed)
    grads = op in ("train", "autograd", "rec_train")
    f64 = {a: x[a].double() for a in ARGS if isinstance(x[a], torch.Tensor)}
    lam = f64.get("lam")
    lam_c = None
    if lam is None:
        lam_c = torch.full((), float(case["lam"]), dtype=torch.float64, device="cuda")
    if case["packed"]:
        ends = x["cu_seqlens"].tolist()
        seqs = [(slice(0, 1), slice(a, b), i) for i, (a, b) in enumerate(zip(ends, ends[1:]))]
    else:
        seqs = [(slice(None), slice(None), slice(None))]
    out = {"o": torch.empty_like(x["v"], dtype=torch.float64)}
    got = {a: torch.zeros_like(t) for a, t in f64.items()} if grads else {}
    finals, dlam_c = [], 0.0
    for rows, toks, n in seqs:
        S0 = f64.get("initial_state")
        if S0 is not None and case["packed"]:
            S0 = S0[n:n + 1]
        part = {a: f64[a][rows, toks] for a in ("q", "k", "v", "beta", "lam", "log_alpha") if a in f64}
        if S0 is not None:
            part["initial_state"] = S0
        part = {a: t.detach().clone().requires_grad_(grads) for a, t in part.items()}
        lc = None if lam_c is None else lam_c.clone().requires_grad_(grads)
        with torch.set_grad_enabled(grads):
            lam_t = part["lam"] if lam_c is None else lc * torch.ones_like(part["beta"])
            o, Sf = _reference(part["q"], part["k"], part["v"], part["beta"], lam_t, part.get("log_alpha"),
                               part.get("initial_state"))
        if grads:
            names = list(part)
            leaves = [part[a] for a in names] + ([lc] if lc is not None else [])
            gs = torch.autograd.grad(o, leaves, x["d_o"][rows, toks].double())
            for a, gr in zip(names, gs):
                if a == "initial_state":
                    got[a][n if not case["packed"] else slice(n, n + 1)] = gr
                else:
                    got[a][rows, toks] = gr
            if lc is not None:
                dlam_c = dlam_c + gs[-1]
        out["o"][rows, toks] = o.detach()
        finals.append(Sf.detach())
    final = torch.cat(finals)
    if op == "decode":
        return {"o": out["o"][:, 0], "state": final}
    out["final_state"] = final
    if op == "autograd":
        out["grads"] = got
    elif grads:
        out["grads"] = {"dq": got["q"], "dk": got["k"], "dv": got["v"], "dbeta": got["beta"],
                        "dlam": got["lam"] if lam is not None else dlam_c, "dlog_alpha": got.get("log_alpha"),
                        "d_initial_state": got.get("initial_state")}
    return out


def _exact_layer(case, seed):
    m, h, dy = _layer_inputs(case, seed)
    H, dk, dv = case["heads"], case["dk"], case["dv"]
    wq, wg, wo = (lin.weight.detach().double().requires_grad_() for lin in (m.w_qkv, m.w_gates, m.w_out))
    bias = m.lambda_bias.detach().double().requires_grad_() if m.fixed_lambda is None else None
    h = h.detach().double().requires_grad_()
    B, T, _ = h.shape
    q, k, v = (h @ wq.T).view(B, T, H, 2 * dk + dv).split([dk, dk, dv], dim=-1)
    g = (h @ wg.T).split(H, dim=-1)
    beta, at = torch.sigmoid(g[0]), 1
    if bias is not None:
        lam, at = torch.sigmoid(g[1] + bias), 2
    else:
        lam = torch.full_like(beta, m.fixed_lambda)
    la = F.logsigmoid(g[at]) if m.use_decay else None
    o, _ = _reference(F.normalize(q, dim=-1), F.normalize(k, dim=-1), v, beta, lam, la, None)
    y = o.reshape(B, T, H * dv) @ wo.T
    leaves = [h, wq, wg, wo] + ([bias] if bias is not None else [])
    gs = torch.autograd.grad(y, leaves, dy.double())
    gates = [gs[2].reshape(-1)] + ([gs[4].reshape(1)] if bias is not None else [])
    return {"y": y.detach(), "dh": gs[0], "qkv": gs[1], "gates": torch.cat(gates), "out": gs[3]}
