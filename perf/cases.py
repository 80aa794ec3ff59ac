"""Performance cases of the alpha-entmax attention library.

Every case is one call, or one forward and backward, through the Python entry
points that a user's program calls, on inputs of the recipe of `synth`: Gaussian
queries times a temperature c (the larger c, the sparser the probabilities),
Gaussian keys, values and output gradients.

ops
    infer   forward(need_bwd=False) with the residual buffers, the output and
            the workspace kept from call to call, as a serving loop does
    step    forward and backward of the masked path, as a training step does
    dense   forward_dense and backward_dense (the no-mask mode)
    rows    rows_forward and rows_backward on a materialized score matrix
"""
import math

import torch

import paper_2502_12082_amd as ea


def _attn(name, op, B, H, n, d, dtype, causal, alpha, c):
    return {"name": name, "op": op, "B": B, "H": H, "n": n, "d": d, "dtype": dtype,
            "causal": causal, "alpha": alpha, "c": c}


def _rows(name, rows, n, dtype, alpha, sigma):
    return {"name": name, "op": "rows", "rows": rows, "n": n, "dtype": dtype, "alpha": alpha,
            "sigma": sigma}


def listed():
    return [
        # one short sequence, one head, fp32: launches and host time
        _attn("tiny_infer_f32", "infer", 1, 1, 256, 64, "f32", False, 1.5, 1.0),
        # a bidirectional encoder layer at inference (heads of a base model)
        _attn("encoder_infer", "infer", 8, 12, 1024, 64, "bf16", False, 1.5, 1.0),
        # fine-tuning such a layer on sequences of a ragged length
        _attn("encoder_step_ragged", "step", 4, 12, 777, 64, "bf16", False, 1.5, 4.0),
        # a causal decoder layer's training step
        _attn("decoder_step", "step", 4, 12, 4096, 64, "bf16", True, 1.5, 8.0),
        # the efficiency sweep's main point: long rows, head dimension 128
        _attn("sweep_step_c1", "step", 1, 16, 8192, 128, "bf16", False, 1.5, 1.0),
        # the same with few zeros (a quarter of the temperature)
        _attn("sweep_step_low_sparsity", "step", 1, 16, 8192, 128, "bf16", False, 1.5, 0.25),
        # alpha = 1.25: denser rows than alpha = 1.5 at the same temperature
        _attn("sweep_step_a125", "step", 1, 16, 4096, 128, "bf16", True, 1.25, 2.0),
        # sparsemax on a ragged causal sequence
        _attn("sparsemax_step_ragged", "step", 2, 8, 3001, 128, "bf16", True, 2.0, 2.0),
        # long context, few heads, causal, very sparse
        _attn("long_step", "step", 1, 8, 32768, 64, "bf16", True, 1.5, 16.0),
        # fp32 inputs and a general alpha (gradient checks, alpha annealing)
        _attn("f32_step_general", "step", 2, 4, 1025, 64, "f32", True, 1.7, 2.0),
        # the no-mask mode's training step
        _attn("dense_step", "dense", 1, 16, 4096, 128, "bf16", False, 1.5, 1.0),
        # the row-wise kernel on score matrices: long aligned rows
        _rows("rows_8192", 8192, 8192, "f32", 1.5, 1.0),
    ]


def draw(rng):
    """Another case of the ranges of the listed ones."""
    def logint(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    def logreal(lo, hi):
        return round(math.exp(rng.uniform(math.log(lo), math.log(hi))), 3)

    if rng.random() < 0.2:
        n = logint(100, 32768)
        if rng.random() < 0.5:
            n = max(8, n // 8 * 8)
        rows = max(1, min(logint(64, 65536), (1 << 26) // n))
        return {"op": "rows", "rows": rows, "n": n, "dtype": rng.choice(["f32", "bf16"]),
                "alpha": rng.choice([1.25, 1.5, 1.5, 1.6, 2.0]), "sigma": logreal(0.3, 6.0)}
    op = rng.choice(["infer", "step", "step", "step", "dense"])
    f32 = rng.random() < 0.2
    d = rng.choice([64, 128])
    n = logint(64, 2048 if f32 else 16384)
    if rng.random() < 0.5:
        n = max(64, n // 64 * 64)
    # at most the largest listed case's products, at fp32's sixteenth of the rate
    budget = 16 * 8192 * 8192 * 128 // (2 * (16 if f32 else 1))
    heads = max(1, min(logint(1, 96), budget // (n * n * d)))
    B = rng.choice([b for b in (1, 2, 4, 8) if b <= heads])
    return {"op": op, "B": B, "H": max(1, heads // B), "n": n, "d": d,
            "dtype": "f32" if f32 else "bf16", "causal": rng.random() < 0.5,
            "alpha": rng.choice([1.25, 1.5, 1.5, 1.5, 1.5, 1.75, 2.0]),
            "c": logreal(0.25, 16.0)}


def _inputs(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16

    def normal(*shape, scale=1.0, dtype=dt):
        return torch.randn(*shape, generator=g, device="cuda").mul_(scale).to(dtype)

    if case["op"] == "rows":
        shape = (case["rows"], case["n"])
        return {"s": normal(*shape, scale=case["sigma"]), "dp": normal(*shape, dtype=torch.float32)}
    shape = (case["B"], case["H"], case["n"], case["d"])
    x = {"q": normal(*shape, scale=case["c"]), "k": normal(*shape), "v": normal(*shape)}
    if case["op"] != "infer":
        x["do"] = normal(*shape)
    return x


def prepare(case, seed):
    state = {"case": case, **_inputs(case, seed)}
    if case["op"] == "infer":
        q = state["q"]
        shape = ea.make_shape(q)
        params = ea.make_params(case["alpha"], None, case["causal"], False, head_dim=case["d"])
        state["res"] = ea.Residuals(shape, params, q.device)
        state["out"] = torch.empty_like(q)
        state["ws"] = ea.forward_workspace(state["res"], q.device)
    return state


def run(state):
    case = state["case"]
    alpha = case["alpha"]
    if case["op"] == "rows":
        p, tau = ea.rows_forward(state["s"], alpha=alpha)
        ds = ea.rows_backward(state["s"], tau, state["dp"], alpha=alpha)
        return {"p": p, "tau": tau, "ds": ds}
    q, k, v = state["q"], state["k"], state["v"]
    causal = case["causal"]
    if case["op"] == "infer":
        o, res = ea.forward(q, k, v, alpha=alpha, causal=causal, need_bwd=False,
                            out=state["out"], res=state["res"], workspace=state["ws"])
        return {"o": o, "tau": res.tau}
    if case["op"] == "dense":
        o, tau, o2, tau_lo = ea.forward_dense(q, k, v, alpha=alpha, causal=causal)
        dq, dk, dv = ea.backward_dense(q, k, v, state["do"], tau, o2, alpha=alpha, causal=causal,
                                       tau_lo=tau_lo)
        return {"o": o, "tau": tau, "dq": dq, "dk": dk, "dv": dv}
    o, res = ea.forward(q, k, v, alpha=alpha, causal=causal)
    dq, dk, dv = ea.backward(q, k, v, state["do"], res)
    return {"o": o, "tau": res.tau, "dq": dq, "dk": dk, "dv": dv}


def work(case):
    """The inputs read once and the outputs written once; the products of the
    path over every valid pair (the score product once a pass over the data:
    2 products of 2 d operations a pair forward, 5 more backward), since how
    many pairs have a nonzero probability depends on the data."""
    e = 4 if case["dtype"] == "f32" else 2
    if case["op"] == "rows":
        m = case["rows"] * case["n"]
        # s and p; s, dp and ds; a few operations an element
        return {"bytes": m * (e + 4) + m * (e + 8) + 8 * case["rows"], "flops": 40 * m}
    bh, n, d = case["B"] * case["H"], case["n"], case["d"]
    m = bh * n * d
    pairs = bh * (n * (n + 1) // 2 if case["causal"] else n * n)
    if case["op"] == "infer":
        return {"bytes": 4 * m * e + 4 * bh * n, "flops": 4 * d * pairs}
    return {"bytes": 4 * m * e + 4 * bh * n + 4 * m * e + 3 * 4 * m, "flops": 14 * d * pairs}


def tolerance(case):
    """About four times the errors against exact(): with bf16 inputs 1.7e-3,
    the rounding of O and of the P operand of dV; in fp32 1.5e-6, more where
    scores are large (the rounding of x - tau)."""
    if case["op"] == "rows" or case["dtype"] == "f32":
        return {"rel": 2e-5}
    return {"rel": 7e-3}


# ------------------------------------------------------------ in 64 bits

def _f32(x):
    return float(torch.tensor(x, dtype=torch.float32))


def _threshold(x, gamma):
    """Root of sum [x - tau]_+^gamma = 1 for each row of x (-inf: no entry)."""
    hi = x.amax(dim=-1, keepdim=True)
    tau = hi - 1.0
    if gamma >= 1.0:  # f convex and decreasing: Newton's steps from below stay below the root
        for _ in range(100):
            z = (x - tau).clamp_(min=0.0)
            if gamma == 1.0:
                f, g = z.sum(-1, keepdim=True), (z > 0).sum(-1, keepdim=True).to(z.dtype)
            else:
                u = z if gamma == 2.0 else z.pow(gamma - 1.0)
                f, g = (u * z).sum(-1, keepdim=True), gamma * u.sum(-1, keepdim=True)
            step = ((f - 1.0) / g).clamp(min=0.0)
            tau = tau + step
            if float(step.max()) < 1e-14:
                break
        return tau
    lo = tau
    for _ in range(60):
        mid = 0.5 * (lo + hi)
        below = (x - mid).clamp_(min=0.0).pow(gamma).sum(-1, keepdim=True) >= 1.0
        lo, hi = torch.where(below, mid, lo), torch.where(below, hi, mid)
    return 0.5 * (lo + hi)


def _maps(x, tau, gamma):
    z = (x - tau).clamp_(min=0.0)
    if gamma == 1.0:
        return z, (z > 0).to(z.dtype)
    u = z.clone() if gamma == 2.0 else torch.where(z > 0, z.pow(gamma - 1.0), torch.zeros_like(z))
    return u * z, u


def exact(case, seed):
    x = _inputs(case, seed)
    alpha = _f32(case["alpha"])
    gamma = 1.0 / (alpha - 1.0)
    if case["op"] == "rows":
        if case["rows"] * case["n"] > 1 << 27:
            return None
        p, tau, ds = [], [], []
        step = max(1, (1 << 25) // case["n"])
        for r in range(0, case["rows"], step):
            y = x["s"][r:r + step].double() * (alpha - 1.0)
            t = _threshold(y, gamma)
            pr, u = _maps(y, t, gamma)
            dp = x["dp"][r:r + step].double()
            ds.append(u * (dp - (u * dp).sum(-1, keepdim=True) / u.sum(-1, keepdim=True)))
            p.append(pr)
            tau.append(t[:, 0])
        return {"p": torch.cat(p), "tau": torch.cat(tau), "ds": torch.cat(ds)}
    B, H, n, d = case["B"], case["H"], case["n"], case["d"]
    if B * H * n * n * d > 1 << 40:
        return None
    scale = _f32(d ** -0.5)
    c = (alpha - 1.0) * scale
    q, k, v = (x[s].reshape(B * H, n, d) for s in ("q", "k", "v"))
    do = x["do"].reshape(B * H, n, d) if "do" in x else None

    def out(*shape):
        return torch.zeros(*shape, dtype=torch.float64, device="cuda")

    o, tau = out(B * H, n, d), out(B * H, n)
    dq, dk, dv = (out(B * H, n, d) if do is not None else None for _ in range(3))
    step = max(64, min(n, (1 << 25) // n))
    for b in range(B * H):
        kd, vd = k[b].double(), v[b].double()
        for r in range(0, n, step):
            e = min(n, r + step)
            m = e if case["causal"] else n
            qr = q[b, r:e].double()
            s = c * (qr @ kd[:m].T)
            if case["causal"]:
                i = torch.arange(r, e, device="cuda")[:, None]
                s.masked_fill_(torch.arange(m, device="cuda")[None, :] > i, -math.inf)
            t = _threshold(s, gamma)
            p, u = _maps(s, t, gamma)
            o[b, r:e] = p @ vd[:m]
            tau[b, r:e] = t[:, 0]
            if do is not None:
                dor = do[b, r:e].double()
                dp = dor @ vd[:m].T
                ds = u * (dp - (u * dp).sum(-1, keepdim=True) / u.sum(-1, keepdim=True))
                dq[b, r:e] = scale * (ds @ kd[:m])
                dk[b, :m] += scale * (ds.T @ qr)
                dv[b, :m] += p.T @ dor
    shape = (B, H, n, d)
    if case["op"] == "infer":
        return {"o": o.reshape(shape), "tau": tau}
    return {"o": o.reshape(shape), "tau": tau, "dq": dq.reshape(shape), "dk": dk.reshape(shape),
            "dv": dv.reshape(shape)}
