"""The work that users of this framework have it do, as measurable cases.

Each listed case is one call (a training step: two) through the package's
public entry points at a size that a serving or training program uses; the
head sizes 8 to 64, the truncation P = 4 and the headline shapes are those of
the repository's benchmark.  ``draw`` spreads further cases over the same ranges.

Inputs.  Queries and keys are N(0, sigma^2) with sigma^2 = 0.5 (0.25 at
P = 2), values and gradients N(0, 1): scores q.k / sqrt(d) of about one half,
the range in which a few terms of the series stand for the exponential.  At an
even P the truncated series has a real root (s = -1 at P = 2, -1.596 at P = 4),
and scores of unit variance give rows whose denominator cancels, which say
nothing about an implementation.
"""
from __future__ import annotations

import math
from itertools import combinations_with_replacement

import torch

import paper_2602_00294_amd as sata

DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
SIZE = {"bf16": 2, "f32": 4}
CONTEXT = 64  # tokens summed into a decode case's state before the call


def listed():
    return [
        # one sequence being generated by one layer: launch latency and one head per workgroup
        dict(name="decode_one_sequence", op="decode", B=1, H=32, dk=32, dv=32, P=4, dtype="bf16"),
        # the benchmark's decode: a batch of 8 sequences, 221 MB of state read and written per step
        dict(name="decode_batch", op="decode", B=8, H=32, dk=32, dv=32, P=4, dtype="bf16"),
        # the same batch with 8 key/value heads that serve 4 query heads each
        dict(name="decode_grouped", op="decode_grouped", B=8, H=8, G=4, dk=32, dv=32, P=4, dtype="bf16"),
        # a short prompt of odd sizes (d_k is not d_v, ragged length): latency, little to fill the chip with
        dict(name="prefill_short_ragged", op="prefill", B=1, H=8, n=1000, dk=24, dv=40, P=3, dtype="bf16", state=True),
        # the benchmark's prefill, with the state that decoding goes on from
        dict(name="prefill_batch", op="prefill", B=8, H=32, n=8192, dk=32, dv=32, P=4, dtype="bf16", state=True),
        # many short heads (d = 16), the benchmark's second decode workload's prompt
        dict(name="prefill_d16", op="prefill", B=64, H=32, n=2048, dk=16, dv=16, P=4, dtype="bf16", state=True),
        # large heads (d = 64): 12.5 MB of state per head
        dict(name="prefill_d64", op="prefill", B=2, H=8, n=4096, dk=64, dv=64, P=4, dtype="bf16", state=True),
        # a long float32 sequence, the benchmark's sweep over P at its middle
        dict(name="prefill_f32_long", op="prefill", B=1, H=64, n=65536, dk=16, dv=16, P=4, dtype="f32", state=True),
        # a prompt with shared key/value heads
        dict(name="prefill_grouped", op="prefill_grouped", B=2, H=8, G=4, n=4096, dk=32, dv=32, P=4, dtype="bf16",
             state=True),
        # one layer's training step: forward without a state, then the gradients (the benchmark's backward)
        dict(name="train_step", op="train", B=8, H=32, n=2048, dk=32, dv=32, P=4, dtype="bf16"),
        # gradients in float32 at odd sizes
        dict(name="backward_f32_ragged", op="backward", B=2, H=8, n=777, dk=16, dv=20, P=3, dtype="f32"),
        # features as a tensor, for programs that do their own contraction (the benchmark's feature map)
        dict(name="feature_map", op="feature_map", rows=65536, dk=32, P=4, dtype="bf16"),
    ]


# ------------------------------------------------------------------ drawn cases

def _log_int(rng, low, high):
    return int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))


def _head_size(rng):
    return rng.choice([8, 16, 24, 32, 32, 48, 64, rng.randint(8, 64)])


def draw(rng):
    """One case of the listed ones' ranges; its scan work is at most the largest listed case's."""
    op = rng.choice(["decode", "decode", "decode_grouped", "prefill", "prefill", "prefill", "prefill_grouped", "train",
                     "backward", "feature_map"])
    dtype = rng.choice(["bf16", "bf16", "f32"])
    while True:
        dk = _head_size(rng)
        dv = dk if rng.random() < 0.7 else _head_size(rng)
        P = rng.choice([2, 3, 4, 4, 4, 5])
        D = math.comb(dk + P - 1, P - 1)
        if D > 50_000:
            continue
        if op == "feature_map":
            rows = _log_int(rng, 64, 500_000)
            if rows * D > 450_000_000:
                continue
            return dict(op=op, rows=rows, dk=dk, P=P, dtype=dtype)
        B, H = _log_int(rng, 1, 32), rng.choice([1, 2, 4, 8, 8, 16, 32, rng.randint(1, 32)])
        if op in ("decode", "decode_grouped"):
            if not 1_000 <= B * H * D * (dv + 1) <= 110_000_000:
                continue
            case = dict(op=op, B=B, H=H, dk=dk, dv=dv, P=P, dtype=dtype)
            if op == "decode_grouped":
                case["G"] = rng.choice([2, 4, 8])
            return case
        n = _log_int(rng, 64, 16384)
        G = rng.choice([2, 4, 8]) if op == "prefill_grouped" else 1
        scan = 4.0 * B * H * G * n * D * (dv + 1)
        limit = {"train": 4e11, "backward": 4e11}.get(op, 1.5e12 if dtype == "bf16" else 2.5e11)
        if scan > limit or B * H * G * n * max(dk, dv) > 100_000_000 or B * H * G * float(n) * n > 3e10:
            continue
        case = dict(op=op, B=B, H=H, n=n, dk=dk, dv=dv, P=P, dtype=dtype)
        if op == "prefill_grouped":
            case["G"] = G
        if op in ("prefill", "prefill_grouped"):
            case["state"] = rng.random() < 0.75
        return case


# ------------------------------------------------------------------ inputs and the calls

def _monomials(d, P):
    """(index tuples padded with d, weights) of all features in the library's order, on the GPU in 64 bits."""
    rows, weights = [], []
    for p in range(P):
        for t in combinations_with_replacement(range(d), p):
            mult = 1.0
            for c in set(t):
                mult *= math.factorial(t.count(c))
            rows.append(t + (d,) * (P - 1 - p))
            weights.append(1.0 / (d ** (p / 4.0) * math.sqrt(mult)))
    index = torch.tensor(rows, dtype=torch.int64, device="cuda").reshape(len(rows), P - 1)
    return index, torch.tensor(weights, dtype=torch.float64, device="cuda")


def _features(x, monomials, dtype):
    """phi(x) of x [..., d] in the given type, by products of gathered coordinates."""
    index, weights = monomials
    x = x.to(dtype)
    x = torch.cat([x, torch.ones_like(x[..., :1])], dim=-1)
    out = weights.to(dtype).expand(*x.shape[:-1], -1)
    for j in range(index.shape[1]):
        out = out * x[..., index[:, j]]
    return out


def _inputs(case, seed):
    """The call's tensors, from the seed alone."""
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 7919 + 13)
    dt = DTYPES[case["dtype"]]
    scale = math.sqrt(0.25 if case["P"] == 2 else 0.5)

    def normal(*shape, s=1.0):
        return (torch.randn(*shape, generator=g, device="cuda", dtype=torch.float32) * s).to(dt)

    op, dk = case["op"], case["dk"]
    if op == "feature_map":
        return dict(x=normal(case["rows"], dk, s=scale))
    B, H, dv, G = case["B"], case["H"], case["dv"], case.get("G", 1)
    if op in ("decode", "decode_grouped"):
        t = dict(q=normal(B, H * G, dk, s=scale), k=normal(B, H, dk, s=scale), v=normal(B, H, dv))
        # a state that has seen CONTEXT tokens
        mono = _monomials(dk, case["P"])
        S = torch.empty(B, H, mono[0].shape[0], dv + 1, device="cuda")
        per = max(1, 100_000_000 // (CONTEXT * mono[0].shape[0]))
        flat = S.view(B * H, *S.shape[2:])
        for i in range(0, B * H, per):
            m = min(per, B * H - i)
            phi = _features(normal(m, CONTEXT, dk, s=scale).float(), mono, torch.float32)
            val = torch.cat([normal(m, CONTEXT, dv).float(), torch.ones(m, CONTEXT, 1, device="cuda")], dim=-1)
            torch.bmm(phi.transpose(1, 2).contiguous(), val, out=flat[i:i + m])
        t["S"] = S
        return t
    n = case["n"]
    t = dict(q=normal(B, H * G, n, dk, s=scale), k=normal(B, H, n, dk, s=scale), v=normal(B, H, n, dv))
    if op in ("train", "backward"):
        t["dy"] = normal(B, H, n, dv)
    return t


def prepare(case, seed):
    t = _inputs(case, seed)
    t["case"] = case
    return t


def run(state):
    case = state["case"]
    op, P = case["op"], case["P"]
    if op == "feature_map":
        return sata.feature_map(state["x"], P)
    q, k, v = state["q"], state["k"], state["v"]
    if op == "decode":
        return sata.decode_step(state["S"], q, k, v, P), state["S"]
    if op == "decode_grouped":
        return sata.decode_step_grouped(state["S"], q, k, v, P), state["S"]
    if op == "prefill":
        return sata.prefill(q, k, v, P, want_state=case["state"])
    if op == "prefill_grouped":
        return sata.prefill_grouped(q, k, v, P, want_state=case["state"])
    if op == "backward":
        return sata.backward(q, k, v, state["dy"], P)
    if op == "train":
        y, _ = sata.prefill(q, k, v, P, want_state=False)
        return (y,) + tuple(sata.backward(q, k, v, state["dy"], P))
    raise ValueError(op)


# ------------------------------------------------------------------ what a pass cannot do without

def work(case):
    """Bytes: each input read once, each output written once.  Flops: of the
    two ways to the causal output (pair by pair, or through the states) the
    one with fewer, and one contraction over the tokens for a state."""
    op, dk, P, size = case["op"], case["dk"], case["P"], SIZE[case["dtype"]]
    D = math.comb(dk + P - 1, P - 1)
    if op == "feature_map":
        return {"bytes": case["rows"] * (D * 4.0 + dk * size), "flops": float(case["rows"] * D)}
    B, H, dv, G = case["B"], case["H"], case["dv"], case.get("G", 1)
    heads = B * H
    if op in ("decode", "decode_grouped"):
        return {"bytes": heads * (8.0 * D * (dv + 1) + size * (dk * (1 + G) + dv * (1 + G))),
                "flops": heads * D * (dv + 1) * 2.0 * (1 + G)}
    n = case["n"]
    pair = (n + 1) / 2.0
    update, rows = 2.0 * D * (dv + 1), heads * G * n
    forward = rows * min(pair * 2.0 * (dk + dv + P), 2.0 * D * (dv + 1) + update / G)
    io = size * n * (heads * G * (dk + dv) + heads * (dk + dv))
    if op in ("prefill", "prefill_grouped"):
        state = heads * D * (dv + 1) * 4.0 if case["state"] else 0.0
        return {"bytes": io + state, "flops": forward + (heads * n * update if case["state"] else 0.0)}
    # gradients: the scores and dy.v again, then one contraction each for dq, dk and dv
    backward = rows * min(pair * (6.0 * dk + 4.0 * dv + 4.0 * P), 10.0 * D * (dv + 1))
    io_b = size * n * heads * (4.0 * dk + 3.0 * dv)
    if op == "backward":
        return {"bytes": io_b, "flops": backward}
    return {"bytes": io + io_b, "flops": forward + backward}


def tolerance(case):
    """Four times what the path shows against `exact`.  bfloat16: outputs are
    stored in 8 bits and state contractions round their operands to 8 bits;
    float32: operands carried to 16 bits in the state contractions (prefill,
    gradients), plain float32 sums of a few terms in decode and feature map."""
    op = case["op"]
    if op == "feature_map":
        return {"rel": 3e-7, "max": 3e-6}
    if case["dtype"] == "bf16":
        return {"rel": 1e-2, "max": 0.4}
    if op in ("decode", "decode_grouped"):
        return {"rel": 2e-6, "max": 4e-4}
    return {"rel": 2e-5, "max": 4e-3}


# ------------------------------------------------------------------ the same outputs in 64 bits

def _series(s, terms):
    """The first `terms` terms of exp(s)."""
    out = torch.ones_like(s)
    for p in range(terms - 1, 0, -1):
        out.mul_(s).div_(p).add_(1.0)
    return out


def _blocks(n, width):
    for r0 in range(0, n, width):
        yield r0, min(n, r0 + width)


def _masked(s, r0):
    """Zero where the key of a column comes after the query of a row; row i is query r0 + i."""
    return s.tril_(diagonal=r0)


def _exact_rows(q, k, v1, P):
    """(y, denominators) of one head: q [n, dk], k [n, dk], v1 = [v | 1]."""
    n, dk = q.shape
    out = torch.empty(n, v1.shape[1], dtype=torch.float64, device=q.device)
    for r0, r1 in _blocks(n, 2048):
        w = _masked(_series(q[r0:r1] @ k[:r1].T / math.sqrt(dk), P), r0)
        out[r0:r1] = w @ v1[:r1]
    return out[:, :-1] / out[:, -1:], out[:, -1:]


def _exact_grads(q, k, v, dy, P):
    n, dk = q.shape
    c = math.sqrt(dk)
    y, z = _exact_rows(q, k, torch.cat([v, torch.ones_like(v[:, :1])], 1), P)
    u = dy / z
    m = (u * y).sum(1, keepdim=True)
    dq, dkk, dvv = torch.empty_like(q), torch.zeros_like(k), torch.zeros_like(v)
    for r0, r1 in _blocks(n, 2048):
        s = q[r0:r1] @ k[:r1].T / c
        dvv[:r1] += _masked(_series(s, P), r0).T @ u[r0:r1]
        g = (u[r0:r1] @ v[:r1].T - m[r0:r1]) / c
        g = _masked(g * _series(s, P - 1), r0) if P > 1 else torch.zeros_like(g)
        dq[r0:r1] = g @ k[:r1]
        dkk[:r1] += g.T @ q[r0:r1]
    return dq, dkk, dvv


def exact(case, seed):
    t = _inputs(case, seed)
    op, P, dk = case["op"], case["P"], case["dk"]
    if op == "feature_map":
        mono = _monomials(dk, P)
        out = torch.empty(case["rows"], mono[0].shape[0], dtype=torch.float64, device="cuda")
        for r0, r1 in _blocks(case["rows"], 8192):
            out[r0:r1] = _features(t["x"][r0:r1], mono, torch.float64)
        return out
    B, H, dv, G = case["B"], case["H"], case["dv"], case.get("G", 1)
    f64 = {name: x.double() for name, x in t.items() if name != "S"}
    one = lambda v: torch.cat([v, torch.ones_like(v[..., :1])], -1)  # noqa: E731
    if op in ("decode", "decode_grouped"):
        mono = _monomials(dk, P)
        S = t["S"].double()
        S += _features(f64["k"], mono, torch.float64)[..., None] * one(f64["v"])[..., None, :]
        phi = _features(f64["q"], mono, torch.float64).view(B * H, G, -1)
        o = torch.bmm(phi, S.view(B * H, *S.shape[2:])).view(B, H * G, dv + 1)
        return o[..., :dv] / o[..., dv:], S
    n = case["n"]
    if op in ("prefill", "prefill_grouped"):
        y = torch.empty(B, H * G, n, dv, dtype=torch.float64, device="cuda")
        S = mono = None
        if case["state"]:
            mono = _monomials(dk, P)
            S = torch.zeros(B, H, mono[0].shape[0], dv + 1, dtype=torch.float64, device="cuda")
        for b in range(B):
            for h in range(H):
                k, v1 = f64["k"][b, h], one(f64["v"][b, h])
                for g in range(G):
                    y[b, h * G + g] = _exact_rows(f64["q"][b, h * G + g], k, v1, P)[0]
                if mono is not None:
                    for r0, r1 in _blocks(n, 4096):
                        S[b, h] += _features(k[r0:r1], mono, torch.float64).T @ v1[r0:r1]
        return y, S
    grads = [torch.empty_like(f64[name]) for name in ("q", "k", "v")]
    y = torch.empty_like(f64["v"])
    for b in range(B):
        for h in range(H):
            q, k, v, dy = (f64[name][b, h] for name in ("q", "k", "v", "dy"))
            if op == "train":
                y[b, h] = _exact_rows(q, k, one(v), P)[0]
            for out, got in zip(grads, _exact_grads(q, k, v, dy, P)):
                out[b, h] = got
    return (y, *grads) if op == "train" else tuple(grads)
