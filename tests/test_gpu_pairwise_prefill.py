"""GPU parity of the prefill computed pair by pair (prefill_direct_kernel.hpp)
and of the state summed over the tokens (prefill_state.hip) at the edges of
their tiles, against the float64 oracle, with the bounds of the arithmetic that
the library reports for the call, whatever way the calls' estimated cost would
take them; and of the scan kernels at lengths that they serve."""
import math
import sys

import numpy as np
import pytest

import oracle
import routes
import sata_synth as syn
from gpu_util import check_prefill_head, check_rows, check_state, operands, to_dev, to_host, y_tol

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def sata():
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    import paper_2602_00294_amd as m
    m.load_library()
    return m


def _half(x, dtype):
    x = (x * np.float32(np.sqrt(0.5))).astype(np.float32)
    return syn.round_to_bf16(x) if dtype == "bf16" else x


def _inputs(workload, B, H, n, dk, dv, dtype):
    q, k, v = syn.make_qkv(workload, B, H, n, dk, dv, dtype)
    return _half(q, dtype), _half(k, dtype), v


# d_k across the contraction steps (16, 32, 64) and their packing, d_v across
# the column tiles with and without normaliser blocks, lengths around a chunk,
# every number of symbols per tuple
SHAPES = [(1, 8, 8, 4), (63, 16, 16, 3), (64, 17, 15, 4), (65, 32, 31, 4), (130, 33, 32, 3), (193, 64, 64, 3),
          (100, 1, 1, 5), (128, 2, 48, 6), (90, 3, 63, 7), (70, 4, 2, 8), (257, 16, 33, 2), (300, 40, 16, 3),
          (200, 31, 49, 2), (150, 8, 16, 6)]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n,dk,dv,P", SHAPES)
def test_pairwise_prefill_matches_oracle(sata, n, dk, dv, P, dtype):
    print(f"pairwise prefill n={n} dk={dk} dv={dv} P={P} {dtype}", file=sys.stderr, flush=True)
    B, H = 1, 3
    q, k, v = _inputs(500 + n, B, H, n, dk, dv, dtype)
    y, S = routes.prefill_by(True, *(to_dev(a, dtype) for a in (q, k, v)), P)
    torch.cuda.synchronize()
    ops = operands(sata, dtype, B, H, n, dk, dv, P, 64)
    for h in range(H):
        check_prefill_head(to_host(y)[0, h], to_host(S)[0, h], q[0, h], k[0, h], v[0, h], P, ops, dtype, 64, f"h{h}")


@pytest.mark.parametrize("B,H,n,d,P,dtype", [
    (4, 40, 700, 32, 4, "bf16"),   # three query tiles per wave
    (3, 43, 600, 64, 3, "bf16"),   # two
    (4, 40, 500, 16, 4, "f32"),    # two, packed operands
    (2, 5, 2100, 8, 4, "bf16"),    # the state in parts
    (1, 2, 1500, 24, 3, "f32"),
])
def test_pairwise_prefill_many_blocks(sata, B, H, n, d, P, dtype):
    """Blocks of several tiles per wave and sequences in parts; sampled heads."""
    print(f"pairwise prefill B={B} H={H} n={n} d={d} P={P} {dtype}", file=sys.stderr, flush=True)
    assert routes.prefill_route(dtype, B, H, n, d, d, P) == "pairs"
    q, k, v = _inputs(520 + d, B, H, n, d, d, dtype)
    y, S = sata.prefill(*(to_dev(a, dtype) for a in (q, k, v)), P)
    y2, S2 = sata.prefill(*(to_dev(a, dtype) for a in (q, k, v)), P)
    y3, _ = sata.prefill(*(to_dev(a, dtype) for a in (q, k, v)), P, want_state=False)
    torch.cuda.synchronize()
    assert torch.equal(y, y2) and torch.equal(S, S2) and torch.equal(y, y3)
    ops = operands(sata, dtype, B, H, n, d, d, P, 64)
    for b, h in {(0, 0), (B // 2, H // 2), (B - 1, H - 1)}:
        check_prefill_head(to_host(y[b, h]), to_host(S[b, h]), q[b, h], k[b, h], v[b, h], P, ops, dtype, 64,
                           f"b{b} h{h}")


@pytest.mark.parametrize("calls", [(("bf16", 32), ("f32", 16)), (("bf16", 64), ("f32", 32))])
@pytest.mark.parametrize("reverse", [False, True])
def test_pairwise_prefill_tables_of_both_types(sata, calls, reverse):
    """bfloat16 and float32 calls of one (d_k, P) whose blocks of features have
    the same shape and those of normalisers not: whichever comes first, every
    element of the second one's state is written."""
    n, dk, P = 100, 32, 4
    sata.release()
    for dtype, dv in calls[::-1] if reverse else calls:
        print(f"pairwise prefill tables {dtype} dv={dv}", file=sys.stderr, flush=True)
        q, k, v = _inputs(530, 1, 1, n, dk, dv, dtype)
        S = torch.full((1, 1, oracle.feature_count(dk, P), dv + 1), float("nan"), device="cuda")
        y, _ = routes.prefill_by(True, *(to_dev(a, dtype) for a in (q, k, v)), P, S=S)
        torch.cuda.synchronize()
        ops = operands(sata, dtype, 1, 1, n, dk, dv, P, 64)
        check_prefill_head(to_host(y)[0, 0], to_host(S)[0, 0], q[0, 0], k[0, 0], v[0, 0], P, ops, dtype, 64,
                           f"{dtype} dv={dv}")


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_pairwise_prefill_unaligned_rows(sata, dtype):
    """Bases that are not 16-byte aligned are read element by element, and y is
    written element by element."""
    n, dk, dv, P = 140, 16, 16, 4
    print(f"pairwise prefill, unaligned rows {dtype}", file=sys.stderr, flush=True)
    arrays = _inputs(540, 1, 1, n, dk, dv, dtype)
    dev = []
    for a in arrays + (np.zeros((1, 1, n, dv), np.float32),):
        t = to_dev(a, dtype)
        buf = torch.empty(a.size + 1, device="cuda", dtype=t.dtype)
        buf[1:] = t.reshape(-1)
        dev.append(buf[1:].view(*a.shape))
    y, S = routes.prefill_by(True, *dev[:3], P, y=dev[3])
    torch.cuda.synchronize()
    ops = operands(sata, dtype, 1, 1, n, dk, dv, P, 64)
    check_prefill_head(to_host(y)[0, 0], to_host(S)[0, 0], *(a[0, 0] for a in arrays), P, ops, dtype, 64, "unaligned")


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_pairwise_prefill_keeps_nonfinite_tokens_to_later_chunks(sata, dtype):
    """A NaN key leaves the rows of earlier 64-token chunks as they are; a NaN
    query leaves every other row."""
    n, d, P = 300, 16, 4
    print(f"pairwise prefill, non-finite tokens {dtype}", file=sys.stderr, flush=True)
    q, k, v = (to_dev(a, dtype) for a in _inputs(550, 1, 1, n, d, d, dtype))
    y0, _ = routes.prefill_by(True, q, k, v, P)
    bad_k, bad_q = k.clone(), q.clone()
    bad_k[0, 0, 150, 3] = float("nan")
    bad_q[0, 0, 150, 3] = float("nan")
    yk, _ = routes.prefill_by(True, q, bad_k, v, P)
    yq, _ = routes.prefill_by(True, bad_q, k, v, P)
    torch.cuda.synchronize()
    assert torch.equal(yk[0, 0, :128], y0[0, 0, :128]) and torch.isnan(yk[0, 0, 150:]).all()
    keep = [t for t in range(n) if t != 150]
    assert torch.equal(yq[0, 0, keep], y0[0, 0, keep]) and torch.isnan(yq[0, 0, 150]).all()


@pytest.mark.parametrize("dk,P", [(16, 8), (8, 8), (64, 4), (32, 5)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_pairwise_range_of_scores(sata, dtype, dk, P):
    """Scores so large that f_P nears 2^112: n |v| times that, 2^121, and the
    factor within 2^(+-3.5) that the kernels leave on the weights are inside
    float32; (P-1)! d_k^((P-1)/2), at least 2^11 here, would not be."""
    n, dv = 96, 16
    print(f"pairwise range dk={dk} P={P} {dtype}", file=sys.stderr, flush=True)
    q, k, v = (np.abs(a) for a in _inputs(570, 1, 1, n, dk, dv, dtype))
    dy = _inputs(571, 1, 1, n, dk, dv, dtype)[2]
    top = np.max(q[0, 0].astype(np.float64) @ k[0, 0].T.astype(np.float64)) / np.sqrt(dk)
    q = q * np.float32(2.0 ** np.floor(np.log2((2.0 ** 112 * math.factorial(P - 1)) ** (1 / (P - 1)) / top)))
    dev = [to_dev(a, dtype) for a in (q, k, v, dy)]
    y, _ = routes.prefill_by(True, *dev[:3], P, want_state=False)
    grads = routes.backward_by(True, *dev, P)
    torch.cuda.synchronize()
    ref, _, kap = oracle.taylor_attention(q[0, 0], k[0, 0], v[0, 0], P)
    check_rows(to_host(y)[0, 0], ref, kap, y_tol("split" if dtype == "f32" else "bf16", dtype), P, "y")
    want = oracle.taylor_attention_backward(q[0, 0], k[0, 0], v[0, 0], dy[0, 0], P)
    for name, g, w in zip(("dq", "dk", "dv"), grads, want):
        g = to_host(g)[0, 0]
        assert np.isfinite(g).all(), name
        # the scores' relative rounding, (P-1) 2^-24, times a - mu's cancellation
        assert np.linalg.norm(g - w) <= (2 ** -8 if dtype == "bf16" else 1e-5) * np.linalg.norm(w), name


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n,dk,dv,P", [(130, 16, 16, 4), (100, 48, 64, 2)])
def test_pairwise_prefill_keeps_nonfinite_values_to_their_tile(sata, n, dk, dv, P, dtype):
    """Head t has a NaN in column 2 of token t's value: the other columns, and the
    rows of earlier tiles of 16 tokens, are bitwise those without it, and the
    rows from t on NaN (the scans keep to the same tiles)."""
    print(f"pairwise prefill, NaN values n={n} dk={dk} dv={dv} P={P} {dtype}", file=sys.stderr, flush=True)
    one = [to_dev(a, dtype) for a in _inputs(560 + n, 1, 1, n, dk, dv, dtype)]
    clean = routes.prefill_by(True, *one, P, want_state=False)[0][0, 0]
    q, k, v = (a.expand(1, n, *a.shape[2:]).contiguous() for a in one)
    t = torch.arange(n, device="cuda")
    v[0, t, t, 2] = float("nan")
    y = routes.prefill_by(True, q, k, v, P, want_state=False)[0][0]
    torch.cuda.synchronize()
    others = [c for c in range(dv) if c != 2]
    assert torch.equal(y[..., others], clean[:, others].expand(n, n, dv - 1))
    earlier = t[None, :] < 16 * (t[:, None] // 16)
    assert torch.equal(y[..., 2][earlier], clean[:, 2].expand(n, n)[earlier])
    assert torch.isnan(y[..., 2][t[None, :] >= t[:, None]]).all()


@pytest.mark.parametrize("B,H,n,d,P,dtype,family", [
    (16, 32, 4000, 16, 4, "bf16", "blocks"),
    (2, 32, 20000, 32, 4, "bf16", "mfma32"),
    (8, 32, 2100, 8, 3, "f32", "features"),     # split operands
    (8, 32, 6000, 8, 2, "bf16", "features"),
])
def test_scan_prefill_of_long_sequences(sata, B, H, n, d, P, dtype, family):
    """Sequences long enough for the chunked scan: sampled rows of two heads and
    their whole states."""
    print(f"scan prefill B={B} H={H} n={n} d={d} P={P} {dtype}", file=sys.stderr, flush=True)
    assert routes.prefill_route(dtype, B, H, n, d, d, P) == routes.scan_route(dtype, B, H, n, d, d, P) == family
    g = torch.Generator(device="cuda").manual_seed(n)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    q, k, v = ((torch.randn(B, H, n, d, generator=g, device="cuda") * s).to(dt) for s in (0.5 ** 0.5, 0.5 ** 0.5, 1.0))
    y, S = sata.prefill(q, k, v, P)
    torch.cuda.synchronize()
    ops = operands(sata, dtype, B, H, n, d, d, P, 64)
    rows = sorted({0, 1, 63, 64, n // 2, n - 65, n - 2, n - 1})
    for b, h in ((0, 0), (B - 1, H - 1)):
        qh, kh, vh = (t[b, h].float().cpu().numpy() for t in (q, k, v))
        ref, _, kap = oracle.taylor_attention_rows(qh, kh, vh, P, rows)
        check_rows(to_host(y[b, h])[rows], ref, kap, y_tol(ops, dtype), P, f"b{b} h{h}")
        check_state(to_host(S[b, h]), kh, vh, P, ops, n, 64, f"state b{b} h{h}")
