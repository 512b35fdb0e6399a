"""GPU parity of the chunked scans by name: the case lists of the other parity
tests, and the edges of each scan kernel, through the scans whatever way the
calls' estimated cost would take them (most of these calls are short and go pair
by pair), against the float64 oracle.  Each test asserts the kernel family that
it means to run."""
import sys

import numpy as np
import pytest

import oracle
import routes
import sata_synth as syn
from gpu_util import (check_prefill_head, check_rows, check_state, check_state_against, operands, to_dev, to_host,
                      torch_dtype, y_tol)
from oracle.metrics import max_row_rel_error
from test_gpu_parity import FEATURE_KERNEL_CASES, PREFILL_CASES, SPLIT_CASES, WIDE_CASES

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def sata():
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    import paper_2602_00294_amd as m
    m.load_library()
    return m


def _say(msg):
    print(msg, file=sys.stderr, flush=True)


def _id(c):
    return "w{}_B{}H{}n{}dk{}dv{}P{}C{}_{}".format(*c)


def _run(case, heads=None, state_heads=None):
    """The scan of one case: every head (or the listed ones) and its state against the oracle."""
    import paper_2602_00294_amd as sata
    workload, B, H, n, dk, dv, P, chunk, dtype = case
    q, k, v = syn.make_qkv(workload, B, H, n, dk, dv, dtype)
    y, S = routes.prefill_by(False, *(to_dev(a, dtype) for a in (q, k, v)), P, chunk)
    torch.cuda.synchronize()
    ops = operands(sata, dtype, B, H, n, dk, dv, P, chunk)
    for b, h in heads or [(b, h) for b in range(B) for h in range(H)]:
        S_h = to_host(S[b, h]) if state_heads is None or (b, h) in state_heads else None
        check_prefill_head(to_host(y[b, h]), S_h, q[b, h], k[b, h], v[b, h], P, ops, dtype, chunk, f"{case} b{b} h{h}")


@pytest.mark.parametrize("case", PREFILL_CASES, ids=_id)
def test_scan_matches_oracle(sata, case):
    _say(f"scan {case} ({routes.scan_route(case[8], *case[1:8])})")
    _run(case)


def test_the_cases_reach_every_family():
    assert {routes.scan_route(c[8], *c[1:8]) for c in PREFILL_CASES} == {"mfma32", "blocks", "features", "float32"}


@pytest.mark.parametrize("case", FEATURE_KERNEL_CASES, ids=_id)
def test_scan_generated_features(sata, case):
    assert routes.scan_route(case[8], *case[1:8]) == "features"
    _say(f"scan, generated features {case}")
    _run(case)


@pytest.mark.parametrize("case", SPLIT_CASES, ids=_id)
def test_scan_in_parts(sata, case):
    *args, parts = case
    workload, B, H, n, dk, dv, P, chunk, dtype = args
    assert sata.prefill_parts(torch_dtype(dtype), B, H, n, dk, dv, P, chunk) == parts > 1
    _say(f"scan in parts {case}")
    _run(tuple(args))


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("case", WIDE_CASES, ids=lambda c: "w{}_dk{}dv{}P{}".format(*c))
def test_scan_wide_slices(sata, case, dtype):
    workload, dk, dv, P = case
    full = (workload, 1, 256, 40, dk, dv, P, 64, dtype)
    assert routes.scan_route(dtype, *full[1:8]) == "features"
    _say(f"scan, wide slices {full}")
    _run(full, [(0, 0), (0, 85), (0, 170), (0, 255)], [(0, 0), (0, 255)])


@pytest.mark.parametrize("d", [16, 32])
def test_scan_chunk_invariance_matrix_cores(sata, d):
    """bf16, P = 4: chunks 32, 64 and 128, different kernels or variants."""
    B, H, n, P = 1, 2, 300, 4
    families = [routes.scan_route("bf16", B, H, n, d, d, P, c) for c in (32, 64, 128)]
    assert families == ["blocks", "mfma32" if d == 32 else "blocks", "blocks"]
    q, k, v = syn.make_qkv(28 + d, B, H, n, d, d, "bf16")
    res = {}
    for c in (32, 64, 128):
        _say(f"scan chunk {c} d={d}")
        y, S = routes.prefill_by(False, *(to_dev(a, "bf16") for a in (q, k, v)), P, c)
        torch.cuda.synchronize()
        res[c] = (to_host(y), to_host(S))
        for h in range(H):
            check_prefill_head(res[c][0][0, h], res[c][1][0, h], q[0, h], k[0, h], v[0, h], P, "bf16", "bf16", c,
                               f"d{d} chunk {c} h{h}")
    for h in range(H):
        S_abs = oracle.state_abs_ref(k[0, h], v[0, h], P)
        for c in (32, 128):
            assert not np.array_equal(res[c][0][0, h], res[64][0][0, h])  # (another kernel's rounding)
            assert max_row_rel_error(res[c][0][0, h], res[64][0][0, h])[0] < 2 * y_tol("bf16", "bf16")
            check_state_against(res[c][1][0, h], res[64][1][0, h], S_abs, 2 * oracle.state_tol("bf16", n, c, P),
                                f"d{d} chunk {c} vs 64 h{h}")


@pytest.mark.parametrize("B,Hkv,G,n,d,P,chunk,dtype,family,parts", [
    (1, 2, 4, 150, 32, 4, 64, "bf16", "mfma32", 1),
    (2, 2, 2, 97, 16, 4, 32, "bf16", "blocks", 1),
    (1, 3, 2, 100, 8, 3, 64, "bf16", "features", 1),
    (1, 3, 2, 70, 8, 4, 64, "f32", "features", 1),
    (1, 1, 2, 4096, 8, 3, 64, "f32", "features", 4),
    (1, 1, 8, 40, 5, 3, 16, "f32", "float32", 1),
])
def test_scan_grouped(sata, B, Hkv, G, n, d, P, chunk, dtype, family, parts):
    """The stride between a member's query heads in each family: rows against the
    oracle, members bitwise the single-head scan's, states too."""
    assert routes.scan_route(dtype, B, Hkv, n, d, d, P, chunk) == family
    assert sata.prefill_parts(torch_dtype(dtype), B, Hkv, n, d, d, P, chunk) == parts
    _say(f"scan grouped B={B} H_kv={Hkv} G={G} n={n} d={d} P={P} chunk={chunk} {dtype}")
    q, _, _ = syn.make_qkv(600 + n, B, Hkv * G, n, d, d, dtype)
    _, k, v = syn.make_qkv(601 + n, B, Hkv, n, d, d, dtype)
    qd, kd, vd = (to_dev(a, dtype) for a in (q, k, v))
    y, S = routes.prefill_by(False, qd, kd, vd, P, chunk)
    torch.cuda.synchronize()
    ops = operands(sata, dtype, B, Hkv, n, d, d, P, chunk)
    yh = to_host(y)
    for b in range(B):
        for hq in range(Hkv * G):
            yr, _, kap = oracle.taylor_attention(q[b, hq], k[b, hq // G], v[b, hq // G], P)
            check_rows(yh[b, hq], yr, kap, y_tol(ops, dtype), P, f"b{b} query head {hq}",
                       oracle.term_scale(q[b, hq], k[b, hq // G], v[b, hq // G], P))
    for g in range(G):
        yg, Sg = routes.prefill_by(False, qd[:, g::G].contiguous(), kd, vd, P, chunk)
        torch.cuda.synchronize()
        assert torch.equal(yg, y[:, g::G]) and torch.equal(Sg, S), f"member {g}"


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_scan_unaligned_rows(sata, dtype):
    """Bases that are not 16-byte aligned are read element by element."""
    n, dk, dv, P = 140, 16, 24, 3
    assert routes.scan_route(dtype, 1, 1, n, dk, dv, P) == "features"
    _say(f"scan, unaligned rows {dtype}")
    arrays = syn.make_qkv(610, 1, 1, n, dk, dv, dtype)
    dev = []
    for a in arrays:
        t = to_dev(a, dtype)
        buf = torch.empty(a.size + 1, device="cuda", dtype=t.dtype)
        buf[1:] = t.reshape(-1)
        dev.append(buf[1:].view(*a.shape))
    y, S = routes.prefill_by(False, *dev, P)
    torch.cuda.synchronize()
    ops = operands(sata, dtype, 1, 1, n, dk, dv, P, 64)
    check_prefill_head(to_host(y)[0, 0], to_host(S)[0, 0], *(a[0, 0] for a in arrays), P, ops, dtype, 64, "unaligned")


def test_scan_in_two_segments(sata):
    """16 heads of 10240 tokens at d = 64, P = 4: the partial sums (63 slices x 65
    floats per head-token) fill the 2 GB of a segment at 8192 tokens, so the state
    is stored and loaded again; rows on both sides of the boundary, and a state."""
    H, n, d, P = 16, 10240, 64, 4
    assert routes.scan_route("bf16", 1, H, n, d, d, P) == "features"
    _say("scan in two segments")
    g = torch.Generator(device="cuda").manual_seed(620)
    q, k, v = ((torch.randn(1, H, n, d, generator=g, device="cuda") * s).to(torch.bfloat16) for s in (0.7, 0.7, 1.0))
    y, S = routes.prefill_by(False, q, k, v, P)
    torch.cuda.synchronize()
    rows = [0, 63, 64, 4095, 8127, 8128, 8191, 8192, 8193, 8255, 8256, n - 1]
    for h in (0, H - 1):
        qh, kh, vh = (t[0, h].float().cpu().numpy() for t in (q, k, v))
        yr, _, kap = oracle.taylor_attention_rows(qh, kh, vh, P, rows)
        check_rows(to_host(y[0, h])[rows], yr, kap, y_tol("bf16", "bf16"), P, f"h{h}")
    # the state by its degree-1 and degree-0 rows (the whole one is 10240 x 47905 features)
    kh, vh = (t[0, 0].double() for t in (k, v))
    one = torch.cat([vh, torch.ones_like(vh[:, :1])], 1)
    want = torch.cat([one.sum(0, keepdim=True), (kh * 64 ** -0.25).T @ one])
    got = S[0, 0, :65].double()
    scale = torch.cat([one.abs().sum(0, keepdim=True), (kh.abs() * 64 ** -0.25).T @ one.abs()])
    assert ((got - want).abs() <= oracle.state_tol("bf16", n, 64, P) * scale).all()


# ------------------------------------------------------------------ gradients

def _gradients(workload, n, dk, dv, P, dtype, quarter=False):
    q, k, v = syn.make_qkv(workload, 1, 1, n, dk, dv, dtype)
    dy = syn.make_qkv(workload + 1, 1, 1, n, dv, dv, dtype)[2]
    s = np.float32(0.5 if quarter else np.sqrt(0.5))
    q, k = ((a * s).astype(np.float32) for a in (q, k))
    if dtype == "bf16":
        q, k = syn.round_to_bf16(q), syn.round_to_bf16(k)
    return q, k, v, dy


@pytest.mark.parametrize("n,dk,dv,P,chunk,dtype", [
    (130, 8, 8, 4, 64, "f32"), (97, 16, 16, 3, 32, "f32"), (64, 4, 6, 5, 16, "f32"), (200, 32, 32, 4, 64, "bf16"),
    (300, 8, 8, 2, 64, "f32"), (150, 4, 4, 6, 64, "f32"), (100, 64, 64, 3, 64, "bf16"),
    (700, 32, 32, 2, 64, "f32"), (260, 64, 64, 2, 32, "f32"), (140, 24, 40, 4, 16, "bf16"), (90, 10, 3, 7, 32, "f32"),
])
def test_scan_backward_matches_oracle(sata, n, dk, dv, P, chunk, dtype):
    """The scans' gradients over head sizes, chunk sizes and degrees (above 3 the
    Jacobian takes the full product rule)."""
    _say(f"scan backward n={n} dk={dk} dv={dv} P={P} chunk={chunk} {dtype}")
    arrays = _gradients(630 + n, n, dk, dv, P, dtype, quarter=P == 2)
    got = routes.backward_by(False, *(to_dev(a, dtype) for a in arrays), P, chunk)
    torch.cuda.synchronize()
    want = oracle.taylor_attention_backward(*(a[0, 0] for a in arrays), P)
    for name, g, w in zip(("dq", "dk", "dv"), got, want):
        err = np.linalg.norm(to_host(g)[0, 0] - w) / np.linalg.norm(w)
        assert err <= y_tol("f32", dtype), f"{name}: {err:.3e}"


@pytest.mark.parametrize("dk,dv,P", [(8, 8, 4), (32, 32, 2), (64, 48, 2)])
def test_scan_backward_chunk_invariance(sata, dk, dv, P):
    _say(f"scan backward chunk invariance dk={dk} P={P}")
    arrays = _gradients(650 + dk, 150, dk, dv, P, "f32", quarter=P == 2)
    dev = [to_dev(a, "f32") for a in arrays]
    outs = {c: [to_host(x) for x in routes.backward_by(False, *dev, P, c)] for c in (16, 32, 64)}
    torch.cuda.synchronize()
    for c in (16, 32):
        assert not all(np.array_equal(a, b) for a, b in zip(outs[c], outs[64]))
        for a, b in zip(outs[c], outs[64]):
            assert np.linalg.norm(a - b) <= 1e-5 * np.linalg.norm(b)
