"""GPU parity of the gradients computed pair by pair (backward_direct.hip) at the
edges of its tiles, against the float64 oracle's gradients, and of the scans
that still serve sequences too long for it.

Inputs are N(0, 1/2) queries and keys (scores of about one half: no denominator
cancels).  Tolerances, per head and gradient in the Frobenius sense: float32
operands are carried to 24 bits and every sum is float32, taken in chunks of 64
tokens, so 32 roundings of 2^-24 (2e-6) bound what a few hundred tokens show
(2e-7 measured); bfloat16 outputs are rounded to 2^-9 per element, 2^-8 in all.
The scans take two bfloat16 numbers per float32 operand: 1e-4."""
import sys

import numpy as np
import pytest

import oracle
import routes
import sata_synth as syn
from gpu_util import to_dev, to_host

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
    dy = syn.make_qkv(workload + 1, B, H, n, dv, dv, dtype)[2]
    return _half(q, dtype), _half(k, dtype), v, dy


def _check(got, q, k, v, dy, P, tol, label):
    want = oracle.taylor_attention_backward(q, k, v, dy, P)
    for name, g, w in zip(("dq", "dk", "dv"), got, want):
        assert np.all(np.isfinite(g)), f"{label} {name}"
        err = np.linalg.norm(g - w) / np.linalg.norm(w)
        assert err <= tol, f"{label} {name}: {err:.3e} > {tol:.1e}"


@pytest.mark.parametrize("B,H,n,dk,dv,P,dtype", [
    (1, 2, 2, 8, 8, 4, "f32"), (1, 1, 63, 16, 16, 4, "f32"), (1, 1, 64, 17, 15, 3, "f32"),
    (1, 1, 65, 32, 33, 4, "f32"), (1, 1, 129, 48, 49, 5, "f32"), (1, 1, 70, 64, 64, 4, "f32"),
    (1, 1, 100, 1, 1, 3, "f32"), (1, 1, 90, 3, 64, 7, "f32"), (1, 1, 50, 12, 12, 8, "f32"),
    (1, 1, 193, 5, 3, 2, "f32"),
    (1, 1, 63, 16, 16, 4, "bf16"), (1, 1, 65, 24, 40, 3, "bf16"), (1, 1, 129, 64, 48, 4, "bf16"),
    (1, 1, 200, 7, 9, 6, "bf16"), (1, 1, 77, 33, 64, 2, "bf16"),
    (3, 5, 61, 8, 8, 4, "f32"),       # heads in no multiple of 8
])
def test_pairwise_backward_matches_oracle(sata, B, H, n, dk, dv, P, dtype):
    print(f"pairwise backward B={B} H={H} n={n} dk={dk} dv={dv} P={P} {dtype}", file=sys.stderr, flush=True)
    assert routes.backward_route(dtype, B, H, n, dk, dv, P) == "pairs"
    q, k, v, dy = _inputs(400 + n, B, H, n, dk, dv, dtype)
    got = [to_host(x) for x in sata.backward(*(to_dev(a, dtype) for a in (q, k, v, dy)), P)]
    torch.cuda.synchronize()
    for b in range(B):
        for h in range(H):
            _check([g[b, h] for g in got], q[b, h], k[b, h], v[b, h], dy[b, h], P,
                   2 ** -8 if dtype == "bf16" else 2e-6, f"b{b} h{h}")


def test_pairwise_backward_two_tiles_per_wave(sata):
    """Enough 128-row blocks for two tiles of own rows per wave; sampled heads."""
    B, H, n, d, P = 16, 16, 200, 16, 4
    print("pairwise backward, two tiles per wave", file=sys.stderr, flush=True)
    q, k, v, dy = _inputs(420, B, H, n, d, d, "bf16")
    got = [to_host(x) for x in sata.backward(*(to_dev(a, "bf16") for a in (q, k, v, dy)), P)]
    torch.cuda.synchronize()
    for b, h in ((0, 0), (7, 9), (15, 15)):
        _check([g[b, h] for g in got], q[b, h], k[b, h], v[b, h], dy[b, h], P, 2 ** -8, f"b{b} h{h}")


def test_pairwise_backward_unaligned_rows(sata):
    """Tensors whose base is not 16-byte aligned are read element by element."""
    n, d, P = 100, 16, 4
    print("pairwise backward, unaligned rows", file=sys.stderr, flush=True)
    arrays = _inputs(430, 1, 1, n, d, d, "f32")
    dev = []
    for a in arrays:
        buf = torch.empty(a.size + 1, device="cuda")
        buf[1:] = to_dev(a, "f32").reshape(-1)
        dev.append(buf[1:].view(*a.shape))
    got = [to_host(x)[0, 0] for x in sata.backward(*dev, P)]
    torch.cuda.synchronize()
    _check(got, *(a[0, 0] for a in arrays), P, 2e-6, "unaligned")


@pytest.mark.parametrize("n,dk,dv,P,dtype", [(2000, 8, 8, 2, "f32"), (2400, 4, 6, 3, "bf16")])
def test_scan_backward_of_long_sequences(sata, n, dk, dv, P, dtype):
    """Few features and many tokens: the scans over the states."""
    print(f"scan backward n={n} dk={dk} dv={dv} P={P} {dtype}", file=sys.stderr, flush=True)
    assert routes.backward_route(dtype, 1, 1, n, dk, dv, P) == "float32"
    q, k, v, dy = _inputs(440 + dk, 1, 1, n, dk, dv, dtype)
    if P == 2:  # keep the denominators away from the series' root
        q, k = (_half(a, dtype) for a in (q, k))
    got = [to_host(x)[0, 0] for x in sata.backward(*(to_dev(a, dtype) for a in (q, k, v, dy)), P)]
    torch.cuda.synchronize()
    _check(got, q[0, 0], k[0, 0], v[0, 0], dy[0, 0], P, 2 ** -8 if dtype == "bf16" else 1e-4, "scan")


@pytest.mark.parametrize("n,dk,dv,P", [(658, 64, 64, 2), (3000, 32, 32, 2), (2200, 48, 48, 3)])
def test_pairwise_backward_is_no_further_from_64_bits_than_the_scans(sata, n, dk, dv, P):
    """Float32 gradients of both ways against the float64 oracle: the pairs round
    no more than the scans do (dv least of all had room: 5% over at d = 64, P = 2)."""
    print(f"pairwise backward precision n={n} dk={dk} P={P}", file=sys.stderr, flush=True)
    arrays = [a.astype(np.float32) for a in _inputs(480 + dk, 1, 1, n, dk, dv, "f32")]
    if P == 2:  # keep the denominators away from the series' root
        arrays[0], arrays[1] = (_half(a, "f32") for a in arrays[:2])
    dev = [to_dev(a, "f32") for a in arrays]
    pairs, scan = (routes.backward_by(w, *dev, P) for w in (True, False))
    torch.cuda.synchronize()
    want = oracle.taylor_attention_backward(*(a[0, 0] for a in arrays), P)
    for name, a, b, w in zip(("dq", "dk", "dv"), pairs, scan, want):
        ea, eb = (np.linalg.norm(to_host(x)[0, 0] - w) / np.linalg.norm(w) for x in (a, b))
        assert ea <= 1.02 * eb, f"{name}: pairs {ea:.3e}, scan {eb:.3e}"


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("n,dk,dv,P,dtype", [(140, 16, 16, 4, "bf16"), (100, 24, 40, 3, "bf16"), (70, 64, 64, 2, "bf16"),
                                             (140, 16, 16, 4, "f32"), (100, 24, 40, 3, "f32"), (70, 48, 64, 5, "f32")])
def test_pairwise_backward_keeps_nonfinite_tokens_to_those_that_depend_on_them(sata, n, dk, dv, P, dtype, value):
    """Head t has one entry of token t that is not finite.  Gradients that do not
    depend on it are bitwise those without it; those that do are not finite."""
    print(f"pairwise backward, {value} n={n} dk={dk} dv={dv} P={P} {dtype}", file=sys.stderr, flush=True)
    one = [to_dev(a, dtype) for a in _inputs(460 + n, 1, 1, n, dk, dv, dtype)]
    clean = [g[0, 0] for g in routes.backward_by(True, *one, P)]
    t, c = torch.arange(n, device="cuda"), 2
    head, row = t[:, None], t[None, :]      # masks [head, row]
    never, always = head < 0, head >= 0
    # rows of dq, dk, dv that depend on the entry, and whether dv does in column c alone
    depend = {"q": (row == head, row <= head, row <= head, False), "k": (row >= head, always, always, False),
              "v": (row >= head, always, never, False), "dy": (row == head, row <= head, row <= head, True)}
    for i, name in enumerate(("q", "k", "v", "dy")):
        x = [a.expand(1, n, *a.shape[2:]).contiguous() for a in one]
        x[i][0, t, t, c] = value
        got = routes.backward_by(True, *x, P)
        torch.cuda.synchronize()
        for j, (what, g, want) in enumerate(zip(("dq", "dk", "dv"), got, clean)):
            bad = depend[name][j].expand(n, n)[..., None].expand(n, n, want.shape[-1]).clone()
            if what == "dv" and depend[name][3]:
                bad &= torch.arange(want.shape[-1], device="cuda") == c
            label = f"{name}: {what}"
            assert not torch.isfinite(g[0][bad]).any(), label
            assert torch.equal(g[0][~bad], want.expand(n, *want.shape)[~bad]), label
