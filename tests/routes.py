"""The library's testing entries (include/sata_testing.h) for the tests: which
kernels a call takes, and calls by one way of the test's choice."""
import ctypes

ROUTES = ("pairs", "mfma32", "blocks", "features", "float32")
_I, _VP = ctypes.c_int, ctypes.c_void_p


def _lib():
    from paper_2602_00294_amd import _binding
    lib = _binding.load_library()
    lib.sata_testing_prefill_route.argtypes = [_I] * 10 + [ctypes.POINTER(_I)]
    lib.sata_testing_scan_route.argtypes = [_I] * 8 + [ctypes.POINTER(_I)]
    lib.sata_testing_backward_route.argtypes = [_I] * 8 + [ctypes.POINTER(_I)]
    lib.sata_testing_prefill.argtypes = [_I] + [_VP] * 3 + [_I] * 9 + [_VP] * 3
    lib.sata_testing_backward.argtypes = [_I] + [_VP] * 4 + [_I] * 8 + [_VP] * 4
    return lib


def _check(status):
    if status:
        from paper_2602_00294_amd import _binding
        raise _binding.SataError(status, "testing entry", _binding.load_library().sata_last_error().decode())


def prefill_route(dtype, B, H_kv, n, dk, dv, P, chunk=64, want_state=True, G=1):
    """Kernel family of sata.prefill / prefill_grouped for 'bf16' or 'f32' tensors (host only)."""
    out = _I(-1)
    _check(_lib().sata_testing_prefill_route(int(dtype == "bf16"), B, H_kv, G, n, dk, dv, P, chunk, int(want_state),
                                             ctypes.byref(out)))
    return ROUTES[out.value]


def scan_route(dtype, B, H_kv, n, dk, dv, P, chunk=64):
    """Kernel family of the scan for these sizes, whether or not the call goes by it (host only)."""
    out = _I(-1)
    _check(_lib().sata_testing_scan_route(int(dtype == "bf16"), B, H_kv, n, dk, dv, P, chunk, ctypes.byref(out)))
    return ROUTES[out.value]


def backward_route(dtype, B, H, n, dk, dv, P, chunk=64):
    """'pairs' or 'float32' (the scans) for sata.backward (host only)."""
    out = _I(-1)
    _check(_lib().sata_testing_backward_route(int(dtype == "bf16"), B, H, n, dk, dv, P, chunk, ctypes.byref(out)))
    return ROUTES[out.value]


def _p(t):
    return _VP(t.data_ptr()) if t is not None and t.numel() else _VP(None)


def _stream():
    import torch
    return _VP(torch.cuda.current_stream().cuda_stream)


def prefill_by(pairs, q, k, v, P, chunk=64, want_state=True, y=None, S=None):
    """prefill (or prefill_grouped, by the head counts) pair by pair or by the
    scan: (y, S), preallocated or not."""
    import torch
    B, Hq, n, dk = q.shape
    H, dv = k.shape[1], v.shape[-1]
    from paper_2602_00294_amd import _binding
    if y is None:
        y = torch.empty(B, Hq, n, dv, dtype=q.dtype, device=q.device)
    if want_state and S is None:
        S = torch.empty(B, H, _binding.feature_count(dk, P), dv + 1, device=q.device)
    _check(_lib().sata_testing_prefill(int(pairs), _p(q), _p(k), _p(v), int(q.dtype == torch.bfloat16), B, H, Hq // H,
                                       n, dk, dv, P, chunk, _p(y), _p(S), _stream()))
    return y, S


def backward_by(pairs, q, k, v, dy, P, chunk=64):
    """backward pair by pair or by the scans: (dq, dk, dv)."""
    import torch
    B, H, n, dk = q.shape
    dv = v.shape[-1]
    out = tuple(torch.empty_like(t) for t in (q, k, v))
    _check(_lib().sata_testing_backward(int(pairs), _p(q), _p(k), _p(v), _p(dy), int(q.dtype == torch.bfloat16), B, H,
                                        n, dk, dv, P, chunk, *(_p(t) for t in out), _stream()))
    return out
