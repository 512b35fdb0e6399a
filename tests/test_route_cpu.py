"""The choice between the pair-by-pair prefill and the chunked scan
(route.hpp), by the library's host-only query: at sizes that were timed both
ways on an MI355X the faster way is taken, and what the choice may depend on."""
import pytest

import routes

# (dtype, key/value heads, tokens, d_k, d_v, P, state wanted, us pair by pair, us by the scan): few heads and long
# sequences, few features, short calls with and without a state, rows that are no whole vectors
TIMED = [
    ("bf16", 1, 32768, 24, 24, 4, True, 289, 231), ("bf16", 2, 16384, 48, 48, 2, True, 210, 138),
    ("bf16", 4, 8192, 20, 33, 4, True, 644, 213), ("bf16", 4, 16384, 8, 8, 2, True, 148, 117),
    ("bf16", 2, 16384, 32, 8, 3, True, 159, 110), ("bf16", 2, 32768, 24, 24, 3, True, 342, 221),
    ("bf16", 1, 65536, 8, 8, 3, True, 588, 338), ("bf16", 1, 32768, 16, 16, 3, True, 302, 215),
    ("bf16", 4, 16384, 8, 8, 4, True, 153, 120), ("bf16", 16, 2048, 24, 24, 3, True, 44, 116),
    ("bf16", 1024, 256, 32, 32, 3, True, 149, 234), ("bf16", 256, 128, 64, 16, 3, True, 45, 133),
    ("bf16", 64, 4096, 16, 16, 4, True, 222, 601), ("bf16", 256, 4096, 24, 24, 3, True, 511, 766),
    ("bf16", 16, 512, 32, 32, 5, True, 118, 600), ("bf16", 64, 4096, 8, 8, 6, True, 342, 839),
    ("bf16", 1024, 16, 16, 16, 4, False, 14, 31), ("bf16", 1024, 16, 16, 16, 3, False, 13, 38),
    ("bf16", 4, 8192, 20, 33, 4, False, 380, 213), ("bf16", 1, 65536, 16, 16, 3, False, 605, 407),
    ("bf16", 1, 32768, 48, 48, 2, False, 373, 244), ("f32", 128, 1024, 24, 24, 3, True, 185, 142),
    ("f32", 1, 32768, 16, 16, 3, True, 585, 302), ("f32", 256, 512, 8, 64, 3, True, 164, 126),
    ("f32", 2, 128, 64, 16, 3, True, 37, 29), ("f32", 8, 64, 48, 48, 2, True, 32, 23),
    ("f32", 256, 1024, 16, 16, 2, True, 184, 127), ("f32", 2, 64, 64, 16, 3, True, 32, 23),
    ("f32", 8, 64, 64, 16, 3, True, 32, 24), ("f32", 1, 16384, 8, 8, 4, True, 232, 158),
    ("f32", 2, 65536, 8, 8, 8, True, 2494, 5271), ("f32", 128, 64, 48, 48, 4, True, 279, 479),
    ("f32", 2, 4096, 32, 32, 3, True, 110, 189), ("f32", 1, 1024, 8, 8, 8, True, 64, 231),
    ("f32", 2, 512, 8, 8, 8, True, 55, 125), ("f32", 1, 4096, 8, 8, 2, True, 72, 142),
    ("f32", 4, 4096, 8, 8, 2, True, 73, 142), ("f32", 256, 128, 16, 16, 3, False, 15, 26),
    ("f32", 256, 16, 8, 64, 3, False, 14, 25), ("f32", 1024, 64, 8, 8, 4, False, 18, 45),
    ("f32", 1, 32768, 16, 16, 2, False, 528, 274), ("f32", 256, 1024, 32, 32, 2, False, 245, 167),
    ("f32", 1, 8192, 48, 48, 2, False, 252, 190),
]


@pytest.mark.parametrize("dtype,heads,n,dk,dv,P,state,pairs_us,scan_us", TIMED)
def test_the_faster_way_is_taken(dtype, heads, n, dk, dv, P, state, pairs_us, scan_us):
    got = routes.prefill_route(dtype, 1, heads, n, dk, dv, P, want_state=state)
    assert (got == "pairs") == (pairs_us < scan_us), got


def test_what_the_route_depends_on():
    for dtype in ("bf16", "f32"):
        for dk, dv, P in ((8, 8, 3), (16, 16, 4), (32, 32, 4), (24, 40, 3), (7, 9, 5), (64, 64, 2)):
            for H in (1, 8, 64, 512):
                for n in (1, 64, 500, 4096, 30000):
                    with_state = routes.prefill_route(dtype, 1, H, n, dk, dv, P)
                    without = routes.prefill_route(dtype, 1, H, n, dk, dv, P, want_state=False)
                    # the state costs the pair-by-pair way more
                    assert with_state != "pairs" or without == "pairs"
                    # members of a group take their single-head prefill's way
                    for G in (2, 8):
                        assert routes.prefill_route(dtype, 1, H, n, dk, dv, P, G=G) == with_state
                    # batch and heads count alike
                    if H > 1:
                        assert routes.prefill_route(dtype, 2, H // 2, n, dk, dv, P) == with_state


def test_shapes_without_pairs():
    assert routes.prefill_route("f32", 1, 4, 100, 65, 8, 2) == "float32"         # d_k above 64
    assert routes.prefill_route("bf16", 1, 4, 100, 8, 8, 1) == "float32"         # a single feature
    assert routes.prefill_route("f32", 1, 4, 100, 8, 8, 4, chunk=32) == "float32"
    assert routes.prefill_route("bf16", 1, 4, (1 << 22) + 1, 8, 8, 4) == "features"
    assert routes.prefill_route("bf16", 1, 64, 200000, 32, 32, 4) == "features"  # 8 GB of readouts: no tuned kernel
    assert routes.prefill_route("bf16", 64, 32, 8192, 16, 16, 4) == "blocks"
    assert routes.prefill_route("bf16", 1, 64, 16384, 32, 32, 4) == "mfma32"
    with pytest.raises(RuntimeError):
        routes.prefill_route("bf16", 1, 4, 100, 8, 8, 4, chunk=48)


@pytest.mark.parametrize("dtype,n", [("f32", 32768), ("bf16", 49152)])
def test_grids_past_a_launch_go_by_the_scan(dtype, n):
    """2^24 blocks of 256 threads are one too many for a launch: 65536 heads (in
    eights) x 256 blocks of 64 x 2 or 3 query rows."""
    assert routes.prefill_route(dtype, 1, 65535, n - 192, 12, 12, 8) == "pairs"
    assert routes.prefill_route(dtype, 1, 65535, n, 12, 12, 8) == "features"
    assert routes.prefill_route(dtype, 1, 8191, n, 12, 12, 8) == "pairs"
    assert routes.prefill_route(dtype, 1, 8191, n, 12, 12, 8, G=8) == "pairs"        # 65528 query heads: 8 heads fewer
    assert routes.prefill_route(dtype, 1, 8191, n + 200, 12, 12, 8, G=8) == "features"
    rows = 16384 if dtype == "f32" else 32768
    assert routes.backward_route(dtype, 1, 65535, rows - 128, 16, 16, 8) == "pairs"
    assert routes.backward_route(dtype, 1, 65535, rows, 16, 16, 8) == "float32"
