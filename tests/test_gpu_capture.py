"""Calls captured into a graph after a warm-up of other sizes: the longer warm-up
leaves the feature table and a workspace, but not what the pair-by-pair way of
the shorter call needs, so the captured call goes by the scans; after a warm-up
of its own it goes pair by pair, and where only scratch is missing too.  Each graph is replayed several times, with
other inputs and the program's own work in between."""
import sys

import pytest

import oracle
import routes

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def sata():
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    import paper_2602_00294_amd as m
    m.load_library()
    return m


def _tensors(seed, n, d, count):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return [torch.randn(1, 2, n, d, generator=g, device="cuda") * 0.5 for _ in range(count)]


def _replays(graph, stream, held, call):
    """Replays with new inputs in the captured buffers; yields the eager result of each."""
    for seed in (11, 12, 13):
        new = _tensors(seed, held[0].shape[2], held[0].shape[3], len(held))
        with torch.cuda.stream(stream):
            for a, b in zip(held, new):
                a.copy_(b)
            graph.replay()
        stream.synchronize()
        yield call(*held)
        torch.cuda.synchronize()


@pytest.mark.parametrize("own_warm_up", [False, True])
def test_captured_prefill(sata, own_warm_up):
    n, d, P, long_n = 1500, 8, 4, 40000
    assert routes.prefill_route("f32", 1, 2, n, d, d, P) == "pairs"
    assert routes.prefill_route("f32", 1, 2, long_n, d, d, P) == "features"
    print(f"captured prefill, own warm-up {own_warm_up}", file=sys.stderr, flush=True)
    torch.cuda.synchronize()
    sata.release()
    stream = torch.cuda.Stream()
    held = _tensors(10, n, d, 3)
    y = torch.empty(1, 2, n, d, device="cuda")
    S = torch.empty(1, 2, oracle.feature_count(d, P), d + 1, device="cuda")
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream):
        sata.prefill(*_tensors(9, long_n, d, 3), P)
        if own_warm_up:
            sata.prefill(*held, P, y=y, S=S)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        sata.prefill(*held, P, y=y, S=S)
    for want_y, want_S in _replays(graph, stream, held, lambda *x: routes.prefill_by(own_warm_up, *x, P)):
        torch.cuda.synchronize()
        assert torch.equal(y, want_y) and torch.equal(S, want_S)


@pytest.mark.parametrize("warm_up", ["no_state", "more_heads"])
def test_captured_prefill_without_scratch(sata, warm_up):
    """A warm-up that leaves no scratch for the parts of the state's sum: the same
    call without a state, or more tokens in all, in heads too short for parts."""
    n, d, P = 1500, 24, 4
    assert routes.prefill_route("f32", 1, 2, n, d, d, P) == "pairs"
    assert routes.prefill_route("f32", 1, 64, 500, d, d, P) == "pairs"
    print(f"captured prefill, warm-up {warm_up}", file=sys.stderr, flush=True)
    torch.cuda.synchronize()
    sata.release()
    stream = torch.cuda.Stream()
    held = _tensors(10, n, d, 3)
    y = torch.empty(1, 2, n, d, device="cuda")
    S = torch.empty(1, 2, oracle.feature_count(d, P), d + 1, device="cuda")
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream):
        if warm_up == "no_state":
            sata.prefill(*held, P, y=y, want_state=False)
        else:
            many = [t[:, :, :500].repeat(1, 32, 1, 1) for t in held]
            sata.prefill(*many, P)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        sata.prefill(*held, P, y=y, S=S)
    for want_y, want_S in _replays(graph, stream, held, lambda *x: routes.prefill_by(True, *x, P)):
        torch.cuda.synchronize()
        # y in the same bits; the state's n terms are added in another order, in
        # float32: at most n 2^-23 of the sum of their sizes
        sizes = routes.prefill_by(True, held[0], held[1].abs(), held[2].abs(), P)[1]
        torch.cuda.synchronize()
        assert torch.equal(y, want_y)
        assert ((S - want_S).abs() <= n * 2.0 ** -23 * sizes).all()


@pytest.mark.parametrize("own_warm_up", [False, True])
def test_captured_backward(sata, own_warm_up):
    n, d, P = 500, 8, 4
    assert routes.backward_route("f32", 1, 2, n, d, d, P) == "pairs"
    print(f"captured backward, own warm-up {own_warm_up}", file=sys.stderr, flush=True)
    torch.cuda.synchronize()
    sata.release()
    stream = torch.cuda.Stream()
    held = _tensors(20, n, d, 4)
    out = None
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream):
        # (the scans need more scratch: their own call leaves it, and the table)
        routes.backward_by(own_warm_up, *held, P)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        out = sata.backward(*held, P)
    for want in _replays(graph, stream, held, lambda *x: routes.backward_by(True, *x, P)):
        torch.cuda.synchronize()
        for a, b in zip(out, want):
            assert torch.equal(a, b)
