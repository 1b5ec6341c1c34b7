"""Calls on several streams, from several threads and under graph capture: what scratch each uses, and their results."""
import threading

import pytest

import paper_2603_04127_amd as dk

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _problem(seed, L=1500):
    g = torch.Generator(device="cuda").manual_seed(seed)
    Q, K, V = (torch.randn(2, 4, L, 64, generator=g, device="cuda") for _ in range(3))
    M = torch.eye(64, device="cuda") + 0.1 * torch.randn(4, 64, 64, generator=g, device="cuda")
    return Q, K, V, M, torch.randn(4, 128, 64, generator=g, device="cuda")


def _scratch(stream):
    with torch.cuda.stream(stream):
        return dk._workspace(1 << 20, torch.device("cuda", torch.cuda.current_device()))[0].data_ptr()


def test_streams_and_threads_have_scratch_of_their_own():
    # neither are ordered against each other
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    got = {}
    t = threading.Thread(target=lambda: got.update(thread=_scratch(a)))
    got.update(a=_scratch(a), b=_scratch(b))
    t.start()
    t.join()
    assert _scratch(a) == got["a"] and len(set(got.values())) == 3
    streams = [torch.cuda.Stream() for _ in range(2 * dk._MAX_WORKSPACES)]
    for s in streams:
        _scratch(s)
    assert len(dk._ws_cache) <= dk._MAX_WORKSPACES


def test_calls_on_two_streams_do_not_meet():
    x, y = _problem(1), _problem(2)
    want = [dk.dark_attn_causal_fwd(*p) for p in (x, y)]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(2)]
    for _ in range(10):
        got = []
        for p, s in zip((x, y), streams):
            with torch.cuda.stream(s):
                got.append(dk.dark_attn_causal_fwd(*p))
        torch.cuda.synchronize()
        assert all(torch.equal(g, w) for g, w in zip(got, want))


def test_a_captured_call_keeps_its_scratch():
    # Replays give the eager result whatever has been called since, and with the scratch of eager calls dropped.
    x = _problem(3)
    want = dk.dark_attn_fwd(*x)
    other = dk.dark_attn_fwd(*_problem(4))
    torch.cuda.synchronize()
    out = torch.empty_like(want)
    graph = torch.cuda.CUDAGraph()
    kept = dict(dk._ws_cache)
    with torch.cuda.graph(graph):
        dk.dark_attn_fwd(*x, out=out)
    assert {k: v.data_ptr() for k, v in dk._ws_cache.items()} == {k: v.data_ptr() for k, v in kept.items()}
    for _ in range(3):
        out.zero_()
        graph.replay()
        again = dk.dark_attn_fwd(*_problem(4))
        torch.cuda.synchronize()
        assert torch.equal(out, want) and torch.equal(again, other)
        dk._ws_cache.clear()
        torch.empty(1 << 24, device="cuda").fill_(float("nan"))
