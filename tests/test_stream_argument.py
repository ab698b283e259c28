"""Memory of calls that are given a stream which is not the current one: what a call allocates comes from that stream's own
pool, so neither stream's work can be written over by the other's.  The allocation rule without a GPU, its effect on one."""
import contextlib

import pytest
import torch

q = pytest.importorskip("paper_2605_21072_amd")
from paper_2605_21072_amd import binding  # noqa: E402


def test_allocations_belong_to_the_stream_that_is_given(monkeypatch):
    inside, made, marked, given = [], [], [], []

    class Stream:
        pass

    other, current = Stream(), Stream()

    @contextlib.contextmanager
    def on(stream):
        inside.append(stream)
        yield
        inside.pop()

    empty = torch.empty

    def logged_empty(*a, **kw):
        t = empty(*a, **kw)
        made.append((t.data_ptr(), inside[-1] if inside else None))
        return t

    class Lib:
        qarvd_linear_workspace = staticmethod(lambda M, K, K_o: 4096)

        @staticmethod
        def qarvd_linear(*a):
            given.extend((a[14], a[17]))           # Y, workspace
            return 0

    monkeypatch.setattr(binding, "load_library", lambda: Lib)
    monkeypatch.setattr(binding, "_dev2d", lambda t, what: None)
    monkeypatch.setattr(binding, "_stream", lambda s: 0)
    monkeypatch.setattr(torch, "empty", logged_empty)
    monkeypatch.setattr(torch.cuda, "Stream", Stream)
    monkeypatch.setattr(torch.cuda, "stream", on)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device=None: current)
    monkeypatch.setattr(torch.Tensor, "record_stream", lambda t, s: marked.append((t.data_ptr(), s)))
    X, f = torch.zeros(4, 64), torch.zeros(8)
    w = q.DualScaleWeight(torch.zeros(8, 128, dtype=torch.int8), f, f, torch.zeros(64, dtype=torch.int32), 0, 8, 64)

    Y = binding.w8a8_linear(X, w, None)
    assert made[-2:] == [(given[1], None), (given[0], None)] and not marked
    Y = binding.w8a8_linear(X, w, None, stream=other)
    assert sorted(made[-2:], key=lambda m: m[0]) == sorted([(given[2], other), (given[3], other)], key=lambda m: m[0])
    assert marked == [(Y.data_ptr(), current)]      # the result; nobody but the call sees the scratch


def layer(seed, M=256, K=1536, N=1536):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    W = torch.randn((N, K), generator=gen, device="cuda") * 0.02
    W[:, 5:9] *= 20
    return torch.randn((M, K), generator=gen, device="cuda"), q.quantize_weight(W)


@pytest.mark.gpu
def test_scratch_is_not_handed_out_while_the_given_stream_is_behind():
    X, w = layer(1)
    want = q.w8a8_linear(X, w, None)
    need = q.load_library().qarvd_linear_workspace(X.shape[0], X.shape[1], w.K_o)
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        torch.cuda._sleep(20_000_000)
    Y = q.w8a8_linear(X, w, None, stream=s)                       # still waiting on s
    fill = [torch.full((need,), 0x5A, dtype=torch.uint8, device="cuda") for _ in range(4)]
    torch.cuda.synchronize()
    assert torch.equal(Y, want)
    assert all(bool((f == 0x5A).all()) for f in fill)


@pytest.mark.gpu
def test_a_stream_that_runs_ahead_leaves_freed_memory_of_the_current_one_alone():
    X, w = layer(2)
    want = q.w8a8_linear(X, w, None)
    s = torch.cuda.Stream()
    sizes = (q.load_library().qarvd_linear_workspace(X.shape[0], X.shape[1], w.K_o), want.numel() * 2)
    held = [torch.full((n,), 0x5A, dtype=torch.uint8, device="cuda") for n in sizes]
    torch.cuda.synchronize()
    torch.cuda._sleep(20_000_000)                                 # the copies below have not run when s does
    copies = [h.clone() for h in held]
    del held
    Y = q.w8a8_linear(X, w, None, stream=s)
    torch.cuda.synchronize()
    assert torch.equal(Y, want)
    assert all(bool((c == 0x5A).all()) for c in copies)


@pytest.mark.gpu
def test_two_given_streams_at_once():
    (X1, w1), (X2, w2) = layer(3), layer(4)
    want = [q.w8a8_linear(X1, w1, None), q.w8a8_linear(X2, w2, None)]
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    for s in (s1, s2):
        with torch.cuda.stream(s):
            torch.cuda._sleep(5_000_000)
    got = [(q.w8a8_linear(X1, w1, None, stream=s1), q.w8a8_linear(X2, w2, None, stream=s2)) for _ in range(8)]
    pair = q.quant_act(X1, w1.perm, w1.K_o, stream=s1)
    Y = q.w8a8_dual_gemm(*pair, w1, None, X1.shape[0], stream=s1)
    del pair
    torch.cuda.synchronize()
    assert all(torch.equal(a, want[0]) and torch.equal(b, want[1]) for a, b in got)
    assert torch.equal(Y, want[0])
