"""Calls on a stream that is not torch's current one, with nothing synchronised after the
call: the memory a call makes must not be taken from, or given back to, work of the current
stream that is not ordered with the call's kernels.  Both host routes, streams of torch's and
streams known by their handle only.  Every comparison is bit for bit with the same call on
the current stream."""
import pytest
import torch

import paper_2606_26631_amd as prcr
from paper_2606_26631_amd import binding

pytestmark = pytest.mark.gpu
B, H, G, D, CAP = 4, 2, 4, 64, 3000


class _Declines:
    def __getattr__(self, name):
        return lambda *args: None


class _Handle:
    """A stream that is no torch.cuda.Stream."""

    def __init__(self, stream):
        self.cuda_stream = stream.cuda_stream


@pytest.fixture(params=["native", "python"])
def route(request, monkeypatch):
    monkeypatch.setattr(binding, "_NATIVE", binding._native() if request.param == "native" else _Declines())


@pytest.fixture(params=["torch", "handle"])
def side(request):
    s = torch.cuda.Stream()
    return s, (s if request.param == "torch" else _Handle(s))


def _busy(stream):
    """Some milliseconds of work on a stream."""
    with torch.cuda.stream(stream):
        a = torch.ones(4096, 4096, device="cuda")
        for _ in range(20):
            a = a @ a * 1e-4


def _decode():
    g = torch.Generator(device="cuda").manual_seed(9)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda").to(torch.bfloat16)
    cache = prcr.Cache(rnd(B, 1, H, CAP, D), rnd(B, 1, H, CAP, D))
    lens = torch.tensor([CAP, 700, 0, 1500], dtype=torch.int32, device="cuda")
    rope = prcr.Rope(D, (8, 12, 12))
    qs = [rnd(B, H * G, D) for _ in range(2)]
    return cache, lambda i, stream=None: prcr.decode_attention(rope, cache, 0, qs[i], lens, lens, stream=stream)


def test_workspace_is_not_given_away_while_the_kernels_run(route, side):
    torch_side, stream = side
    cache, call = _decode()
    ref = call(0)
    words = prcr.decode_workspace_bytes(cache, B, H * G) // 4
    torch.cuda.synchronize()
    print("workspace on a side stream", flush=True)
    _busy(torch_side)
    out = call(0, stream)
    taken = [torch.full((words,), float("nan"), device="cuda") for _ in range(8)]
    torch.cuda.synchronize()
    assert torch.equal(out, ref)
    assert all(t.isnan().all() for t in taken)


def test_outputs_are_not_blocks_still_read_on_the_current_stream(route, side):
    _, stream = side
    _, call = _decode()
    call(0)
    x = torch.arange(B * H * G * D, dtype=torch.float32, device="cuda")
    want = x.clone()
    torch.cuda.synchronize()
    print("outputs on a side stream", flush=True)
    _busy(torch.cuda.current_stream())
    y = x.clone()
    del x                                       # its block is the current stream's to hand out
    out = call(0, stream)
    torch.cuda.synchronize()
    assert torch.equal(y, want) and torch.isfinite(out).all()


def test_outputs_are_kept_until_the_current_stream_has_read_them(route, side):
    torch_side, stream = side
    _, call = _decode()
    ref = call(0)
    torch.cuda.synchronize()
    print("outputs of a side stream read on the current one", flush=True)
    out = call(0, stream)
    torch.cuda.current_stream().wait_stream(torch_side)
    _busy(torch.cuda.current_stream())
    got = out.clone()
    del out
    others = [call(1, stream) for _ in range(4)]
    torch.cuda.synchronize()
    assert torch.equal(got, ref)
    assert all(torch.equal(o, others[0]) for o in others)


@pytest.mark.parametrize("n", [12, 0])
def test_revisit_outputs_on_a_side_stream(route, side, n):
    torch_side, stream = side
    M = 64
    ints = lambda a: torch.tensor(a, dtype=torch.int32, device="cuda")
    rows = torch.randn(1, M, 2, H, D, device="cuda")
    mem = prcr.Memory(rows, rows.clone(), ints([[[0, m // 8, m % 8] for m in range(M)]]), ints([M]))
    off, idx, p_txt, lens = ints([0, n]), ints(list(range(3, 3 + n))), ints([99]), ints([100])
    rope = prcr.Rope(D, (8, 12, 12))

    def call(stream=None):
        cache = prcr.Cache(torch.zeros(1, 2, H, 128, D, device="cuda"), torch.zeros(1, 2, H, 128, D, device="cuda"))
        torch.cuda.synchronize()
        if stream is not None:
            _busy(torch_side)
        outs = prcr.revisit(rope, mem, off, idx, p_txt, cache, lens, stream=stream)
        # Blocks of the outputs' sizes on the current stream, written at once.
        blocks = [torch.full((s,), -7, dtype=torch.int64, device="cuda") for s in (1, 3 * n + 1, n + 1) for _ in range(4)]
        torch.cuda.synchronize()
        assert all((b == -7).all() for b in blocks)
        return [*outs, cache.k, cache.v]

    print("revisit on a side stream", flush=True)
    for a, b in zip(call(stream), call()):
        assert torch.equal(a, b)
