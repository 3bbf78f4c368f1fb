"""The two host routes of every entry point: the native module's call and the Python path
give the same bits, and a call that one refuses the other refuses with the same error."""
import numpy as np
import pytest
import torch

import paper_2606_26631_amd as prcr
from paper_2606_26631_amd import binding

gpu = pytest.mark.gpu
B, M, NL, H, D, S = 3, 20, 2, 2, 64, 48


class _Declines:
    """Stands for a native module that takes no call."""

    def __getattr__(self, name):
        return lambda *args: None


def _ints(a, dtype=torch.int32):
    return torch.tensor(a, dtype=dtype, device="cuda")


def _setup(paged, key_only):
    g = torch.Generator(device="cuda").manual_seed(4)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda", dtype=torch.float32).to(torch.bfloat16)
    coords = _ints([[[0, m // 5, m % 5] for m in range(M)]] * B)
    v_slot = _ints([list(range(M))] * B) if key_only else None
    mem = prcr.Memory(rnd(B, M, NL, H, D), None if key_only else rnd(B, M, NL, H, D), coords, _ints([M] * B),
                      v_slot)
    if paged:
        table = _ints(np.random.default_rng(1).permutation(B * 4).reshape(B, 4).tolist())
        cache = prcr.Cache(rnd(NL, B * 4, 16, H, D), rnd(NL, B * 4, 16, H, D), table)
    else:
        cache = prcr.Cache(rnd(B, NL, H, 64, D), rnd(B, NL, H, 64, D))
    x = dict(rope=prcr.Rope(D, (8, 12, 12)), mem=mem, cache=cache, off=_ints([0, 5, 5, 12]),
             idx=_ints([1, 3, 7, 8, 19, 0, 2, 4, 6, 8, 10, 12]), p_txt=_ints([40, 41, 42]), cl=_ints([41, 40, 44]),
             raw_k=rnd(B, S, H, D), raw_v=rnd(B, S, H, D), rows=_ints([list(range(4, 4 + M))] * B),
             pos=_ints([[[s, s, s] for s in range(S)]] * B), n_tok=_ints([S, S - 5, 9]),
             vis=_ints([[m - 4 if 4 <= m < 4 + M else -1 for m in range(S)]] * B), start=_ints([0, 1, 2]),
             q=rnd(B, H * 3, D), new_pos=torch.rand(12, 3, dtype=torch.float64, device="cuda") * 50,
             err=torch.zeros(1, dtype=torch.int32, device="cuda"))
    return x


def _calls(x, **kw):
    """Every entry point, as (name, call)."""
    stream = kw.pop("stream", None)
    e = dict(err=x["err"], stream=stream)
    r, m, c = x["rope"], x["mem"], x["cache"]
    return [
        ("store_raw", lambda: prcr.store_raw(m, 1, x["raw_k"], x["raw_v"], x["rows"], **e)),
        ("reassign_coords", lambda: prcr.reassign_coords(m, x["off"], x["idx"], x["p_txt"], "uir", 3, **e)),
        ("rebind_inject", lambda: prcr.rebind_inject(r, m, x["off"], x["idx"], x["new_pos"], c, x["cl"], **e)),
        ("revisit", lambda: prcr.revisit(r, m, x["off"], x["idx"], x["p_txt"], c, x["cl"], "shift", **e)),
        ("revisit", lambda: prcr.revisit(r, m, x["off"], x["idx"], x["p_txt"], c, x["cl"], store_positions=False, **e)),
        ("prefill_capture", lambda: prcr.prefill_capture(r, m, 0, x["raw_k"], x["raw_v"], x["pos"], x["n_tok"],
                                                         x["vis"], c, x["start"], **e)),
        ("decode_attention", lambda: prcr.decode_attention(r, c, 1, x["q"], x["cl"], x["cl"], **e)),
        ("decode_attention", lambda: prcr.decode_attention(r, c, 1, x["q"], x["cl"], x["cl"], scale=0.3, **e)),
        ("decode_attention_static", lambda: prcr.decode_attention_static(r, c, 0, x["q"], x["cl"], x["cl"], **e)),
    ]


@gpu
@pytest.mark.parametrize("paged", [False, True], ids=["contiguous", "paged"])
@pytest.mark.parametrize("key_only", [False, True], ids=["values", "key_only"])
def test_native_call_equals_the_python_path(monkeypatch, paged, key_only):
    native = binding._native()
    side = torch.cuda.Stream()
    got = []
    for route in ("native", "python"):
        taken = []

        class Recorder:
            def __getattr__(self, name):
                def call(*args):
                    out = getattr(native, name)(*args)
                    taken.append((name, out is not None))
                    return out
                return call

        monkeypatch.setattr(binding, "_NATIVE", Recorder() if route == "native" else _Declines())
        for stream in (None, side):
            x = _setup(paged, key_only)
            side.wait_stream(torch.cuda.current_stream())
            outs = []
            for name, call in _calls(x, stream=stream):
                print(route, name, flush=True)
                r = call()
                outs += [r] if not isinstance(r, tuple) else list(r)
                torch.cuda.synchronize()
            state = [x["cache"].k, x["cache"].v, x["mem"].k, x["mem"].v, x["mem"].coords, x["mem"].v_slot, x["err"]]
            got.append(outs + state)
        if route == "native":
            assert len(taken) == 18 and all(t for _, t in taken), taken
    for other in got[1:]:
        assert len(other) == len(got[0])
        for a, b in zip(got[0], other):
            assert (a is None) == (b is None)
            if a is not None:
                assert a.dtype == b.dtype and a.shape == b.shape
                assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))


@gpu
def test_native_call_uses_the_outputs_it_is_given():
    x = _setup(False, False)
    dev = dict(device="cuda")
    np_, nx = torch.empty(12, 3, dtype=torch.float64, **dev), torch.empty(B, dtype=torch.int32, **dev)
    nl, sm = torch.empty(B, dtype=torch.int32, **dev), torch.empty(12, dtype=torch.int64, **dev)
    r = prcr.revisit(x["rope"], x["mem"], x["off"], x["idx"], x["p_txt"], x["cache"], x["cl"], new_pos=np_,
                     next_pos=nx, new_cache_len=nl, slot_mapping=sm)
    assert all(a is b for a, b in zip(r, (np_, nx, nl, sm)))
    out = torch.empty(B, H * 3, D, dtype=torch.float32, **dev)
    ws = torch.empty(prcr.decode_workspace_bytes(x["cache"], B, H * 3), dtype=torch.uint8, **dev)
    assert prcr.decode_attention(x["rope"], x["cache"], 0, x["q"], x["cl"], x["cl"], out=out, workspace=ws) is out
    torch.cuda.synchronize()
    assert torch.equal(nl.cpu(), x["cl"].cpu() + torch.tensor([5, 0, 7], dtype=torch.int32))


@gpu
def test_refusals_are_the_same_on_both_routes(monkeypatch):
    """Every call is refused on the host, before a launch."""
    x = _setup(False, False)
    paged = _setup(True, False)["cache"]
    r, m, c, off, idx = x["rope"], x["mem"], x["cache"], x["off"], x["idx"]
    cl, pt, q = x["cl"], x["p_txt"], x["q"]
    bad_off = _ints([0, 5, 12])
    both = torch.zeros(2 * B, dtype=torch.int32, device="cuda")
    bad = [
        lambda: prcr.store_raw(m, 2, x["raw_k"], x["raw_v"], x["rows"]),
        lambda: prcr.store_raw(m, 0, x["raw_k"].float(), x["raw_v"], x["rows"]),
        lambda: prcr.store_raw(m, 0, x["raw_k"], None, x["rows"]),
        lambda: prcr.store_raw(m, 0, x["raw_k"], x["raw_v"], x["rows"][:, :-1]),
        lambda: prcr.store_raw(m, "0", x["raw_k"], x["raw_v"], x["rows"].cpu()),
        lambda: prcr.reassign_coords(m, bad_off, idx, pt),
        lambda: prcr.reassign_coords(m, off, idx.long(), pt),
        lambda: prcr.reassign_coords(m, off, idx, pt, "nearest"),
        lambda: prcr.reassign_coords(m, off, idx, pt, l_ext=-1),
        lambda: prcr.reassign_coords(m, off, idx, pt, next_pos=m.n_visual),
        lambda: prcr.reassign_coords(m, off, idx, pt, new_pos=x["new_pos"].t()),
        lambda: prcr.reassign_coords(m, off, idx, pt, err=both[:0]),
        lambda: prcr.rebind_inject(r, m, off, idx, x["new_pos"], c, cl, new_cache_len=cl),
        lambda: prcr.rebind_inject(r, m, off, idx, x["new_pos"][:-1], c, cl),
        lambda: prcr.rebind_inject(prcr.Rope(D, (8, 8, 8)), m, off, idx, x["new_pos"], c, cl),
        lambda: prcr.rebind_inject(prcr.Rope(D, (10, 11, 11)), m, off, idx, x["new_pos"], c, cl),
        lambda: prcr.rebind_inject(r, m, off, idx, x["new_pos"], prcr.Cache(c.k[:2], c.v[:2]), cl),
        lambda: prcr.revisit(r, m, off, idx, pt, c, cl, next_pos=both[:B], new_cache_len=both[2:2 + B]),
        lambda: prcr.revisit(r, m, off, idx, pt, c, cl, next_pos=pt),
        lambda: prcr.revisit(r, m, off, idx, pt.cpu(), c, cl),
        lambda: prcr.revisit(None, m, off, idx, pt, c, cl),
        lambda: prcr.prefill_capture(r, m, -1, x["raw_k"], x["raw_v"], x["pos"], x["n_tok"], x["vis"], c, x["start"]),
        lambda: prcr.prefill_capture(r, m, 0, x["raw_k"], x["raw_v"], x["pos"][:, :-1], x["n_tok"], x["vis"], c, x["start"]),
        lambda: prcr.decode_attention(r, c, 0, q[:, :5].contiguous(), cl, cl),
        lambda: prcr.decode_attention(r, c, 0, q, cl, cl[:2]),
        lambda: prcr.decode_attention(r, paged, 7, q, cl, cl),
        lambda: prcr.decode_attention(r, c, 0, q, cl, cl, scale=float("nan")),
        lambda: prcr.decode_attention(r, c, 0, q, cl, cl, workspace=both),
        lambda: prcr.decode_attention(prcr.Rope(128, (16, 24, 24)), c, 0, q, cl, cl),
        lambda: prcr.decode_attention_static(r, c, 0, q.float(), cl, cl),
    ]
    native = binding._native()
    for i, call in enumerate(bad):
        said = []
        for route in (native, _Declines()):
            monkeypatch.setattr(binding, "_NATIVE", route)
            try:
                call()
                said.append(None)
            except Exception as e:      # noqa: BLE001 - whatever it is, it has to be the same
                said.append((type(e), str(e)))
        assert said[0] == said[1], (i, said)
        assert said[0] is not None, i
    torch.cuda.synchronize()


def test_native_module_declines_what_is_no_tensor_and_leaves_no_error():
    n = binding._native()
    for name, count in (("store_raw", 7), ("reassign_coords", 10), ("rebind_inject", 11), ("revisit", 16),
                        ("prefill_capture", 13), ("decode_attention", 11), ("decode_attention_static", 10)):
        for arg in (None, 1, "pcr", torch.zeros(2, 2), object(), prcr.Rope(64, (8, 12, 12))):
            assert getattr(n, name)(*[arg] * count) is None
        with pytest.raises(TypeError):
            getattr(n, name)(None)
