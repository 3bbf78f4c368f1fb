"""Decode attention where every sequence is one chunk, so that the kernel writes the
outputs without a merge launch, and where workgroups of a split sequence have no keys:
against the float64 oracle.  An output that shares memory with the queries must still be
right (that call keeps the merge launch), as must one whose workspace holds anything.

Tolerance: float32 sums of at most 300 weighted values, relative error 300 * 2^-24 of
max |V| < 6 at these draws: 2e-4 has a margin."""
import numpy as np
import pytest
import torch

import oracle
import paper_2606_26631_amd as prcr
import workloads
from gpu_util import DEV, to_dev

pytestmark = pytest.mark.gpu


# batch x KV heads of 768 and more have one workgroup per sequence and KV head; 2 x 2 has
# many more workgroups than its short sequences have rounds of keys.
@pytest.mark.parametrize("B,H,G,dtype,cap,in_place", [
    (96, 8, 4, "bf16", 300, False), (96, 8, 2, "f32", 300, False), (96, 8, 1, "f32", 300, True),
    (2, 2, 8, "bf16", 9000, False), (2, 2, 2, "f32", 9000, False), (2, 2, 1, "f32", 9000, True)])
def test_decode_chunks_written_or_merged(B, H, G, dtype, cap, in_place):
    D = 64
    g = torch.Generator().manual_seed(B + G)
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    rng = np.random.default_rng(B + G)
    lens = rng.integers(0, 300, B).astype(np.int32)
    lens[0], lens[-1] = 0, 299
    k, v = (torch.randn((B, 1, H, cap, D), generator=g).to(tdt) for _ in range(2))
    q = torch.randn((B, H * G, D), generator=g).to(tdt)
    q_pos = rng.integers(0, 20000, B).astype(np.int32)
    cache = prcr.Cache(k.to(DEV), v.to(DEV))
    rope = prcr.Rope(D, (8, 12, 12), False, 1e6)
    err = torch.zeros(1, dtype=torch.int32, device=DEV)
    need = prcr.decode_workspace_bytes(cache, B, H * G)
    assert (need == B * H * G * (D + 2) * 4) == (B == 96)
    ws = torch.full((need // 4,), float("nan"), device=DEV)
    qd = q.to(DEV)
    print(f"decode direct: {B} x {H} KV heads G={G} {dtype} in place {in_place}", flush=True)
    out = prcr.decode_attention(rope, cache, 0, qd, to_dev(q_pos), to_dev(lens), out=qd if in_place else None,
                                workspace=ws, err=err)
    torch.cuda.synchronize()
    assert int(err.item()) == 0
    npy = workloads.as_numpy_storage
    ref = oracle.decode_attention(rope.__dict__ | {"sections": rope.sections},
                                  {"paged": False, "s_max": cap, "k": npy(k), "v": npy(v)}, 0, npy(q), q_pos,
                                  lens, D ** -0.5, dtype)
    out = out.cpu().numpy()
    assert not out[0].any()
    assert np.abs(out - ref).max() <= 2e-4


# Two waves and four, merges of one wave per head, of four and of sixteen, both element
# types, and calls of one chunk per sequence (which may then not write the output directly).
@pytest.mark.parametrize("B,H,G,dtype,cap", [(5, 2, 4, "bf16", 900), (5, 2, 7, "bf16", 9000), (96, 8, 4, "bf16", 300),
                                             (2, 1, 2, "f32", 9000), (5, 8, 1, "f32", 700)])
def test_output_over_the_lengths(B, H, G, dtype, cap):
    """The lengths lie in the output's own memory: the merge's workgroups write there while
    others still run, so none may read a length.  Same bits as with lengths of their own."""
    D = 64
    g = torch.Generator(device=DEV).manual_seed(B + cap)
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    rnd = lambda *s: torch.randn(s, generator=g, device=DEV).to(tdt)
    cache = prcr.Cache(rnd(B, 1, H, cap, D), rnd(B, 1, H, cap, D))
    q = rnd(B, H * G, D)
    lens = torch.randint(0, min(cap, 300), (B,), generator=g, device=DEV, dtype=torch.int32)
    lens[-1] = cap
    pos = lens.clone()
    rope = prcr.Rope(D, (8, 12, 12), False, 1e6)
    words = prcr.decode_workspace_bytes(cache, B, H * G) // 4
    ref = prcr.decode_attention(rope, cache, 0, q, pos, lens)
    for at in (0, B * H * G * D // 2 - 1, B * H * G * D - B):
        print(f"output over the lengths: {B} x {H} G={G} {dtype} capacity {cap} at {at}", flush=True)
        out = torch.full((B, H * G, D), float("nan"), device=DEV)
        inside = out.view(torch.int32).view(-1)[at:at + B]
        inside.copy_(lens)
        ws = torch.full((words,), float("nan"), device=DEV)
        prcr.decode_attention(rope, cache, 0, q, pos, inside, out=out, workspace=ws)
        torch.cuda.synchronize()
        assert torch.equal(out, ref)
