"""Decode attention of bf16 caches at the edges of its tiles of 32 keys, against the
float64 oracle: lengths around one tile, one round of a workgroup's tiles and several
rounds, groups that fill the kernel's 4 or 8 heads and groups that do not, both head
dims, contiguous caches, blocks of whole half tiles (16, 48) and other blocks (8, 5).
Every slot past a sequence's length holds NaN, and one sequence has an infinite value
under a key with weight: its feature must come out infinite and no other may change.

Tolerance: scores and weights are float32 sums of exact products (three bf16 parts of
each query element and weight), at most 512 terms deep before the float32 merges, each
with relative error 2^-24: |out - ref| <= 5e-5 * max |V| + 1e-6 has a wide margin.  Over
all outputs the rounding averages out to a few 2^-24 (5e-7 measured), and a query or
weight that lost the last of its three parts is 2^-17 = 8e-6 off: 2e-6 tells them apart."""
import numpy as np
import pytest
import torch

import oracle
import paper_2606_26631_amd as prcr
import workloads
from gpu_util import DEV, to_dev

pytestmark = pytest.mark.gpu

LENS = np.array([1, 15, 16, 17, 31, 32, 33, 64, 127, 128, 129, 160, 255, 257, 700, 0], np.int32)
CASES = [(128, 4, 0), (128, 8, 0), (128, 5, 16), (128, 3, 48), (128, 7, 8), (128, 1, 5),
         (64, 4, 16), (64, 6, 0), (64, 8, 8), (64, 2, 0)]


@pytest.mark.parametrize("D,G,bs", CASES)
def test_decode_tile_edges(D, G, bs):
    B, NL, H, layer = len(LENS), 2, 3, 1
    g = torch.Generator().manual_seed(10 * D + G + bs)
    rng = np.random.default_rng(D + G + bs)
    rows = lambda n: torch.randn((n, H, D), generator=g).to(torch.bfloat16)
    if bs:
        need = -(-LENS // bs)
        n_blocks = int(need.sum()) + 2
        perm = rng.permutation(n_blocks).astype(np.int32)
        table = np.full((B, int(need.max())), -1, np.int32)
        shape, at = (NL, n_blocks, bs, H, D), 0
        for b in range(B):
            table[b, :need[b]] = perm[at:at + need[b]]
            at += need[b]
        table[table < 0] = perm[-1]
        cache_o = {"paged": True, "block_size": bs, "block_table": table,
                   "max_blocks": table.shape[1], "n_blocks": n_blocks}
    else:
        table, cap = None, int(LENS.max()) + 5
        shape, cache_o = (B, NL, H, cap, D), {"paged": False, "s_max": cap}
    k = torch.full(shape, float("nan"), dtype=torch.bfloat16)
    v = k.clone()
    for b in range(B):
        n = int(LENS[b])
        kr, vr = rows(n), rows(n)
        if b == 8:
            vr[n // 2, 0, 7] = float("inf")
        if bs:
            j = np.arange(n)
            k[layer, table[b, j // bs], j % bs], v[layer, table[b, j // bs], j % bs] = kr, vr
        else:
            k[b, layer, :, :n], v[b, layer, :, :n] = kr.transpose(0, 1), vr.transpose(0, 1)
    # slot 0 of the layer stands in for dead keys: it must not reach any result either
    cache_o["k"], cache_o["v"] = workloads.as_numpy_storage(k), workloads.as_numpy_storage(v)
    q = torch.randn((B, H * G, D), generator=g).to(torch.bfloat16)
    q_pos = rng.integers(0, 20000, B).astype(np.int32)
    print(f"decode tile edges: D={D} G={G} block {bs}", flush=True)
    cache = prcr.Cache(k.to(DEV), v.to(DEV), None if table is None else to_dev(table))
    rope = prcr.Rope(D, (8, 12, 12) if D == 64 else (16, 24, 24), False, 1e6)
    err = torch.zeros(1, dtype=torch.int32, device=DEV)
    out = prcr.decode_attention(rope, cache, layer, q.to(DEV), to_dev(q_pos), to_dev(LENS), err=err)
    torch.cuda.synchronize()
    assert int(err.item()) == 0
    out = out.cpu().numpy()
    ref = oracle.decode_attention(rope.__dict__ | {"sections": rope.sections}, cache_o, layer,
                                  workloads.as_numpy_storage(q), q_pos, LENS, D ** -0.5, "bf16")
    assert np.array_equal(np.isinf(out), np.isinf(ref)) and np.isinf(ref).sum() == G
    assert not out[-1].any()
    fine = np.isfinite(ref)
    assert np.isfinite(out[fine]).all()
    assert np.abs(out[fine] - ref[fine]).max() <= 5e-5 * 6 + 1e-6      # |V| < 6 at these draws
    assert np.linalg.norm(out[fine] - ref[fine]) <= 2e-6 * np.linalg.norm(ref[fine])
