"""A NaN key or query makes its head's output NaN in decode attention, as it does in the
float64 oracle, however the call is split: one chunk per sequence, written without a merge;
chunks merged by one wave per head and by several; bf16 and float32.  Sequences and heads
without a NaN are as if there were none, and an empty sequence is zero.

Tolerance of the finite outputs: float32 sums of at most 700 weighted values, relative error
700 * 2^-24 of max |V| < 6 at these draws: 4e-4 has a margin."""
import numpy as np
import pytest
import torch

import oracle
import paper_2606_26631_amd as prcr
import workloads
from gpu_util import DEV, to_dev

pytestmark = pytest.mark.gpu


# 64 x 4 sequences and KV heads of at most 700 slots are one chunk each (bf16), three for
# float32; 100 x 8 are one for both; the others are merged from up to 7 and up to 64 chunks.
@pytest.mark.parametrize("B,H,G,dtype,cap,bs", [
    (64, 4, 7, "bf16", 700, 0), (64, 4, 2, "f32", 700, 0), (100, 8, 4, "bf16", 700, 16), (100, 8, 1, "f32", 300, 0),
    (4, 8, 4, "bf16", 700, 16), (4, 8, 8, "bf16", 4096, 0), (4, 3, 2, "f32", 700, 24)])
def test_nan_keys_and_queries_reach_the_output(B, H, G, dtype, cap, bs):
    D = 64
    g = torch.Generator().manual_seed(B + G + cap)
    rng = np.random.default_rng(B + H + G)
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    rnd = lambda *s: torch.randn(s, generator=g).to(tdt)
    most = min(cap, 700)
    lens = rng.integers(2, most, B).astype(np.int32)
    lens[0], lens[1], lens[2], lens[3] = most - 1, 0, most - 100, 5
    if bs:
        per = -(-cap // bs)
        table = rng.permutation(B * per).astype(np.int32).reshape(B, per)
        k, v = rnd(1, B * per, bs, H, D), rnd(1, B * per, bs, H, D)
        at = lambda b, h, j: k[0, table[b, j // bs], j % bs, h]
        co = {"paged": True, "block_size": bs, "block_table": table, "max_blocks": per, "n_blocks": B * per}
        dev_table = to_dev(table)
    else:
        k, v = rnd(B, 1, H, cap, D), rnd(B, 1, H, cap, D)
        at = lambda b, h, j: k[b, 0, h, j]
        co, dev_table = {"paged": False, "s_max": cap}, None
    q = rnd(B, H * G, D)
    at(0, 1, int(lens[0]) - 1)[11] = float("nan")          # one key of the longest sequence
    for j in range(5):
        at(3, H - 1, j)[:] = float("nan")                  # every key of a short one
    q[2, 0, 3] = float("nan")                              # a query
    cache = prcr.Cache(k.to(DEV), v.to(DEV), dev_table)
    rope = prcr.Rope(D, (8, 12, 12), False, 1e6)
    q_pos = rng.integers(0, 20000, B).astype(np.int32)
    print(f"decode NaN: {B} x {H} KV heads G={G} {dtype} capacity {cap} block {bs}", flush=True)
    out = prcr.decode_attention(rope, cache, 0, q.to(DEV), to_dev(q_pos), to_dev(lens))
    torch.cuda.synchronize()
    out = out.cpu().numpy()
    npy = workloads.as_numpy_storage
    co["k"], co["v"] = npy(k), npy(v)
    ref = oracle.decode_attention(rope.__dict__ | {"sections": rope.sections}, co, 0, npy(q), q_pos, lens,
                                  D ** -0.5, dtype)
    assert np.isnan(ref).sum() == (2 * G + 1) * D
    assert np.array_equal(np.isnan(out), np.isnan(ref))
    assert not out[1].any()
    fine = ~np.isnan(ref)
    assert np.abs(out[fine] - ref[fine]).max() <= 4e-4
