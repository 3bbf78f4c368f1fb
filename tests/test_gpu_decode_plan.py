"""How decode attention splits a call must not show in its results: lengths on both sides of
every line of the plan (one chunk or several by the chunk's 512 or 256 keys, workgroups of two or
four waves by the cache's capacity, splits without keys), with workgroup counts that do and
do not fill the chip's 256 compute units, and batches that the workgroups order by length in
each of the ways they do, against the float64 oracle.

Tolerance: as in test_gpu_attention.py, float32 sums of values of at most max |V|."""
import numpy as np
import pytest
import torch

import oracle
import paper_2606_26631_amd as prcr
import workloads
from gpu_util import DEV, to_dev

pytestmark = pytest.mark.gpu

# (sequences, KV heads, query heads per KV head, capacity, block size, lengths)
CASES = [
    (1, 8, 4, 2048, 0, (2048,)),                      # 256 chunks of 64 keys: two waves
    (1, 8, 4, 2112, 0, (2048,)),                      # one more: four
    (1, 1, 5, 16384, 16, (16001,)),                   # two waves, paged, 256 splits
    (3, 2, 7, 700, 24, (700, 1, 65)),                 # two waves, entries per key
    (64, 4, 7, 1040, 16, (1022, 1023, 1024, 1025, 1026, 511, 512, 513)),   # one or two chunks of 256
    (40, 4, 2, 1700, 0, (1535, 1536, 1537, 1023, 1025, 200)),              # 160 pairs: uneven rounds
    (33, 6, 8, 1100, 8, (1024, 1025, 1100, 0)),                            # 198 pairs
    (32, 8, 1, 1100, 0, (511, 512, 513, 1100, 257, 0)),                    # one head: two chunks from 512 keys
    (16, 8, 2, 2100, 16, (2049, 1023, 1025, 900, 130, 64)),                # two heads: four or two chunks
    (70, 3, 3, 1300, 0, (1200, 1300, 513, 64)),                            # more than 64 sequences, one chunk
    # More than 64 sequences (taken in their own order) in several chunks, with a second
    # round of workgroups, whose rows go in reverse, inside the grid.
    (100, 1, 4, 1700, 0, (1700, 1650, 900, 513, 0)),                       # five chunks of 340
    (70, 3, 7, 1600, 16, (1600, 1537, 1000, 511, 0)),                      # three, the last reversed
    (130, 2, 4, 2200, 24, (2200, 1600, 1025, 1024, 700)),                  # three, the second reversed
    # Workgroups of two waves that rank many sequences: up to 32 each wave alone, beyond
    # that the two waves half of them each; lengths that tie, empty sequences.
    (17, 1, 4, 900, 0, (900, 900, 513, 0, 0)),
    (32, 1, 8, 512, 16, (512, 512, 511, 0, 0, 0)),
    (33, 1, 4, 256, 0, (256, 256, 255, 0, 0, 33, 33)),
    (40, 1, 7, 256, 8, (256, 256, 130, 0, 0, 33, 33)),
    (64, 1, 2, 256, 16, (256, 256, 255, 0, 0, 65, 65)),
]


@pytest.mark.parametrize("B,H,G,cap,bs,some", CASES)
def test_decode_result_does_not_show_the_plan(B, H, G, cap, bs, some):
    D = 64
    rng = np.random.default_rng(B + H + cap)
    lens = rng.integers(0, 40, B).astype(np.int32)
    lens[rng.choice(B, min(B, len(some)), replace=False)] = some
    g = torch.Generator().manual_seed(cap + G)
    rnd = lambda *s: torch.randn(s, generator=g).to(torch.bfloat16)
    if bs:
        per = (cap + bs - 1) // bs
        table = rng.permutation(B * per).astype(np.int32).reshape(B, per)
        k, v = rnd(1, B * per, bs, H, D), rnd(1, B * per, bs, H, D)
        co = {"paged": True, "block_size": bs, "block_table": table, "max_blocks": per, "n_blocks": B * per}
        cache = prcr.Cache(k.to(DEV), v.to(DEV), to_dev(table))
    else:
        k, v = rnd(B, 1, H, cap, D), rnd(B, 1, H, cap, D)
        co = {"paged": False, "s_max": cap}
        cache = prcr.Cache(k.to(DEV), v.to(DEV))
    q, q_pos = rnd(B, H * G, D), rng.integers(0, 20000, B).astype(np.int32)
    rope = prcr.Rope(D, (8, 12, 12), False, 1e6)
    ws = torch.full((prcr.decode_workspace_bytes(cache, B, H * G) // 4,), float("nan"), device=DEV)
    print(f"decode plan: {B} x {H} KV heads, G={G}, capacity {cap}, block {bs}", flush=True)
    args = (rope, cache, 0, q.to(DEV), to_dev(q_pos), to_dev(lens))
    out = prcr.decode_attention(*args, workspace=ws)
    same = prcr.decode_attention_static(*args)
    torch.cuda.synchronize()
    assert torch.equal(out, same)
    out = out.cpu().numpy()
    npy = workloads.as_numpy_storage
    co["k"], co["v"] = npy(k), npy(v)
    ref = oracle.decode_attention(rope.__dict__ | {"sections": rope.sections}, co, 0, npy(q), q_pos, lens,
                                  D ** -0.5, "bf16")
    vmax = float(v.float().abs().max())
    assert np.abs(out - ref).max() <= 5e-5 * vmax + 1e-6
