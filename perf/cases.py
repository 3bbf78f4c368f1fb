"""The work a program has this library do, as cases that can be timed and compared.

A decoder that revisits visual evidence calls the library at four points: it captures the
prompt's keys and values while prefilling (prefill_capture, or store_raw when the model
writes its own cache), it revisits selected visual tokens between decoded text tokens
(reassign_coords + rebind_inject, or the single-launch revisit for small selections), and
it attends over the grown cache at every layer of every decoded token (decode_attention).
Each case is one of these, with its tensors resident on the GPU, called the way the
package's own example calls it.  Shapes are those of workloads.py and bench.py (Qwen-VL
style decoders: 28 layers x 4 KV heads and 36 or 64 layers x 8 KV heads, head_dim 128,
bf16; a small head_dim-64 float32 decoder).
"""
import math
import random

import numpy as np
import torch

import paper_2606_26631_amd as prcr

# Rotary forms: name -> (head_dim, sections, interleaved, theta).
ROPES = {
    "d128_sections": (128, (16, 24, 24), False, 1e6),
    "d128_interleaved": (128, (22, 21, 21), True, 5e6),
    "d128_interleaved_24": (128, (24, 20, 20), True, 5e6),
    "d128_1d": (128, (64, 0, 0), False, 1e6),
    "d64_sections": (64, (8, 12, 12), False, 1e6),
    "d64_interleaved": (64, (11, 11, 10), True, 1e6),
    "d64_1d": (64, (32, 0, 0), False, 1e6),
}
# A drawn case's bounds: the listed paged revisit's traffic and resident bytes.
MOST_BYTES = 1.88e9
MOST_RESIDENT = 14e9


def listed():
    return [
        # The smallest call a program makes: one float32 sequence of a two-layer decoder
        # revisits a 6 x 6 region of a 16 x 16 image.  Launches and host time only.
        dict(name="revisit_tiny_f32", kind="revisit", calls="two", rope="d64_sections",
             dtype="f32", batch=1, layers=2, kv_heads=2, frames=1, grid_h=16, grid_w=16,
             k_lo=36, k_hi=36, len_lo=300, len_hi=300, block=0, key_only=False, mode="pcr"),
        # The paper's efficiency study, smaller end: one sequence of an 8B-class decoder
        # (36 x 8 KV heads) revisits 32 of an image's 768 visual tokens in one launch.
        dict(name="revisit_8b_k32", kind="revisit", calls="one", rope="d128_interleaved_24",
             dtype="bf16", batch=1, layers=36, kv_heads=8, frames=1, grid_h=24, grid_w=32,
             k_lo=32, k_hi=32, len_lo=1024, len_hi=1024, block=0, key_only=False, mode="pcr"),
        # The larger end: 128 tokens at a 32B-class decoder's 64 x 8 KV heads.
        dict(name="revisit_32b_k128", kind="revisit", calls="one", rope="d128_interleaved_24",
             dtype="bf16", batch=1, layers=64, kv_heads=8, frames=1, grid_h=24, grid_w=32,
             k_lo=128, k_hi=128, len_lo=1024, len_hi=1024, block=0, key_only=False, mode="pcr"),
        # Video: 8 sequences revisit 1024 tokens each of 8 frames of 24 x 24.
        dict(name="revisit_video", kind="revisit", calls="two", rope="d128_sections",
             dtype="bf16", batch=8, layers=28, kv_heads=4, frames=8, grid_h=24, grid_w=24,
             k_lo=1024, k_hi=1024, len_lo=4736, len_hi=4736, block=0, key_only=False,
             mode="pcr"),
        # Serving: 32 sequences of mixed length in a paged cache, 512 tokens each.
        dict(name="revisit_paged", kind="revisit", calls="two", rope="d128_sections",
             dtype="bf16", batch=32, layers=28, kv_heads=4, frames=1, grid_h=48, grid_w=48,
             k_lo=512, k_hi=512, len_lo=2400, len_hi=6000, block=16, key_only=False,
             mode="pcr"),
        # One GPU's share of an 8-way split of the KV heads (one head per GPU), with the
        # memory that keeps keys only and finds its values in the prompt's cache slots.
        dict(name="revisit_shard_key_only", kind="revisit", calls="two",
             rope="d128_interleaved", dtype="bf16", batch=32, layers=36, kv_heads=1, frames=1,
             grid_h=64, grid_w=32, k_lo=256, k_hi=256, len_lo=2500, len_hi=4000, block=0,
             key_only=True, mode="pcr"),
        # Prefill of one layer of 36: 8 prompts of 2560 tokens, 2048 of them visual.
        dict(name="prefill_8kv", kind="prefill", rope="d128_interleaved", dtype="bf16",
             batch=8, layers=36, kv_heads=8, frames=1, grid_h=64, grid_w=32, before_lo=256,
             before_hi=256, after_lo=256, after_hi=256, block=0, key_only=False),
        # The same with 4 KV heads, prompts of different lengths and images of odd size,
        # into a paged cache.
        dict(name="prefill_ragged_paged", kind="prefill", rope="d128_sections", dtype="bf16",
             batch=6, layers=28, kv_heads=4, frames=1, grid_h=47, grid_w=35, before_lo=11,
             before_hi=600, after_lo=5, after_hi=300, block=16, key_only=False),
        # Raw-row capture of one layer for a model that writes its own cache.
        dict(name="store_raw", kind="store", rope="d128_interleaved", dtype="bf16", batch=16,
             layers=36, kv_heads=8, frames=1, grid_h=64, grid_w=32, before_lo=256, before_hi=256,
             after_lo=256, after_hi=256, block=0, key_only=False),
        # Decode attention of two layers, 32 sequences, 32 query heads over 8 KV heads.
        dict(name="decode_batch", kind="decode", rope="d128_interleaved", dtype="bf16",
             batch=32, layers=2, kv_heads=8, group=4, len_lo=2756, len_hi=4256, block=0,
             workspace="caller", graph=False),
        # The same over a paged cache: 64 sequences, 28 query heads over 4 KV heads.
        dict(name="decode_paged", kind="decode", rope="d128_sections", dtype="bf16", batch=64,
             layers=2, kv_heads=4, group=7, len_lo=2912, len_hi=6512, block=16,
             workspace="caller", graph=False),
        # One sequence's next token after a revisit: every layer's decode attention, the
        # layers captured in one HIP graph as a decode loop captures them.
        dict(name="decode_one_seq_graph", kind="decode", rope="d128_interleaved_24",
             dtype="bf16", batch=1, layers=36, kv_heads=8, group=4, len_lo=1152, len_hi=1152,
             block=0, workspace="caller", graph=True),
    ]


# ------------------------------------------------------------------ drawn cases
def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _draw_one(rng):
    kind = rng.choice(["revisit", "revisit", "decode", "decode", "prefill", "store"])
    dtype = "f32" if rng.random() < 0.2 else "bf16"
    rope = rng.choice(sorted(r for r in ROPES if ROPES[r][0] == (64 if rng.random() < 0.25 else 128)))
    case = dict(kind=kind, rope=rope, dtype=dtype)
    kv_heads = rng.choice([1, 2, 3, 4, 4, 5, 6, 8, 8, 8])
    block = rng.choice([0, 0, 0, 0, 16, 16, 32, 64, 8, 24])
    if kind == "decode":
        lo = _log_int(rng, 16, 6000)
        case.update(batch=_log_int(rng, 1, 96), layers=_log_int(rng, 1, 36), kv_heads=kv_heads,
                    group=rng.choice([1, 2, 3, 4, 4, 5, 6, 7, 8, 8]), len_lo=lo,
                    len_hi=int(lo * rng.uniform(1.0, 2.5)), block=block,
                    workspace=rng.choice(["caller", "caller", "static"]),
                    graph=rng.random() < 0.3)
        return case
    frames = rng.choice([1, 1, 1, 1, 2, 4, 8])
    gh, gw = _log_int(rng, 6, 64), _log_int(rng, 6, 64)
    case.update(kv_heads=kv_heads, frames=frames, grid_h=gh, grid_w=gw, block=block,
                key_only=rng.random() < 0.25)
    if kind == "revisit":
        most = min(1024, frames * gh * gw)
        hi = _log_int(rng, 4, most)
        lo = max(1, int(hi * rng.choice([1.0, 1.0, 0.6, 0.1])))
        visual = frames * gh * gw
        len_lo = visual + _log_int(rng, 8, 2000)
        case.update(calls="one" if hi <= 128 else "two", batch=_log_int(rng, 1, 64),
                    layers=_log_int(rng, 2, 64), k_lo=lo, k_hi=hi, len_lo=len_lo,
                    len_hi=len_lo + _log_int(rng, 1, 3000),
                    mode=rng.choice(["pcr", "pcr", "pcr", "shift", "lpa", "uir", "identity"]))
    else:
        blo, alo = _log_int(rng, 1, 400), _log_int(rng, 1, 300)
        case.update(batch=_log_int(rng, 1, 32), layers=_log_int(rng, 1, 64), before_lo=blo,
                    before_hi=int(blo * rng.uniform(1.0, 3.0)), after_lo=alo,
                    after_hi=int(alo * rng.uniform(1.0, 3.0)))
    return case


def draw(rng):
    while True:
        case = _draw_one(rng)
        if work(case)["bytes"] <= MOST_BYTES and _resident(case) <= MOST_RESIDENT:
            return case


# ------------------------------------------------------- what a case consists of
def _elem(case):
    return 4 if case["dtype"] == "f32" else 2


def _visual(case):
    return case["frames"] * case["grid_h"] * case["grid_w"]


def _resident(case):
    """Upper bound of a case's resident bytes (memory, caches, projections)."""
    row = case["layers"] * case["kv_heads"] * ROPES[case["rope"]][0] * _elem(case) * 2
    if case["kind"] == "decode":
        return case["batch"] * (case["len_hi"] + 64) * row
    if case["kind"] == "revisit":
        return case["batch"] * (_visual(case) + case["len_hi"] + case["k_hi"] + 64) * row
    tokens = _visual(case) + case["before_hi"] + case["after_hi"]
    return case["batch"] * (_visual(case) + 2 * tokens + 320) * row


def _layout(case):
    """The case's sequence lengths, selections and block tables (host arrays).  They depend
    on the case alone, so that a case's work is the same for every seed; the order of the
    sequences, which tokens are selected and where the blocks lie come from the seed."""
    rng = random.Random(repr(sorted((k, v) for k, v in case.items() if k != "name")))
    B = case["batch"]
    spread = lambda lo, hi: [rng.randint(lo, hi) for _ in range(B)]
    if case["kind"] == "decode":
        return {"lens": spread(case["len_lo"], case["len_hi"])}
    if case["kind"] == "revisit":
        return {"lens": spread(case["len_lo"], case["len_hi"]),
                "ks": spread(case["k_lo"], case["k_hi"])}
    return {"before": spread(case["before_lo"], case["before_hi"]),
            "after": spread(case["after_lo"], case["after_hi"])}


def _blocks(rng, tokens, block):
    """Block table for sequences of `tokens` slots, blocks drawn from one shuffled pool."""
    need = [(n + block - 1) // block for n in tokens]
    pool = rng.permutation(sum(need)).astype(np.int32)
    table = np.full((len(need), max(need)), -1, np.int32)
    at = 0
    for b, n in enumerate(need):
        table[b, :n] = pool[at:at + n]
        at += n
    return table, sum(need)


def _grid(case):
    t, h, w = np.meshgrid(np.arange(case["frames"]), np.arange(case["grid_h"]),
                          np.arange(case["grid_w"]), indexing="ij")
    return np.stack([t.ravel(), h.ravel(), w.ravel()], axis=1).astype(np.int32)


class _Inputs:
    """Tensors of one case and seed, made on the GPU."""

    def __init__(self, case, seed):
        self.case, self.dev = case, torch.device("cuda")
        self.rng = np.random.default_rng([int(seed), 11])
        self.gen = torch.Generator(device=self.dev)
        self.gen.manual_seed(int(seed))
        self.dtype = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
        self.head_dim, self.sections, self.interleaved, self.theta = ROPES[case["rope"]]
        self.build()

    def ints(self, a, dtype=np.int32):
        return torch.from_numpy(np.ascontiguousarray(a, dtype=dtype)).to(self.dev)

    def normal(self, *shape):
        return torch.randn(shape, generator=self.gen, device=self.dev, dtype=self.dtype)

    def keys(self, shape, head_axis):
        """Keys ~ N(0, 1) with four channels per KV head eight times as large, as the keys
        of rotary decoders have outlier channels."""
        k = self.normal(*shape)
        H, D = self.case["kv_heads"], self.head_dim
        scale = torch.ones(H, D, dtype=self.dtype)
        for h in range(H):
            scale[h, self.rng.choice(D, 4, replace=False).tolist()] = 8.0
        view = [1] * len(shape)
        view[head_axis], view[-1] = H, D
        return k.mul_(scale.to(self.dev).view(view))

    def cache(self, tokens):
        """Contiguous or paged cache with room for `tokens` slots per sequence."""
        c, D = self.case, self.head_dim
        B, NL, H = c["batch"], c["layers"], c["kv_heads"]
        self.table = None
        if c["block"]:
            table, n_blocks = _blocks(self.rng, tokens, c["block"])
            shape, head_axis = (NL, n_blocks, c["block"], H, D), 3
            self.table_host, self.table = table, self.ints(table)
        else:
            shape, head_axis = (B, NL, H, max(tokens) + 32, D), 2
        self.cache_k = self.keys(shape, head_axis)
        self.cache_v = self.normal(*shape)

    def build(self):
        c, D = self.case, self.head_dim
        B, NL, H = c["batch"], c["layers"], c["kv_heads"]
        lay = _layout(c)
        order = self.rng.permutation(B)
        if c["kind"] == "decode":
            lens = np.array(lay["lens"])[order]
            self.cache(lens.tolist())
            self.lens = lens
            self.cache_len, self.q_pos = self.ints(lens), self.ints(lens)
            self.q = self.normal(NL, B, H * c["group"], D)
            return
        M = _visual(c)
        coords = np.broadcast_to(_grid(c), (B, M, 3)).copy()
        if c["kind"] == "revisit":
            lens, ks = np.array(lay["lens"])[order], np.array(lay["ks"])[order]
            self.lens = lens
            sel = [np.sort(self.rng.choice(M, size=int(k), replace=False)) for k in ks]
            self.off_host = np.concatenate([[0], np.cumsum(ks)]).astype(np.int32)
            self.sel_host = np.concatenate(sel).astype(np.int32)
            self.sel_off, self.sel_idx = self.ints(self.off_host), self.ints(self.sel_host)
            self.coords = self.ints(coords)
            self.n_visual = self.ints(np.full(B, M))
            self.p_txt_host = lens - 1
            self.p_txt, self.cache_len = self.ints(lens - 1), self.ints(lens)
            self.mem_k = self.keys((B, M, NL, H, D), 3)
            self.mem_v = self.v_slot = None
            if c["key_only"]:
                self.slot_host = np.broadcast_to(
                    np.minimum(64, lens - M)[:, None] + np.arange(M)[None, :], (B, M)).copy()
                self.v_slot = self.ints(self.slot_host)
            else:
                self.mem_v = self.normal(B, M, NL, H, D)
            self.cache((lens + ks).tolist())
            return
        # Prefill and raw-row capture: text, one image (or video), text.
        before, after = np.array(lay["before"])[order], np.array(lay["after"])[order]
        n_tok = before + M + after
        S = int(n_tok.max())
        pos = np.zeros((B, S, 3), np.int32)
        vis = np.full((B, S), -1, np.int32)
        g = coords[0]
        for b in range(B):
            i, j, n = int(before[b]), int(before[b]) + M, int(n_tok[b])
            pos[b, :i] = np.arange(i)[:, None]
            pos[b, i:j] = i + g
            pos[b, j:n] = i + int(g.max()) + 1 + np.arange(n - j)[:, None]
            vis[b, i:j] = np.arange(M)
        self.n_tok, self.pos_host, self.before = n_tok, pos, before
        self.raw_k, self.raw_v = self.keys((B, S, H, D), 2), self.normal(B, S, H, D)
        self.n_visual = self.ints(np.full(B, M))
        self.mem_k = torch.zeros(B, M, NL, H, D, dtype=self.dtype, device=self.dev)
        self.mem_v = None if c["key_only"] else torch.zeros_like(self.mem_k)
        self.v_slot = torch.zeros(B, M, dtype=torch.int32, device=self.dev) if c["key_only"] else None
        self.layer = NL // 2
        if c["kind"] == "store":
            self.coords = self.ints(coords)
            self.vis_rows = self.ints(before[:, None] + np.arange(M)[None, :])
        else:
            self.coords = torch.zeros(B, M, 3, dtype=torch.int32, device=self.dev)
            self.pos, self.vis, self.n_tokens = self.ints(pos), self.ints(vis), self.ints(n_tok)
            self.start = torch.zeros(B, dtype=torch.int32, device=self.dev)
            self.cache((n_tok + 256).tolist())


def prepare(case, seed):
    x = _Inputs(case, seed)
    state = {"case": case, "x": x,
             "rope": prcr.Rope(x.head_dim, x.sections, x.interleaved, x.theta)}
    if case["kind"] != "decode":
        state["mem"] = prcr.Memory(x.mem_k, x.mem_v, x.coords, x.n_visual, x.v_slot)
    if case["kind"] != "store":
        state["cache"] = prcr.Cache(x.cache_k, x.cache_v, x.table)
    if case["kind"] == "decode" and case["graph"]:
        _decode(state, 1)            # the library's code is loaded before the capture
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            outs = _decode(state, case["layers"])
        state["graph"], state["outs"] = graph, outs
    return state


def _decode(state, layers):
    x = state["x"]
    call = (prcr.decode_attention_static if state["case"]["workspace"] == "static"
            else prcr.decode_attention)
    return [call(state["rope"], state["cache"], layer, x.q[layer], x.q_pos, x.cache_len)
            for layer in range(layers)]


def run(state):
    c, x = state["case"], state["x"]
    if c["kind"] == "decode":
        if c["graph"]:
            state["graph"].replay()
            return state["outs"]
        return _decode(state, c["layers"])
    rope, mem = state["rope"], state["mem"]
    if c["kind"] == "store":
        prcr.store_raw(mem, x.layer, x.raw_k, x.raw_v, x.vis_rows)
        return [x.mem_k, x.mem_v]
    cache = state["cache"]
    if c["kind"] == "prefill":
        prcr.prefill_capture(rope, mem, x.layer, x.raw_k, x.raw_v, x.pos, x.n_tokens, x.vis,
                             cache, x.start)
        return [x.cache_k, x.cache_v, x.mem_k, x.mem_v, x.coords, x.v_slot]
    if c["calls"] == "one":
        new_pos, next_pos, new_len, slots = prcr.revisit(
            rope, mem, x.sel_off, x.sel_idx, x.p_txt, cache, x.cache_len, c["mode"], 2)
    else:
        new_pos, next_pos = prcr.reassign_coords(mem, x.sel_off, x.sel_idx, x.p_txt, c["mode"], 2)
        new_len, slots = prcr.rebind_inject(rope, mem, x.sel_off, x.sel_idx, new_pos, cache,
                                            x.cache_len)
    return [x.cache_k, x.cache_v, new_pos, next_pos, new_len, slots]


# --------------------------------------------------------------- work, tolerance
def work(case):
    D, s, H = ROPES[case["rope"]][0], _elem(case), case["kv_heads"]
    lay = _layout(case)
    if case["kind"] == "decode":
        keys, B, Hq, NL = sum(lay["lens"]), case["batch"], H * case["group"], case["layers"]
        table = sum(-(-n // case["block"]) for n in lay["lens"]) * 4 if case["block"] else 0
        return {"bytes": NL * (keys * H * D * 2 * s + B * Hq * D * (s + 4) + table + 8 * B),
                "flops": NL * keys * Hq * D * 4}
    if case["kind"] == "revisit":
        k = sum(lay["ks"])
        # rows in and out, then per token its index, coordinates, position and slot
        return {"bytes": k * case["layers"] * H * D * 4 * s + k * (4 + 12 + 24 + 8),
                "flops": k * case["layers"] * H * D * 3}
    visual = case["batch"] * _visual(case)
    keep = 1 if case["key_only"] else 2
    if case["kind"] == "store":
        return {"bytes": visual * H * D * s * 2 * keep + visual * 4, "flops": 0}
    rows = sum(lay["before"]) + sum(lay["after"]) + visual
    return {"bytes": (rows * 4 + visual * keep) * H * D * s + rows * 16 + visual * 12,
            "flops": rows * H * D * 3}


def tolerance(case):
    if case["kind"] == "store":
        return "exact"
    if case["kind"] == "decode":
        return {"rel": 2e-6, "max": 2e-5}
    if case["dtype"] == "f32":
        return {"rel": 2e-7, "max": 5e-7}
    # keys are rounded once to bf16: half a unit in the last place from the exact value
    return {"rel": 3e-3, "max": 8e-3}


# ------------------------------------------------------------- 64-bit reference
def _axis(x, device):
    i = np.arange(x.head_dim // 2)
    st, sh, sw = x.sections
    if x.interleaved:
        a = np.where((i % 3 == 1) & (i < 3 * sh), 1, np.where((i % 3 == 2) & (i < 3 * sw), 2, 0))
    else:
        a = np.where(i < st, 0, np.where(i < st + sh, 1, 2))
    return torch.from_numpy(a).to(device)


def _angles(x, pos):
    """Angles of every rotary pair at positions pos [..., 3] (float64)."""
    D = x.head_dim
    inv = x.theta ** (-2.0 * torch.arange(D // 2, dtype=torch.float64, device=x.dev) / D)
    return pos.double()[..., _axis(x, x.dev)] * inv


def _rotate(rows, ang):
    lo, hi = rows.double().chunk(2, dim=-1)
    cs, sn = ang.cos(), ang.sin()
    return torch.cat([lo * cs - hi * sn, hi * cs + lo * sn], dim=-1)


def _new_positions(case, coords, p_txt):
    """Positions of one sequence's selected tokens (float64) and its next text position."""
    K, L = len(coords), 2
    p, c = float(p_txt), coords.astype(np.float64)
    lo, hi = c.min(0), c.max(0)
    j = np.arange(1, K + 1)[:, None]
    mode = case["mode"]
    if mode == "identity":
        return c, p_txt + 1
    if mode == "shift":
        return p + 1 + (c - lo), p_txt + 2 + int((hi - lo).max())
    if mode == "lpa":
        return np.broadcast_to(p + j, (K, 3)), p_txt + K + 1
    if mode == "uir":
        return np.broadcast_to(p + j / (K + 1), (K, 3)), p_txt + 1
    u = np.where(hi > lo, (c - lo) / np.maximum(hi - lo, 1), 0.5)
    return (p - L) + (L + 1) * (1 + (K - 1) * u) / (K + 1), p_txt + 1


def exact(case, seed):
    x = _Inputs(case, seed)
    c, B, NL, H = case, case["batch"], case["layers"], case["kv_heads"]
    bs = c["block"]

    def pool(b, slots):
        """Slots of sequence b as (block, offset) of the paged pool."""
        slots = np.asarray(slots)
        return (torch.from_numpy(x.table_host[b, slots // bs].astype(np.int64)).to(x.dev),
                torch.from_numpy(slots % bs).to(x.dev))

    if c["kind"] == "decode":
        if sum(x.lens) * H * c["group"] * NL > 2e8:
            return None
        outs = []
        pos = x.q_pos.double()[:, None].expand(B, 3)
        ang = _angles(x, pos)[:, None, :]
        for layer in range(NL):
            q = _rotate(x.q[layer], ang) * x.head_dim ** -0.5
            rows = []
            for b in range(B):
                n = int(x.lens[b])
                if bs:
                    blk, off = pool(b, np.arange(n))
                    k, v = (t[layer][blk, off].permute(1, 0, 2).contiguous().double()
                            for t in (x.cache_k, x.cache_v))
                else:
                    k, v = (t[b, layer, :, :n].double() for t in (x.cache_k, x.cache_v))
                s = torch.matmul(q[b].view(H, c["group"], -1), k.transpose(1, 2).contiguous())
                rows.append(torch.matmul(s.softmax(-1), v).reshape(H * c["group"], -1))
            outs.append(torch.stack(rows))
        return outs
    if c["kind"] == "store":
        out = [x.mem_k.double(), None if x.mem_v is None else x.mem_v.double()]
        for b in range(B):
            i = int(x.before[b])
            out[0][b, :, x.layer] = x.raw_k[b, i:i + _visual(c)].double()
            if out[1] is not None:
                out[1][b, :, x.layer] = x.raw_v[b, i:i + _visual(c)].double()
        return out
    ck, cv = x.cache_k.double(), x.cache_v.double()
    if c["kind"] == "prefill":
        mk = x.mem_k.double()
        mv = None if x.mem_v is None else x.mem_v.double()
        coords, v_slot = x.coords.clone(), None if x.v_slot is None else x.v_slot.clone()
        for b in range(B):
            n, i, M = int(x.n_tok[b]), int(x.before[b]), _visual(c)
            k = _rotate(x.raw_k[b, :n], _angles(x, x.pos[b, :n])[:, None, :])
            v = x.raw_v[b, :n].double()
            if bs:
                blk, off = pool(b, np.arange(n))
                ck[x.layer][blk, off], cv[x.layer][blk, off] = k, v
            else:
                ck[b, x.layer, :, :n], cv[b, x.layer, :, :n] = k.transpose(0, 1), v.transpose(0, 1)
            mk[b, :, x.layer] = x.raw_k[b, i:i + M].double()
            if mv is not None:
                mv[b, :, x.layer] = x.raw_v[b, i:i + M].double()
            else:
                v_slot[b] = torch.arange(i, i + M, dtype=torch.int32, device=x.dev)
            coords[b] = x.pos[b, i:i + M]
        return [ck, cv, mk, mv, coords, v_slot]
    grid = _grid(c)
    pos, nxt, slots = [], [], []
    for b in range(B):
        s0, s1, n = int(x.off_host[b]), int(x.off_host[b + 1]), int(x.lens[b])
        m = x.sel_host[s0:s1]
        p, q = _new_positions(c, grid[m], int(x.p_txt_host[b]))
        pos.append(p)
        nxt.append(q)
        at = n + np.arange(s1 - s0)
        mi = torch.from_numpy(m.astype(np.int64)).to(x.dev)
        ang = _angles(x, torch.from_numpy(np.ascontiguousarray(p)).to(x.dev))[:, None, None, :]
        k = _rotate(x.mem_k[b][mi], ang)                      # [K, NL, H, D]
        if bs:
            blk, off = pool(b, at)
            if x.mem_v is None:
                vb, vo = pool(b, x.slot_host[b][m])
                v = x.cache_v[:, vb, vo].double()             # [NL, K, H, D]
            else:
                v = x.mem_v[b][mi].double().transpose(0, 1)
            ck[:, blk, off], cv[:, blk, off] = k.transpose(0, 1), v
            slots.append(x.table_host[b, at // bs].astype(np.int64) * bs + at % bs)
        else:
            if x.mem_v is None:
                v = x.cache_v[b][:, :, torch.from_numpy(x.slot_host[b][m].astype(np.int64)).to(x.dev)].double()
            else:
                v = x.mem_v[b][mi].double().permute(1, 2, 0, 3)
            ck[b, :, :, n:n + s1 - s0], cv[b, :, :, n:n + s1 - s0] = k.permute(1, 2, 0, 3), v
            slots.append(b * x.cache_k.shape[3] + at)
    new_len = x.lens + np.diff(x.off_host)
    return [ck, cv, torch.from_numpy(np.concatenate(pos)).to(x.dev), x.ints(nxt), x.ints(new_len),
            x.ints(np.concatenate(slots), np.int64)]
