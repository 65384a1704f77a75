"""The work that users of this framework have it do, as cases to measure.

A case is one call (or one decode step) through the public entry points:

  attention   one layer's paged decode attention over scattered local blocks
  swap-in     one layer group's prefetch: scattered slice blocks into staging
  swap-out    staged blocks written back to scattered slice slots
  step        a decode step over some layers of a paged cache: per layer group
              the prefetch, per layer append and attention, then the group's
              write-back
  slab-step   the same step on a slab-managed slice (swaps of whole slabs,
              attention; half of the slabs in the used range set aside)
  reclaim     the lender takes blocks back and lends them again: reclaim with
              table rewrite, lend, allocation, migration into the slice, free

Sequence lengths are evenly spaced quantiles of the case's distribution in a
seeded order, so the work of a case does not depend on the seed; placements,
values and queries do. The shapes are those of ``synth/configs.py`` (a tiny
MHA cache, an 8B-shaped GQA cache, one GPU's share of a 70B-shaped cache, the
copy stress block sizes) and generic ones around them.
"""
import math
import statistics

import numpy as np
import torch

from paper_2609_27040_amd import ema
from paper_2609_27040_amd.kvcache import PagedKVCache, SlabKVCache

D = 128
DT = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}
LAYOUT = {"attn": ema.LAYOUT_ATTN, "nhd": ema.LAYOUT_NHD}
LARGEST = 1.3e9          # bytes of a drawn case at most


def listed():
    return [
        # one layer of the tiny MHA cache: the smallest call, all latency
        {"name": "attention-tiny", "kind": "attention", "q_heads": 8, "kv_heads": 8, "block": 16,
         "dtype": "f16", "out": "f32", "batch": 8, "dist": "uniform", "lo": 64, "hi": 512},
        # one layer of an 8B-shaped decode batch: the ordinary call
        {"name": "attention-8b", "kind": "attention", "q_heads": 32, "kv_heads": 8, "block": 16,
         "dtype": "bf16", "out": "f32", "batch": 64, "dist": "uniform", "lo": 1024, "hi": 4096},
        # one GPU's share of a 70B-shaped layer: one KV head, very unequal lengths
        {"name": "attention-70b-share", "kind": "attention", "q_heads": 8, "kv_heads": 1,
         "block": 32, "dtype": "bf16", "out": "bf16", "batch": 128, "dist": "lognormal",
         "lo": 128, "hi": 16384},
        # a large batch of short chats
        {"name": "attention-chats", "kind": "attention", "q_heads": 32, "kv_heads": 8, "block": 16,
         "dtype": "bf16", "out": "bf16", "batch": 512, "dist": "uniform", "lo": 17, "hi": 1000},
        # a few long documents
        {"name": "attention-long", "kind": "attention", "q_heads": 32, "kv_heads": 8, "block": 16,
         "dtype": "bf16", "out": "bf16", "batch": 4, "dist": "uniform", "lo": 20001, "hi": 120001},
        # a group of four 8B-shaped layers, 30 % in the slice, swapped in
        {"name": "swap-in-8b", "kind": "swap-in", "kv_heads": 8, "block": 16, "layout": "attn",
         "blocks": 9801},
        # the same bytes from a token-major slice at a larger block size
        {"name": "swap-in-token-major", "kind": "swap-in", "kv_heads": 8, "block": 64,
         "layout": "nhd", "blocks": 2401},
        # staged blocks back to a token-major slice
        {"name": "swap-out-token-major", "kind": "swap-out", "kv_heads": 8, "block": 16,
         "layout": "nhd", "blocks": 6001},
        # a decode step of a lightly loaded server
        {"name": "step-small", "kind": "step", "q_heads": 32, "kv_heads": 8, "block": 16,
         "dtype": "bf16", "out": "bf16", "layout": "attn", "batch": 3, "dist": "uniform",
         "lo": 100, "hi": 900, "layers": 8, "group": 4, "slice": 0.3},
        # four layers of the 8B-shaped decode step with append and write-back
        {"name": "step-8b", "kind": "step", "q_heads": 32, "kv_heads": 8, "block": 16,
         "dtype": "bf16", "out": "bf16", "layout": "attn", "batch": 64, "dist": "uniform",
         "lo": 1024, "hi": 4096, "layers": 4, "group": 4, "slice": 0.3},
        # a decode step on a slab-managed slice
        {"name": "slab-step", "kind": "slab-step", "q_heads": 32, "kv_heads": 8, "block": 16,
         "dtype": "bf16", "out": "bf16", "layout": "attn", "batch": 16, "dist": "uniform",
         "lo": 1024, "hi": 4096, "layers": 4, "group": 2, "slice": 0.3, "slab": 10},
        # the lender takes a tenth of its blocks back, and lends them again
        {"name": "reclaim", "kind": "reclaim", "kv_heads": 8, "block": 16, "layout": "attn",
         "batch": 64, "dist": "uniform", "lo": 1024, "hi": 4096, "layers": 4, "slice": 0.3,
         "share": 0.1},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["attention"] * 5 + ["swap-in", "swap-in", "swap-out", "step", "slab-step",
                                           "reclaim"])
    c = {"kind": kind}
    c["kv_heads"] = rng.choice([1, 2, 4, 8])
    if kind in ("swap-in", "swap-out"):
        c["block"] = rng.choice([16, 32, 64, 256])
        c["layout"] = rng.choice(["attn", "nhd"])
        c["blocks"] = _log(rng, 3, min(20000, LARGEST / (2 * _block_bytes(c))))
        return c
    c["block"] = rng.choice([16, 16, 32, 64])
    c["dist"] = "uniform"
    if kind == "reclaim":
        c["layout"] = rng.choice(["attn", "attn", "nhd"])
        c["layers"] = rng.choice([2, 4])
        c["slice"] = rng.choice([0.3, 0.5])
        c["share"] = rng.choice([0.01, 0.05, 0.25])
    else:
        c["q_heads"] = c["kv_heads"] * rng.choice([1, 4, 4, 8, 16])
        c["dtype"] = rng.choice(["bf16", "bf16", "f16"])
        c["out"] = rng.choice(["f32", c["dtype"]])
    if kind in ("step", "slab-step"):
        c["layout"] = "attn" if kind == "slab-step" else rng.choice(["attn", "nhd"])
        c["layers"], c["group"] = rng.choice([(2, 1), (4, 2), (4, 4)])
        c["slice"] = rng.choice([0.3, 0.5])
        if kind == "slab-step":
            c["slab"] = rng.choice([1, 10, 30])
    if kind == "attention" and rng.random() < 0.25:
        c["dist"], c["lo"], c["hi"] = "lognormal", 128, 16384
        c["batch"] = _log(rng, 4, 128)
    else:
        c["batch"] = _log(rng, 1, 512 if kind == "attention" else 64)
        c["hi"] = _log(rng, 33, 120000 if kind == "attention" else 4096)
        c["lo"] = 1 + int(c["hi"] * rng.choice([0.02, 0.25, 0.9]))
    while work(c)["bytes"] > LARGEST:
        if c["batch"] > 1:
            c["batch"] = max(1, c["batch"] * 2 // 3)
        else:
            c["hi"] = c["hi"] // 2
            c["lo"] = min(c["lo"], c["hi"])
    return c


def _block_bytes(case):
    return 2 * case["block"] * case["kv_heads"] * D * 2


def _quantiles(case):
    n = case["batch"]
    q = (np.arange(n) + 0.5) / n
    if case["dist"] == "lognormal":          # median 2048, sigma 1
        z = np.array([statistics.NormalDist().inv_cdf(float(x)) for x in q])
        x = 2048.0 * np.exp(z)
    else:
        x = case["lo"] + (case["hi"] - case["lo"]) * q
    return np.clip(np.rint(x), case["lo"], case["hi"]).astype(np.int64)


def _blocks(case):
    return int((-(-_quantiles(case) // case["block"])).sum())


def _slice_blocks(case):
    """Slice-resident logical blocks of one layer."""
    return max(1, int(case["slice"] * _blocks(case) + 0.5))


def _last_in_slice(case):
    """Expected number of sequences whose last block is in the slice, per layer."""
    return case["batch"] * case["slice"]


def _attention_work(case):
    tok = int(_quantiles(case).sum())
    out = 4 if case["out"] == "f32" else 2
    return {"bytes": tok * 2 * case["kv_heads"] * D * 2 + case["batch"] * case["q_heads"] * D * (2 + out)
            + 4 * _blocks(case) + 4 * case["batch"],
            "flops": 4 * tok * case["q_heads"] * D}


def work(case):
    bb = _block_bytes(case)
    kind = case["kind"]
    if kind in ("swap-in", "swap-out"):
        return {"bytes": case["blocks"] * (2 * bb + 8), "flops": 0}
    if kind == "attention":
        return _attention_work(case)
    L = case["layers"]
    if kind == "reclaim":      # the movers travel out and back, the tables are read
        n = _returned(case)
        entries = L * case["batch"] * int(-(-_quantiles(case).max() // case["block"]))
        return {"bytes": 4 * n * bb + 4 * entries, "flops": 0}
    w = _attention_work(case)
    per_layer = w["bytes"]
    if kind == "step":
        per_layer += 2 * _slice_blocks(case) * bb + case["batch"] * case["kv_heads"] * D * 8 \
            + 2 * _last_in_slice(case) * bb
    else:                      # whole slabs travel
        slabs = -(-_slice_blocks(case) // case["slab"])
        per_layer += 2 * slabs * case["slab"] * bb
    return {"bytes": L * per_layer, "flops": L * w["flops"]}


def tolerance(case):
    if case["kind"] in ("swap-in", "swap-out", "reclaim"):
        return "exact"
    # 16-bit outputs: a last place that rounds the other way; fp32 outputs:
    # probabilities of 16 significant bits, sums in another order
    if case["out"] == "bf16":
        return {"rel": 2e-3, "max": 1.6e-2}
    if case["out"] == "f16":
        return {"rel": 3e-4, "max": 2e-3}
    return {"rel": 2e-5, "max": 8e-4}


# ---- states -----------------------------------------------------------------------

class _Handle:
    """Gives a slice back when the last user of it (a state, or an output that
    is one of its pools) is gone."""

    def __init__(self, h):
        self.h = h

    def __del__(self):
        torch.cuda.synchronize()
        ema.slice_destroy(self.h)


class _PoolBytes:
    def __init__(self, owner, base, nbytes):
        self.owner = owner
        self.__cuda_array_interface__ = {"shape": (nbytes // 8,), "typestr": "<i8",
                                         "data": (base, False), "version": 3, "strides": None}


def _pools(owner):
    """Both pools as int64 tensors [blocks][words] that keep the slice alive."""
    info = ema.slice_get_info(owner.h)
    got = []
    for n, base in ((info["n_local"], info["local_base"]), (info["n_slice"], info["slice_base"])):
        nbytes = n * info["block_bytes"]
        if n:
            t = torch.as_tensor(_PoolBytes(owner, base, nbytes), device="cuda")
            got.append(t.view(n, -1))
        else:
            got.append(torch.empty((0, info["block_bytes"] // 8), dtype=torch.int64, device="cuda"))
    return got


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(27040 + int(seed))
    return g


def _fill(pools, gen, dtype):
    """iid N(0,1) rounded to the 16-bit type, both pools in turn."""
    for p in pools:
        flat = p.view(-1).view(DT[dtype])
        chunk = 1 << 27
        for s in range(0, flat.numel(), chunk):
            n = min(chunk, flat.numel() - s)
            flat[s:s + n].copy_(torch.randn(n, generator=gen, device="cuda"))


def _normal(shape, gen, dtype):
    return torch.randn(shape, generator=gen, device="cuda").to(DT[dtype])


def _i32(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).to("cuda")


def _lens(case, rng):
    return rng.permutation(_quantiles(case))


def _logical(lens, bs):
    """Rows (sequence, logical block) of every block, and the table width."""
    nb = -(-lens // bs)
    maxblk = int(nb.max())
    b, j = np.nonzero(np.arange(maxblk)[None, :] < nb[:, None])
    return np.stack([b, j], axis=1), maxblk


def _attention_plan(case, seed):
    """Lengths and block table of an attention case: scattered local ids."""
    rng = np.random.default_rng(seed)
    lens = _lens(case, rng)
    rows, maxblk = _logical(lens, case["block"])
    table = np.full((case["batch"], maxblk), -1, np.int64)
    table[rows[:, 0], rows[:, 1]] = rng.permutation(len(rows))
    return lens, table, rows


def _cache_plan(case, seed):
    """Lengths, table width and the allocation orders of a step's cache: of
    every layer's blocks a random share in the slice, in scattered order."""
    rng = np.random.default_rng(seed)
    lens = _lens(case, rng)
    rows, maxblk = _logical(lens, case["block"])
    k = _slice_blocks(case)
    local, away = [], []
    for l in range(case["layers"]):
        p = rng.permutation(len(rows))
        lr = np.concatenate([np.full((len(rows), 1), l), rows], axis=1)
        away.append(lr[p[:k]])
        local.append(lr[p[k:]])
    local, away = np.concatenate(local), np.concatenate(away)
    return lens, maxblk, local[rng.permutation(len(local))], away[rng.permutation(len(away))]


def _slab_plan(case, seed):
    """Lengths, table width, which blocks are at slab positions, the order in
    which blocks are placed, and the slabs set aside meanwhile."""
    rng = np.random.default_rng(seed)
    lens = _lens(case, rng)
    rows, maxblk = _logical(lens, case["block"])
    order = rows[rng.permutation(len(rows))]
    in_slab = np.zeros((case["batch"], maxblk), bool)
    pick = rng.permutation(len(rows))[:_slice_blocks(case)]
    in_slab[rows[pick, 0], rows[pick, 1]] = True
    need = -(-len(pick) // case["slab"])
    gaps = np.zeros(2 * need, bool)
    if need:
        gaps[1 + rng.choice(2 * need - 1, size=need, replace=False)] = True
    return lens, maxblk, in_slab, order, gaps


def _dtype(case):
    return case.get("dtype", "bf16")


def prepare(case, seed):
    return {"attention": _prepare_attention, "swap-in": _prepare_swap, "swap-out": _prepare_swap,
            "step": _prepare_step, "slab-step": _prepare_slab,
            "reclaim": _prepare_reclaim}[case["kind"]](case, seed)


def run(state):
    return state["run"](state)


def _prepare_attention(case, seed):
    lens, table, rows = _attention_plan(case, seed)
    bb = _block_bytes(case)
    own = _Handle(ema.slice_create(case["kv_heads"], D, case["block"], case["dtype"],
                                   ema.LAYOUT_ATTN, len(rows) * bb, 0))
    ids = ema.slice_alloc_blocks(own.h, ema.POOL_LOCAL, rows[:, 0])
    gen = _generator(seed)
    _fill(_pools(own), gen, case["dtype"])
    assert len(ids) == len(rows)
    q = _normal((case["batch"], case["q_heads"], D), gen, case["dtype"])
    return {"run": _run_attention, "own": own, "q": q, "table": _i32(table), "lens": _i32(lens),
            "out": torch.empty(q.shape, dtype=DT[case["out"]], device="cuda")}


def _run_attention(s):
    ema.paged_decode_attention(s["own"].h, s["q"], s["table"], s["lens"], s["out"])
    return s["out"]


def _prepare_swap(case, seed):
    rng = np.random.default_rng(seed)
    bb, n = _block_bytes(case), case["blocks"]
    n_slice = n + n // 4 + 1
    own = _Handle(ema.slice_create(case["kv_heads"], D, case["block"], _dtype(case),
                                   LAYOUT[case["layout"]], n * bb, n_slice * bb))
    stage = ema.slice_alloc_blocks(own.h, ema.POOL_LOCAL, np.full(n, ema.STAGING))
    away = ema.slice_alloc_blocks(own.h, ema.POOL_SLICE, np.arange(n_slice) % 64)
    pools = _pools(own)
    _fill(pools, _generator(seed), _dtype(case))
    away = away[rng.permutation(n_slice)[:n]]
    out = case["kind"] == "swap-out"
    return {"run": _run_swap, "own": own, "src": _i32(stage if out else away),
            "dst": _i32(away if out else stage), "pool": pools[1 if out else 0],
            "call": ema.slice_writeback if out else ema.slice_prefetch}


def _run_swap(s):
    s["call"](s["own"].h, s["src"], s["dst"])
    return s["pool"]


def _prepare_step(case, seed):
    lens, maxblk, local, away = _cache_plan(case, seed)
    c = PagedKVCache(kv_heads=case["kv_heads"], head_dim=D, block_size=case["block"],
                     dtype=case["dtype"], slice_layout=LAYOUT[case["layout"]],
                     layers=case["layers"], lens=lens, maxblk=maxblk, local_order=local,
                     slice_order=away, q_heads=case["q_heads"], staging_slots=2 * case["group"],
                     group=case["group"])
    own = _Handle(c.h)
    pools = _pools(own)
    gen = _generator(seed)
    _fill(pools, gen, case["dtype"])
    c.q = _normal((case["batch"], case["q_heads"], D), gen, case["dtype"])
    new = [_normal((2, case["batch"], case["kv_heads"], D), gen, case["dtype"])
           for _ in range(case["layers"])]
    return {"run": _run_step, "own": own, "cache": c, "new": [(x[0], x[1]) for x in new],
            "outs": [c.new_out(DT[case["out"]]) for _ in range(case["layers"])], "pools": pools}


def _run_step(s):
    c = s["cache"]
    for k, layers in enumerate(c.groups):
        c.prefetch_group(k)
        for l in layers:
            c.append(l, *s["new"][l])
            c.attention(l, s["outs"][l])
        c.writeback_group(k)
    return s["outs"] + s["pools"]


def _prepare_slab(case, seed):
    lens, maxblk, in_slab, order, gaps = _slab_plan(case, seed)
    c = SlabKVCache(kv_heads=case["kv_heads"], head_dim=D, block_size=case["block"],
                    dtype=case["dtype"], slice_layout=LAYOUT[case["layout"]],
                    layers=case["layers"], lens=lens, maxblk=maxblk, in_slab=in_slab, order=order,
                    q_heads=case["q_heads"], slab_blocks=case["slab"], group=case["group"],
                    slab_layout=ema.SLAB_GROUP_MAJOR, extra_slabs=int(gaps.sum()),
                    gap_slabs=gaps)
    own = _Handle(c.h)
    pools = _pools(own)
    gen = _generator(seed)
    _fill(pools, gen, case["dtype"])
    c.q = _normal((case["batch"], case["q_heads"], D), gen, case["dtype"])
    return {"run": _run_slab, "own": own, "cache": c, "pools": pools,
            "outs": [c.new_out(DT[case["out"]]) for _ in range(case["layers"])]}


def _run_slab(s):
    c = s["cache"]
    for k, layers in enumerate(c.groups):
        c.prefetch_group(k)
        for l in layers:
            c.attention(l, s["outs"][l])
    return s["outs"] + [s["pools"][0]]


def _returned(case):
    return max(1, int(case["share"] * case["layers"] * _slice_blocks(case)))


def _prepare_reclaim(case, seed):
    lens, maxblk, local, away = _cache_plan(case, seed)
    c = PagedKVCache(kv_heads=case["kv_heads"], head_dim=D, block_size=case["block"],
                     dtype=_dtype(case), slice_layout=LAYOUT[case["layout"]],
                     layers=case["layers"], lens=lens, maxblk=maxblk, local_order=local,
                     slice_order=away, q_heads=case["kv_heads"], staging_slots=1,
                     extra_local=_returned(case))
    own = _Handle(c.h)
    pools = _pools(own)
    _fill(pools, _generator(seed), _dtype(case))
    tables = torch.from_numpy(c.tables.astype(np.int32)).pin_memory()
    return {"run": _run_reclaim, "own": own, "cache": c, "n": _returned(case), "pools": pools,
            "canon": tables, "owner": ema.slice_owners(own.h)[1],
            "rewritten": torch.empty_like(c.tables_dev)}


def _run_reclaim(s):
    h, c = s["own"].h, s["cache"]
    r = ema.slice_reclaim(h, s["n"], c.tables_dev.view(-1))
    s["rewritten"].copy_(c.tables_dev)
    # later the lender lends the slots again, and the borrower moves back in
    ema.slice_lend(h, s["n"])
    src, dst = r["moves"][:, 0], r["moves"][:, 1]
    back = ema.slice_alloc_blocks(h, ema.POOL_SLICE, s["owner"][src - c.n_local])
    ema.slice_migrate(h, _i32(dst), _i32(back))
    ema.slice_free_blocks(h, dst)
    c.tables_dev.copy_(s["canon"], non_blocking=True)
    return [r["moves"], back, s["rewritten"], c.tables_dev] + s["pools"]


# ---- what the outputs are, in 64 bits ------------------------------------------------

def _kv64(blocks, case, layout):
    """K, V [kv_head][token][channel] in float64 of blocks [n][elements]."""
    n, H, bs = len(blocks), case["kv_heads"], case["block"]
    half = H * bs * D
    k, v = blocks[:, :half], blocks[:, half:]
    if layout == "attn":
        k = k.reshape(n, H, bs, D).permute(1, 0, 2, 3)
        v = v.reshape(n, H, D, bs).permute(1, 0, 3, 2)
    else:
        k = k.reshape(n, bs, H, D).permute(2, 0, 1, 3)
        v = v.reshape(n, bs, H, D).permute(2, 0, 1, 3)
    return (k.to(torch.float64).reshape(H, n * bs, D), v.to(torch.float64).reshape(H, n * bs, D))


def _attend64(q, k, v):
    """softmax(q k^T / sqrt(D)) v, one sequence: q [q_heads][D], k, v [kv_head][token][D]."""
    H = k.shape[0]
    qh = q.to(torch.float64).reshape(H, -1, D)
    s = torch.matmul(qh, k.transpose(1, 2).contiguous()) / math.sqrt(D)
    return torch.matmul(torch.softmax(s, dim=-1), v).reshape(-1, D)


def _empty_pools(case, n_local, n_slice):
    words = _block_bytes(case) // 8
    return [torch.empty((n, words), dtype=torch.int64, device="cuda") for n in (n_local, n_slice)]


def exact(case, seed):
    return {"attention": _exact_attention, "step": _exact_step,
            "slab-step": _exact_slab}.get(case["kind"], lambda c, s: None)(case, seed)


def _exact_attention(case, seed):
    lens, table, rows = _attention_plan(case, seed)
    pools = _empty_pools(case, len(rows), 0)
    gen = _generator(seed)
    _fill(pools, gen, case["dtype"])
    q = _normal((case["batch"], case["q_heads"], D), gen, case["dtype"])
    elems = pools[0].view(DT[case["dtype"]])
    out = torch.zeros(q.shape, dtype=torch.float64, device="cuda")
    for b, n in enumerate(lens):
        ids = torch.from_numpy(table[b, :-(-n // case["block"])]).to("cuda")
        k, v = _kv64(elems[ids], case, "attn")
        out[b] = _attend64(q[b], k[:, :n], v[:, :n])
    return out


def _gather64(case, pools, ids, n_local, layout):
    """K, V in float64 of one sequence's blocks by unified id."""
    loc = ids < n_local
    k = v = None
    H, bs = case["kv_heads"], case["block"]
    for pool, pick, base, lay in ((pools[0], loc, 0, "attn"), (pools[1], ~loc, n_local, layout)):
        if not pick.any():
            continue
        at = torch.from_numpy(np.nonzero(pick)[0]).to("cuda")
        kk, vv = _kv64(pool[torch.from_numpy(ids[pick] - base).to("cuda")].view(DT[case["dtype"]]),
                       case, lay)
        if k is None:
            k = torch.empty((H, len(ids), bs, D), dtype=torch.float64, device="cuda")
            v = torch.empty_like(k)
        k[:, at] = kk.view(H, -1, bs, D)
        v[:, at] = vv.view(H, -1, bs, D)
    return k.reshape(H, -1, D), v.reshape(H, -1, D)


def _exact_step(case, seed):
    lens, maxblk, local, away = _cache_plan(case, seed)
    L, k_slice = case["layers"], _slice_blocks(case)
    n_local = len(local) + 2 * case["group"] * k_slice
    pools = _empty_pools(case, n_local, len(away))
    gen = _generator(seed)
    _fill(pools, gen, case["dtype"])
    q = _normal((case["batch"], case["q_heads"], D), gen, case["dtype"])
    new = [_normal((2, case["batch"], case["kv_heads"], D), gen, case["dtype"]) for _ in range(L)]
    tables = np.full((L, case["batch"], maxblk), -1, np.int64)
    tables[local[:, 0], local[:, 1], local[:, 2]] = np.arange(len(local))
    tables[away[:, 0], away[:, 1], away[:, 2]] = n_local + np.arange(len(away))
    outs = []
    for l in range(L):
        out = torch.zeros(q.shape, dtype=torch.float64, device="cuda")
        for b, n in enumerate(lens):
            ids = tables[l, b, :-(-n // case["block"])]
            k, v = _gather64(case, pools, ids, n_local, case["layout"])
            k[:, n - 1] = new[l][0, b].to(torch.float64)
            v[:, n - 1] = new[l][1, b].to(torch.float64)
            out[b] = _attend64(q[b], k[:, :n], v[:, :n])
        outs.append(out)
    return outs + [None, None]


def _exact_slab(case, seed):
    lens, maxblk, in_slab, order, gaps = _slab_plan(case, seed)
    L, S, g = case["layers"], case["slab"], case["group"]
    n_pos = int(in_slab.sum())
    n_slabs = -(-n_pos // S) + int(gaps.sum())
    kept = np.nonzero(~gaps)[0]
    sl = in_slab[order[:, 0], order[:, 1]]
    away, local = order[sl], order[~sl]
    n_local = len(local) * L + 2 * n_slabs * g * S
    pools = _empty_pools(case, n_local, n_slabs * L * S)
    gen = _generator(seed)
    _fill(pools, gen, case["dtype"])
    q = _normal((case["batch"], case["q_heads"], D), gen, case["dtype"])
    t = np.arange(len(away))
    outs = []
    for l in range(L):
        table = np.full((case["batch"], maxblk), -1, np.int64)
        table[local[:, 0], local[:, 1]] = np.arange(len(local)) * L + l
        if len(away):
            table[away[:, 0], away[:, 1]] = \
                n_local + ((l // g * n_slabs + kept[t // S]) * g + l % g) * S + t % S
        out = torch.zeros(q.shape, dtype=torch.float64, device="cuda")
        for b, n in enumerate(lens):
            k, v = _gather64(case, pools, table[b, :-(-n // case["block"])], n_local, case["layout"])
            out[b] = _attend64(q[b], k[:, :n], v[:, :n])
        outs.append(out)
    return outs + [None]
