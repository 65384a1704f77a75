"""Edges of the stream-K attention's wave-level ranges, against the float64
oracle: a pair that crosses many workgroups between empty sequences (more
partials than one combine round reads), pairs of one tile each (several per
wave, pieces merged within a workgroup), a wave's piece of more than 64 blocks
(several id lists), tables that hold ids outside the local pool (their tokens
are left out and counted), and an output that is not aligned for wide stores.

Bar: 2e-3, as for every attention test (16-bit probabilities in two parts,
fp32 accumulation)."""
import numpy as np
import pytest
import torch

import oracle
import synth
from harness import Workload, oracle_mirror, rel_err

pytestmark = pytest.mark.gpu
TOL = 2e-3


@pytest.fixture(scope="module")
def ema():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_27040_amd import ema as m
    return m


CASES = {
    # one pair over every workgroup of 256: 1022 tiles over 1024 waves
    "one-long": (4, 1, 16, "bf16", [0, 32690, 0]),
    # 4 heads of one long sequence: each crosses 36 workgroups of 256
    "long-16-heads": (64, 4, 32, "f16", [0, 0, 9000, 33]),
    # one tile a pair, eight pairs a wave and more
    "short": (16, 8, 16, "f16", [1 + i % 32 for i in range(1500)]),
    # tiles of one and two blocks, whole and cut
    "mixed": (8, 2, 64, "bf16", [0, 1, 31, 32, 33, 63, 64, 65, 1023, 1025, 4097, 0]),
}


@pytest.mark.parametrize("name", CASES)
def test_ranges(ema, name):
    hq, hkv, bs, dtype, lens = CASES[name]
    print(f"stream {name}", flush=True)
    cfg = synth.KVConfig("stream", 1, hq, hkv, 128, dtype, bs, len(lens), ("uniform", 0, 0), 0.0,
                         4100 + len(lens))
    w = Workload(cfg, lens=lens, staging_slots=1)
    try:
        st = oracle_mirror(w)
        out = w.new_out()
        out.fill_(float("nan"))
        w.attention(0, out)
        again = w.new_out()
        w.attention(0, again)
        flat = torch.full((out.numel() + 1,), float("nan"), device="cuda")
        odd = flat[1:].view(out.shape)                     # 4 bytes past a 16-byte boundary
        ema.paged_decode_attention(w.h, w.q, w.attn_dev[0], w.lens_dev, odd)
        torch.cuda.synchronize()
        assert ema.slice_device_errors(w.h) == 0
        assert torch.equal(out, again)
        assert torch.equal(out, odd)
        ref = oracle.paged_decode_attention(w.q16, w.attn_tables[0], w.lens, st.read_block, w.hkv,
                                            w.D, w.bs, w.cfg.dtype)
        assert rel_err(out.cpu().numpy(), ref) <= TOL
    finally:
        w.close()


@pytest.mark.parametrize("tiles", [14, 17, 18, 62, 63, 254, 255, 1022, 1023, 2500])
@pytest.mark.parametrize("hq,others", [(1, 0), (16, 0), (8, 3), (4, 300)])
def test_partials_of_one_pair(ema, hq, others, tiles):
    """A pair cut over n workgroups, n at the edges of the combine's rounds (4,
    5, 16, 17, 64, 65 and 256 of 256 workgroups): alone, with a few more pairs
    (a record per pair) and after more pairs than workgroups (a record per
    workgroup)."""
    print(f"partials hq={hq} others={others} tiles={tiles}", flush=True)
    lens = [1 + i % 40 for i in range(others)] + [32 * tiles - 5]
    cfg = synth.KVConfig("partials", 1, hq, 1, 128, "f16", 64, len(lens), ("uniform", 0, 0), 0.0,
                         4500 + tiles)
    w = Workload(cfg, lens=lens, staging_slots=1)
    try:
        st = oracle_mirror(w)
        table = torch.full((len(lens), w.attn_dev.shape[2] + 16), -1, dtype=torch.int32, device="cuda")
        table[:, :w.attn_dev.shape[2]] = w.attn_dev[0]
        out = w.new_out()
        for _ in range(2):
            out.fill_(float("nan"))
            w.attention(0, out, table=table)
            torch.cuda.synchronize()
            assert ema.slice_device_errors(w.h) == 0
            ref = oracle.paged_decode_attention(w.q16, w.attn_tables[0], w.lens, st.read_block,
                                                w.hkv, w.D, w.bs, w.cfg.dtype)
            assert rel_err(out.cpu().numpy(), ref) <= TOL
    finally:
        w.close()


@pytest.mark.parametrize("hq,hkv,bs,dtype,batch,width", [
    (8, 8, 16, "f16", 8, 32), (32, 8, 16, "bf16", 64, 32), (4, 1, 32, "bf16", 256, 16),
    (16, 1, 64, "f16", 3, 4), (6, 3, 128, "bf16", 5, 2), (4, 2, 256, "bf16", 4, 1),
    (16, 8, 16, "f16", 64, 16), (8, 1, 64, "bf16", 65, 8),
    # one past each line of the rule: 257 pairs, 513 pairs, 17 tiles, 64 pairs of 9 tiles
    (2, 1, 16, "bf16", 257, 32), (1, 1, 16, "f16", 513, 16), (1, 1, 64, "f16", 64, 5),
    (4, 2, 32, "f16", 4, 17), (8, 1, 64, "bf16", 4, 5)])
def test_short_tables(ema, hq, hkv, bs, dtype, batch, width):
    """Both sides of the line between the direct and the stream-K form: lengths
    from 0 to the table's width, ids outside the pool, and the same outputs
    from the entry point that allocates nothing."""
    rng = np.random.default_rng(batch + bs)
    lens = rng.integers(0, width * bs + 1, batch)
    edge = [0, 1, 31, 32, 33, width * bs, max(1, width * bs - 1)]
    lens[:min(len(edge), batch)] = edge[:batch]
    lens[-1] = width * bs
    cfg = synth.KVConfig("direct", 1, hq, hkv, 128, dtype, bs, batch, ("uniform", 0, 0), 0.0,
                         4400 + batch)
    w = Workload(cfg, lens=lens.tolist(), staging_slots=1)
    try:
        st = oracle_mirror(w)
        assert w.attn_dev.shape[2] == width
        out, na = w.new_out(), w.new_out()
        out.fill_(float("nan"))
        w.attention(0, out)
        ema.paged_decode_attention_noalloc(w.h, w.q, w.attn_dev[0], w.lens_dev, na)
        flat = torch.full((out.numel() + 1,), float("nan"), device="cuda")
        odd = flat[1:].view(out.shape)
        ema.paged_decode_attention(w.h, w.q, w.attn_dev[0], w.lens_dev, odd)
        torch.cuda.synchronize()
        assert ema.slice_device_errors(w.h) == 0
        assert torch.equal(out, na) and torch.equal(out, odd)
        got = out.cpu().numpy()
        ref = oracle.paged_decode_attention(w.q16, w.attn_tables[0], w.lens, st.read_block, w.hkv,
                                            w.D, w.bs, w.cfg.dtype)
        assert rel_err(got, ref) <= TOL
        assert (got[lens == 0] == 0).all()
        # a sequence whose only block is no local block gives zeros and is counted
        tab = w.attn_tables[0].copy()
        tab[-1, :] = w.local_view.shape[0]
        w.attention(0, out, table=torch.as_tensor(tab.astype(np.int32), device="cuda"))
        torch.cuda.synchronize()
        assert ema.slice_device_errors(w.h) >= 1
        assert torch.equal(out[:-1], na[:-1]) and torch.count_nonzero(out[-1]) == 0
    finally:
        w.close()


@pytest.mark.parametrize("hq,hkv,bs,dtype,batch,lo,hi,bound", [
    (32, 8, 16, "bf16", 64, 1024, 4096, 2.9e-6), (32, 8, 16, "bf16", 64, 17, 1000, 2.9e-6),
    (8, 1, 32, "bf16", 64, 128, 6000, 2.9e-6), (16, 1, 64, "bf16", 32, 100, 9000, 2.9e-6),
    (8, 8, 16, "bf16", 8, 64, 512, 2.9e-6),
    (32, 8, 16, "f16", 64, 1024, 4096, 3.1e-7), (32, 8, 16, "f16", 64, 17, 1000, 2.0e-7),
    (8, 8, 64, "f16", 64, 200, 1500, 2.4e-7), (64, 8, 16, "f16", 256, 17, 300, 1.9e-7),
    (32, 2, 32, "f16", 4, 30000, 90000, 3.4e-7), (8, 8, 16, "f16", 8, 64, 512, 2.0e-7)])
def test_error_against_64_bits(ema, hq, hkv, bs, dtype, batch, lo, hi, bound):
    """2-norm of the error over 2-norm of the result, normal values, fp32 output.

    bf16: probabilities are two parts rounded to nearest, which leaves a
    remainder of 2^-8 rounded to 8 bits: 2.5e-6 of a probability (root mean
    square over its binade), so 2.5e-6 of a sum over independent values, plus
    the fp32 sums' few 1e-7: 2.9e-6. A truncated high part gives twice that (3.5
    to 4.4e-6 measured).
    f16 keeps 22 bits, so the scores' and the sums' fp32 roundings show. The
    bounds are what four waves to a pair, each with every fourth tile, measured
    (3.09e-7, 1.94e-7, 2.33e-7, 1.80e-7, 3.42e-7 and 1.90e-7 in this order, to the
    next tenth): a wave with all of a pair's tiles must not be further off. Added
    up in the matrix cores from tile to tile it is: 3.87e-7, 2.14e-7, 2.71e-7,
    1.96e-7, 3.47e-7 and 1.95e-7."""
    print(f"error {hq}/{hkv} bs={bs} {dtype} B={batch} {lo}-{hi}", flush=True)
    lens = np.rint(lo + (hi - lo) * (np.arange(batch) + 0.5) / batch).astype(int)
    lens = np.random.default_rng(batch).permutation(lens)
    cfg = synth.KVConfig("error", 1, hq, hkv, 128, dtype, bs, batch, ("uniform", 0, 0), 0.0, 4600)
    w = Workload(cfg, lens=lens.tolist(), fill="device", staging_slots=1)
    try:
        dt = {"bf16": torch.bfloat16, "f16": torch.float16}[dtype]
        out = w.new_out()
        off = ref2 = 0.0
        for seed in range(3):
            g = torch.Generator(device="cuda")
            g.manual_seed(seed)
            flat = w.local_view.view(-1).view(dt)
            flat.copy_(torch.randn(flat.numel(), generator=g, device="cuda"))
            w.q.copy_(torch.randn(w.q.shape, generator=g, device="cuda"))
            w.attention(0, out)
            halves = flat.view(w.local_view.shape[0], 2, -1)
            for b, n in enumerate(lens):
                ids = torch.as_tensor(w.attn_tables[0][b, :-(-n // bs)], device="cuda")
                k = halves[ids, 0].view(-1, hkv, bs, 128).permute(1, 0, 2, 3)
                v = halves[ids, 1].view(-1, hkv, 128, bs).permute(1, 0, 3, 2)
                k, v = (x.double().reshape(hkv, -1, 128)[:, :n].contiguous() for x in (k, v))
                s = torch.matmul(w.q[b].double().view(hkv, -1, 128), k.transpose(1, 2).contiguous())
                ref = torch.matmul(torch.softmax(s / 128 ** 0.5, dim=-1), v).reshape(-1, 128)
                off += float((out[b].double() - ref).square().sum())
                ref2 += float(ref.square().sum())
        assert ema.slice_device_errors(w.h) == 0
        assert (off / ref2) ** 0.5 <= bound, (off / ref2) ** 0.5
    finally:
        w.close()


@pytest.mark.parametrize("hq,hkv,bs,dtype,batch,longest", [
    (8, 8, 16, "f16", 8, 512), (32, 8, 16, "bf16", 32, 500), (1, 1, 128, "f16", 200, 200),
    (4, 2, 64, "bf16", 20, 256), (4, 4, 32, "f16", 1, 40),
    # pairs whose runs just have a slot each in the workspace, and one more
    (8, 1, 16, "bf16", 128, 300), (8, 1, 32, "bf16", 129, 512), (32, 2, 256, "bf16", 32, 256),
    (16, 1, 16, "f16", 65, 512),
    (32, 8, 16, "bf16", 64, 256), (1, 1, 256, "bf16", 257, 256), (8, 1, 64, "bf16", 64, 512),
    (4, 1, 128, "f16", 65, 512), (2, 2, 256, "bf16", 100, 512),
    # past the rule by a pair or a token, and long
    (2, 1, 16, "bf16", 257, 512), (2, 1, 32, "f16", 300, 257), (2, 1, 64, "f16", 513, 256),
    (4, 2, 32, "f16", 9, 513), (8, 1, 64, "bf16", 4, 513),
    (16, 4, 16, "bf16", 30, 3000)])
def test_wider_tables_give_the_same_bits(ema, hq, hkv, bs, dtype, batch, longest):
    """One batch through tables just wide enough and wider ones, on both sides
    of the direct form's line."""
    print(f"widths {hq}/{hkv} bs={bs} B={batch} {longest}", flush=True)
    rng = np.random.default_rng(longest + batch)
    lens = rng.integers(0, longest + 1, batch)
    lens[batch // 2], lens[0] = 0, longest
    cfg = synth.KVConfig("widths", 1, hq, hkv, 128, dtype, bs, batch, ("uniform", 0, 0), 0.0, 4700)
    w = Workload(cfg, lens=lens.tolist(), staging_slots=1)
    try:
        width = w.attn_dev.shape[2]
        out = w.new_out()
        w.attention(0, out)
        for more in (1, 40, 1000):
            table = torch.full((batch, width + more), -1, dtype=torch.int32, device="cuda")
            table[:, :width] = w.attn_dev[0]
            for call in (ema.paged_decode_attention, ema.paged_decode_attention_noalloc):
                wide = w.new_out()
                wide.fill_(float("nan"))
                call(w.h, w.q, table, w.lens_dev, wide)
                assert torch.equal(out, wide), (more, call.__name__)
        assert ema.slice_device_errors(w.h) == 0
        st = oracle_mirror(w)
        ref = oracle.paged_decode_attention(w.q16, w.attn_tables[0], w.lens, st.read_block, w.hkv,
                                            w.D, w.bs, w.cfg.dtype)
        assert rel_err(out.cpu().numpy(), ref) <= TOL
    finally:
        w.close()


def test_several_id_lists_per_wave(ema):
    """80 sequences of about 4k tokens at 8 KV heads and block size 16: 80 tiles
    a wave, so its pieces go over several lists of 64 ids, 32 tiles each
    (sampled sequences against the oracle)."""
    lens = [4096 - 7 * (i % 5) for i in range(80)]
    cfg = synth.KVConfig("lists", 1, 32, 8, 128, "bf16", 16, len(lens), ("uniform", 0, 0), 0.0, 4200)
    w = Workload(cfg, lens=lens, fill="device", staging_slots=1)
    try:
        tiles = sum((n + 31) // 32 for n in lens) * w.hkv
        assert tiles / 1024 > 64 * 16 / 32
        out = w.new_out()
        w.attention(0, out)
        torch.cuda.synchronize()
        assert ema.slice_device_errors(w.h) == 0
        got = out.cpu().numpy()
        for b in (0, 3, 41, 79):
            ids = torch.as_tensor(w.attn_tables[0][b], device="cuda")
            rows = w.local_view[ids].cpu().numpy()
            at = {int(u): r for u, r in zip(w.attn_tables[0][b], rows)}
            ref = oracle.paged_decode_attention(w.q16[b:b + 1], w.attn_tables[0][b:b + 1],
                                                w.lens[b:b + 1], at.__getitem__, w.hkv, w.D, w.bs,
                                                w.cfg.dtype)
            assert rel_err(got[b:b + 1], ref) <= TOL
    finally:
        w.close()


@pytest.mark.parametrize("bs", [16, 32, 128])
def test_ids_outside_the_pool_are_left_out(ema, bs):
    """Blocks whose id is no local block contribute nothing, and are counted."""
    lens = [700, 0, 40, 2000]
    cfg = synth.KVConfig("bad", 1, 8, 2, 128, "bf16", bs, len(lens), ("uniform", 0, 0), 0.0, 4300 + bs)
    w = Workload(cfg, lens=lens, staging_slots=1)
    try:
        st = oracle_mirror(w)
        tab = w.attn_tables[0].copy()
        n_total = w.local_view.shape[0]
        bad = {(0, 1): -1, (0, 2): n_total, (3, 5): 2 ** 31 - 1, (3, 0): -7}
        for (b, j), u in bad.items():
            tab[b, j] = u
        out = w.new_out()
        w.attention(0, out, table=torch.as_tensor(tab.astype(np.int32), device="cuda"))
        torch.cuda.synchronize()
        assert ema.slice_device_errors(w.h) >= len(bad)
        got = out.cpu().numpy()
        for b, n in enumerate(lens):
            keep = [t for t in range(n) if (b, t // bs) not in bad]
            if not keep:
                assert (got[b] == 0).all()
                continue
            K, V = oracle.attention._gather_sequence(st.read_block, w.attn_tables[0][b], n, w.hkv,
                                                     w.D, bs)
            ref = oracle.attention.contiguous_decode_attention(
                oracle.attention.to_float64(w.q16[b], "bf16"),
                oracle.attention.to_float64(K[:, keep], "bf16"),
                oracle.attention.to_float64(V[:, keep], "bf16"))
            assert rel_err(got[b], ref) <= TOL
    finally:
        w.close()
