"""Every copy kernel at the edges of its work units: layout changes in 16 KiB
tiles (block sizes from 32 on) and 4 KiB units (block size 16, odd head counts
at 32), straight copies inside either pool, and same-layout lists around the
rounds that deal whole blocks to the XCDs. Byte-exact against the layouts as
the generator's own packer states them; an id out of range leaves its
destination alone and is counted once."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ema():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_27040_amd import ema as m
    return m


class Pools:
    def __init__(self, ema, H, bs, layout, n_local, n_slice):
        self.ema, self.H, self.bs, self.layout = ema, H, bs, layout
        self.bb = 2 * bs * H * 128 * 2
        self.n_local = n_local
        self.h = ema.slice_create(H, 128, bs, "bf16", layout, n_local * self.bb, n_slice * self.bb)
        rng = np.random.default_rng(H * 1000 + bs)
        self.host = [rng.integers(0, 256, (n, self.bb), dtype=np.uint8) for n in (n_local, n_slice)]
        self.dev = [ema.pool_view(self.h, p) for p in (ema.POOL_LOCAL, ema.POOL_SLICE)]
        for d, a in zip(self.dev, self.host):
            d.copy_(torch.from_numpy(a))

    def row(self, u):
        return (0, u) if u < self.n_local else (1, u - self.n_local)

    def copy_host(self, s, d):
        (ps, s), (pd, d) = self.row(s), self.row(d)
        b = self.host[ps][s]
        if ps != pd and self.layout == synth.LAYOUT_NHD:
            lay = [synth.LAYOUT_ATTN, self.layout]
            k, v = synth.unpack_block(b, lay[ps], self.H, self.bs, 128)
            b = synth.pack_block(k, v, lay[pd])
        self.host[pd][d] = b

    def run(self, src, dst):
        i32 = lambda a: torch.as_tensor(np.asarray(a, np.int32), device="cuda")
        self.ema.slice_migrate(self.h, i32(src), i32(dst))
        torch.cuda.synchronize()

    def check(self):
        for d, a in zip(self.dev, self.host):
            assert torch.equal(d.cpu(), torch.from_numpy(a))

    def close(self):
        self.dev = None
        self.ema.slice_destroy(self.h)


@pytest.mark.parametrize("H,bs", [(1, 16), (3, 16), (8, 16), (1, 32), (3, 32), (2, 32), (6, 32),
                                  (4, 32), (1, 64), (2, 64), (3, 64), (8, 64), (5, 128), (4, 128),
                                  (1, 256), (2, 256)])
def test_layout_changes(ema, H, bs):
    print(f"tiles H={H} bs={bs}", flush=True)
    p = Pools(ema, H, bs, synth.LAYOUT_NHD, 7, 8)
    try:
        # in, out, and within each pool, in one list
        src, dst = [7, 9, 0, 1, 2, 10], [3, 4, 11, 12, 5, 13]
        p.run(src, dst)
        for s, d in zip(src, dst):
            p.copy_host(s, d)
        p.check()
        assert ema.slice_device_errors(p.h) == 0
        p.run([8, -1, 15], [6, 0, 1])              # an id below and one past the pools
        p.copy_host(8, 6)
        p.check()
        assert ema.slice_device_errors(p.h) == 2
    finally:
        p.close()


@pytest.mark.parametrize("H,bs,n", [(1, 16, 33), (3, 16, 7), (3, 16, 8), (3, 16, 9), (8, 16, 17),
                                    (8, 32, 8), (8, 64, 9), (5, 128, 8), (8, 256, 9), (8, 256, 5)])
def test_same_layout_rounds(ema, H, bs, n):
    """n blocks of 8 KiB to 1 MiB: fewer than a round of 8 runs of up to
    256 KiB, whole rounds, and rounds with a remainder; as a list and as runs."""
    print(f"rounds H={H} bs={bs} n={n}", flush=True)
    p = Pools(ema, H, bs, synth.LAYOUT_ATTN, n + 1, n + 3)
    try:
        rng = np.random.default_rng(n)
        src = p.n_local + rng.permutation(n + 3)[:n]
        dst = rng.permutation(n + 1)[:n]
        p.run(src, dst)
        for s, d in zip(src, dst):
            p.copy_host(s, d)
        p.check()
        stage = ema.slice_alloc_blocks(p.h, ema.POOL_LOCAL, np.full(n + 1, ema.STAGING))
        away = ema.slice_alloc_blocks(p.h, ema.POOL_SLICE, np.zeros(n + 3, np.int32))
        first = [int(away[2])], [int(stage[0])], [n]
        ema.slice_prefetch_runs(p.h, *first)
        torch.cuda.synchronize()
        for k in range(n):
            p.copy_host(int(away[2]) + k, int(stage[0]) + k)
        p.check()
        assert ema.slice_device_errors(p.h) == 0
    finally:
        p.close()


def test_lists_longer_than_a_grid_row(ema):
    """A same-layout list past 32768 blocks, the list kernel's second grid
    layer: every block lands where it should, and ids out of range on both
    sides of the line leave their destinations alone."""
    n = 32768 + 6
    print(f"long list n={n}", flush=True)
    p = Pools(ema, 1, 16, synth.LAYOUT_ATTN, n, n)
    try:
        rng = np.random.default_rng(5)
        src, dst = n + rng.permutation(n), rng.permutation(n)
        bad = {0: -1, 32767: 2 * n, 32768: 2 ** 31 - 1, n - 1: -2 ** 31}
        for i, u in bad.items():
            (src if i % 2 else dst)[i] = u
        p.run(src, dst)
        ok = np.array([i for i in range(n) if i not in bad])
        p.host[0][dst[ok]] = p.host[1][src[ok] - n]
        p.check()
        assert ema.slice_device_errors(p.h) == len(bad)
    finally:
        p.close()
