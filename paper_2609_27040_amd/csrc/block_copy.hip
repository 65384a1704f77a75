// Block-table-driven gather/scatter of layer-blocks between the local pool and
// the slice (prefetch before use, migration, reclaim write-back / compaction).
//
// When both pools share one layout (the slice in the local layout), every
// copy is a straight 16-byte-per-lane copy: a wavefront moves 2 KiB of a
// block (two wave instructions of 1 KiB each way, fully coalesced; 1, 4, 8
// and 16 KiB per wavefront move fewer bytes per second). Lists of up to 2^22
// pieces (8 GiB) of scattered blocks of up to 64 KiB go one wavefront per
// workgroup; long ascending runs, larger blocks and larger lists go four
// wavefronts (8 KiB contiguous) per workgroup, which measured faster or
// steadier for them. In lists of scattered blocks above 64 KiB a block's pieces,
// up to 256 KiB of them, are dealt to one XCD (see xcd_item); ascending runs
// keep their order (dealt, a reclaim of 5 % moved 5.65-5.95 TB/s instead of
// 6.0-6.3). In order, 512 MiB take 176 us in one run and 165 in 20, at any block
// size from 64 KiB; with pieces numbered in 64 bits one run took 0.3-0.8 % less.
//
// Otherwise blocks change layout. K rows (256 bytes) only change order, V is
// transposed between [token][channel] (NHD) and [channel][token] (ATTN) in
// LDS so that both the global reads and the global writes stay 16 bytes per
// lane. From block size 32 on the work unit is a 16 KiB tile per workgroup
// (block_relayout_kernel): whole 256-byte token rows on the token-major side,
// whole 64- or 128-byte channel rows on the other. At block size 16, and where
// the heads do not divide into tiles, it is 4 KiB per wavefront, four per
// workgroup (block_copy_kernel): 16 tokens (one block's channel rows, which
// are contiguous) of one head, V through the wave's own LDS tile. Measured,
// TB/s of read + write, 8 KV heads, lists of 400 MB, 4 KiB units / 16 KiB
// tiles: into ATTN at block size 16 5.83 / 5.67, 32 5.77 / 5.80, 64 4.55 / 5.70
// and 256 4.92 / 5.73 (4 KiB units read 64 bytes of a token row there, and
// wrote the tile eight lanes to an LDS bank); out of ATTN 5.26 / 5.17, 5.11 /
// 5.46, 4.86 / 5.31 and 4.87 / 5.42. Copies that write scattered blocks stay
// at 5.2-5.9 in either layout.
#include "kernels.h"

#include <algorithm>

namespace ema {
namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int kUnitBytes = 4096;    // work unit of the layout-changing kernel
constexpr int kPieceBytes = 2048;   // work unit of the same-layout kernel
constexpr int kTileBytes = 16384;   // work unit of the tiled layout change
constexpr int64_t kXcdRunBytes = 262144;   // of a block, copied on one XCD
constexpr int kWaves = 4;
constexpr int kTileRow = 128 + 8;   // u16 per LDS tile row (padded, keeps 16 B alignment)

// u16 per wave of the 4 KiB unit's tile: 16 x kTileRow (out of ATTN, and into
// it at block size 16), 32 x 72 (into ATTN at block size 32).
__host__ __device__ constexpr int tile_elems(int bs) {
  return bs > 16 ? 32 * (64 + 8) : 16 * kTileRow;
}

// Block data is touched once per copy: streaming (non-temporal) loads and
// stores keep it from displacing other data in L2 and the memory-side cache,
// and keep written lines from being flushed later under another kernel's reads.
__device__ __forceinline__ u32x4 ld16(const char* p) {
  return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
}
__device__ __forceinline__ void st16(char* p, u32x4 v) {
  __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(p));
}

// LDS writes of this wave must land before other lanes of the wave read them.
__device__ __forceinline__ void wave_lds_sync() {
  __asm__ volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
}

// Source and destination of copy i (wave-uniform i).
__device__ __forceinline__ void copy_ids(const CopyIds& c, int32_t i, int32_t& s, int32_t& d) {
  if (c.n_runs > 0) {
    int r = 0;
    for (int q = 1; q < c.n_runs; ++q)
      if (c.run_off[q] <= i) r = q;
    s = c.run_src[r] + (i - c.run_off[r]);
    d = c.run_dst[r] + (i - c.run_off[r]);
  } else {
    s = c.src[i];
    d = c.dst ? c.dst[i] : c.dst_base + i;
  }
}

// Work item of workgroup g when `run` consecutive items (of one block) are to
// stay on one XCD: workgroups go to the 8 XCDs in turn, so within a round of
// 8 * run items XCD x gets items [x * run, (x + 1) * run). Items from `limit`
// on (the last, incomplete round) keep their order. A block's pages are then
// looked up by one XCD's translation caches instead of all eight, and its
// lines written together: 500 MB lists of scattered blocks, TB/s in order /
// in runs of up to 256 KiB: swap-in of 64 KiB blocks 6.08 / 6.26, 256 KiB 5.98 /
// 6.35, 1 MiB 5.94 / 6.33; swap-out of 256 KiB blocks 5.4-5.6 / 6.0, 1 MiB
// 5.6-5.8 / 6.1; blocks of 16 and 32 KiB the same. Runs of 16-64 KiB gain less.
__device__ __forceinline__ uint32_t xcd_item(uint32_t g, uint32_t run, uint32_t limit) {
  if (g >= limit) return g;
  const uint32_t round = 8 * run;
  const uint32_t r = g / round;
  const uint32_t q = g - r * round;
  return r * round + (q & 7) * run + (q >> 3);
}

// The table-rewrite share of a reclaim launch: workgroup g rewrites entries
// [g * kRewriteEntries, (g + 1) * kRewriteEntries), threads strided so that
// reads and writes stay coalesced. Only changed entries are written.
__device__ __forceinline__ void rewrite_tables(const TableRewrite& rw, const CopyIds& ids, int g) {
  const int64_t e0 = int64_t(g) * kRewriteEntries;
  const int64_t e1 = e0 + kRewriteEntries < rw.n_entries ? e0 + kRewriteEntries : rw.n_entries;
  for (int64_t e = e0 + threadIdx.x; e < e1; e += blockDim.x) {
    const int32_t t = rw.tables[e];
    if (t < 0) continue;
    int32_t nt = t;
    const uint32_t r = uint32_t(t - rw.base);
    if (r < uint32_t(rw.n_range)) {
      if (rw.range_map) {
        nt = rw.range_map[r];
      } else {                                   // movers: the launch's copy runs
        for (int q = 0; q < ids.n_runs; ++q) {
          const int32_t o = t - ids.run_src[q];
          const int32_t len = ids.run_off[q + 1] - ids.run_off[q];
          if (o >= 0 && o < len) nt = ids.run_dst[q] + o;
        }
      }
    } else if (uint32_t(t - rw.bits_base) < uint32_t(rw.n_bits)) {
      const uint32_t b = uint32_t(t - rw.bits_base);
      if ((rw.released_bits[b >> 5] >> (b & 31)) & 1u) nt = -1;
    }
    if (nt != t) rw.tables[e] = nt;
  }
}

__global__ __launch_bounds__(256) void block_copy_kernel(PoolView pv, CopyIds ids,
                                                         int32_t n, int32_t* err_count,
                                                         TableRewrite rw) {
  extern __shared__ __attribute__((aligned(16))) uint16_t lds_tile[];
  if (int(blockIdx.x) < rw.n_groups) {
    rewrite_tables(rw, ids, blockIdx.x);
    return;
  }
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int upb = int(pv.block_bytes / kUnitBytes);
  const int64_t unit = (int64_t(blockIdx.x) - rw.n_groups) * kWaves + wave;
  if (unit >= int64_t(n) * upb) return;
  const int32_t i = int32_t(unit / upb);
  const int k = int(unit - int64_t(i) * upb);
  int32_t s, d;
  copy_ids(ids, __builtin_amdgcn_readfirstlane(i), s, d);
  const int32_t n_total = pv.n_local + pv.n_slice;
  if (s < 0 || s >= n_total || d < 0 || d >= n_total) {
    if (k == 0 && lane == 0) atomicAdd(err_count, 1);
    return;
  }
  const bool s_local = s < pv.n_local;
  const bool d_local = d < pv.n_local;
  const char* sb = s_local ? pv.local + int64_t(s) * pv.block_bytes
                           : pv.slice + int64_t(s - pv.n_local) * pv.block_bytes;
  char* db = d_local ? pv.local + int64_t(d) * pv.block_bytes
                     : pv.slice + int64_t(d - pv.n_local) * pv.block_bytes;
  const int s_nhd = s_local ? 0 : pv.slice_layout;
  const int d_nhd = d_local ? 0 : pv.slice_layout;

  if (s_nhd == d_nhd) {
    const int64_t off = int64_t(k) * kUnitBytes + lane * 16;
    const u32x4 v0 = ld16(sb + off);
    const u32x4 v1 = ld16(sb + off + 1024);
    const u32x4 v2 = ld16(sb + off + 2048);
    const u32x4 v3 = ld16(sb + off + 3072);
    st16(db + off, v0);
    st16(db + off + 1024, v1);
    st16(db + off + 2048, v2);
    st16(db + off + 3072, v3);
    return;
  }

  // Layout change. Unit k -> (half, head h, group tg): a 16-token group, or
  // for V into ATTN a group of T tokens x 2048/T channels (BS/16 groups
  // either way).
  const int H = pv.kv_heads;
  const int BS = pv.block_size;
  const int tgs = BS / 16;
  const int uph = H * tgs;
  const int half = k / uph;
  const int r = k - half * uph;
  const int h = r / tgs;
  const int tg = r - h * tgs;
  const int64_t half_bytes = pv.block_bytes / 2;

  if (half == 0) {
    // K: 16 rows of 256 B; ATTN row (h, t) at (h*BS + t)*256, NHD row at (t*H + h)*256.
    u32x4 v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int t = tg * 16 + j * 4 + (lane >> 4);
      const int64_t row = s_nhd ? int64_t(t * H + h) : int64_t(h * BS + t);
      v[j] = ld16(sb + row * 256 + (lane & 15) * 16);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int t = tg * 16 + j * 4 + (lane >> 4);
      const int64_t row = d_nhd ? int64_t(t * H + h) : int64_t(h * BS + t);
      st16(db + row * 256 + (lane & 15) * 16, v[j]);
    }
    return;
  }

  uint16_t* tw = lds_tile + wave * tile_elems(BS);
  const char* sv = sb + half_bytes;
  char* dv = db + half_bytes;
  if (s_nhd) {
    // NHD -> ATTN, unit (h, channel group): all T = BS tokens (16 or 32) of
    // C = 2048/T channels. Read C channels of each of the T token rows (LR
    // lanes per row) into the tile as [t][c], then write C transposed rows of
    // T tokens (LC lanes each).
    const int T = BS;
    const int C = 2048 / T;
    const int cgs = 128 / C;                  // channel groups per token group
    const int t_base = (tg / cgs) * T;
    const int c0 = (tg % cgs) * C;
    const int LR = C / 8;
    const int stride = C + 8;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int t = j * (64 / LR) + lane / LR;
      const int c = (lane % LR) * 8;
      const u32x4 v = ld16(sv + (int64_t((t_base + t) * H + h) * 128 + c0 + c) * 2);
      *reinterpret_cast<u32x4*>(&tw[t * stride + c]) = v;
    }
    wave_lds_sync();
    const int LC = T / 8;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int item = j * 64 + lane;
      const int cc = item / LC;
      const int t0 = (item % LC) * 8;
      uint32_t w[4];
#pragma unroll
      for (int q = 0; q < 4; ++q)
        w[q] = uint32_t(tw[(t0 + 2 * q) * stride + cc]) |
               (uint32_t(tw[(t0 + 2 * q + 1) * stride + cc]) << 16);
      const u32x4 out = {w[0], w[1], w[2], w[3]};
      st16(dv + (int64_t(h * 128 + c0 + cc) * BS + t_base + t0) * 2, out);
    }
  } else {
    // ATTN -> NHD, unit (h, token group): 16 tokens of all 128 channels. Read
    // 16 bytes (8 tokens of a channel) per lane, two lanes per channel row;
    // the lanes of channels 2k and 2k + 1 (lane ^ 2) trade four tokens, so that
    // each holds both channels of four tokens and scatters them into the
    // [token][channel] tile as whole words; then write 16 whole 256-B token
    // rows. (8192 blocks of 64 KiB 210 us; in single channels, twice the LDS
    // writes, 213, but up to 16 blocks 3.0 instead of 3.2.)
    u32x4 v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int item = j * 64 + lane;
      v[j] = ld16(sv + (int64_t(h * 128 + (item >> 1)) * BS + tg * 16 + (item & 1) * 8) * 2);
    }
    const bool odd = lane & 2;                  // an odd channel
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int c = (j * 64 + lane) >> 1;
      const int t0 = (lane & 1) * 8 + (odd ? 4 : 0);
#pragma unroll
      for (int q = 0; q < 2; ++q) {             // tokens t0 + 2q, t0 + 2q + 1
        const uint32_t keep = odd ? v[j][2 + q] : v[j][q];
        const uint32_t give = odd ? v[j][q] : v[j][2 + q];
        const uint32_t got = __builtin_amdgcn_mov_dpp(int(give), 0x4e, 0xf, 0xf, true);   // lane ^ 2
        const uint32_t even_c = odd ? got : keep, odd_c = odd ? keep : got;
        uint32_t* w = reinterpret_cast<uint32_t*>(&tw[(t0 + 2 * q) * kTileRow + (c & ~1)]);
        w[0] = (even_c & 0xffffu) | (odd_c << 16);
        w[kTileRow / 2] = (even_c >> 16) | (odd_c & 0xffff0000u);
      }
    }
    wave_lds_sync();
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int tl = j * 4 + (lane >> 4);
      const int cp = (lane & 15) * 8;
      const u32x4 out = *reinterpret_cast<const u32x4*>(&tw[tl * kTileRow + cp]);
      st16(dv + (int64_t((tg * 16 + tl) * H + h) * 128 + cp) * 2, out);
    }
  }
}

// Layout change in 16 KiB tiles, one per workgroup: T = min(BS, 64) tokens of
// 64 / T heads for V, 16 tokens of 4 heads (or fewer heads and more tokens
// where H is not a multiple of 4) for K, always 64 (token, head) rows of 256
// bytes. In the token-major layout such a tile is pieces of several adjacent
// heads per token, in the local layout whole rows.
template <int T>
__global__ __launch_bounds__(256) void block_relayout_kernel(PoolView pv, CopyIds ids, int32_t n,
                                                             int32_t* err_count, TableRewrite rw) {
  constexpr int kHeads = 64 / T;            // heads of a V tile
  constexpr int kGroups = T / 8;            // 8-token groups of a tile row
  __shared__ __attribute__((aligned(16))) uint16_t tile[64 * 128];
  if (int(blockIdx.x) < rw.n_groups) {
    rewrite_tables(rw, ids, blockIdx.x);
    return;
  }
  const int tid = threadIdx.x;
  const int tpb = int(pv.block_bytes / kTileBytes);
  const int32_t unit = int32_t(blockIdx.x) - rw.n_groups;   // a launch has at most 2^23 tiles
  if (unit >= n * tpb) return;
  const int32_t i = unit / tpb;
  const int k = unit - i * tpb;
  int32_t s, d;
  copy_ids(ids, __builtin_amdgcn_readfirstlane(i), s, d);
  const int32_t n_total = pv.n_local + pv.n_slice;
  if (s < 0 || s >= n_total || d < 0 || d >= n_total) {
    if (k == 0 && tid == 0) atomicAdd(err_count, 1);
    return;
  }
  const bool s_local = s < pv.n_local;
  const bool d_local = d < pv.n_local;
  const char* sb = s_local ? pv.local + int64_t(s) * pv.block_bytes
                           : pv.slice + int64_t(s - pv.n_local) * pv.block_bytes;
  char* db = d_local ? pv.local + int64_t(d) * pv.block_bytes
                     : pv.slice + int64_t(d - pv.n_local) * pv.block_bytes;
  u32x4 v[4];
  if (s_local == d_local) {                 // same layout: a straight copy
    const int64_t off = int64_t(k) * kTileBytes + tid * 16;
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = ld16(sb + off + j * 4096);
#pragma unroll
    for (int j = 0; j < 4; ++j) st16(db + off + j * 4096, v[j]);
    return;
  }
  const int H = pv.kv_heads;
  const int BS = pv.block_size;
  const int half_tiles = tpb / 2;
  const int64_t half_bytes = pv.block_bytes / 2;
  if (k < half_tiles) {
    // K: 256-byte rows change order only; row (h, t) is row h*BS + t of the
    // local layout and t*H + h of the token-major one
    const int hk = H % 4 == 0 ? 4 : H % 2 == 0 ? 2 : 1;
    const int tk = 64 / hk < BS ? 64 / hk : BS;
    const int hg = 64 / tk;
    const int tgs = BS / tk;
    const int h0 = (k / tgs) * hg;
    const int t0 = (k % tgs) * tk;
    int64_t nhd[4], att[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int row = j * 16 + (tid >> 4);
      const int t = t0 + row / hg, h = h0 + row % hg;
      nhd[j] = (int64_t(t) * H + h) * 256 + (tid & 15) * 16;
      att[j] = (int64_t(h) * BS + t) * 256 + (tid & 15) * 16;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = ld16(sb + (s_local ? att[j] : nhd[j]));
#pragma unroll
    for (int j = 0; j < 4; ++j) st16(db + (d_local ? att[j] : nhd[j]), v[j]);
    return;
  }
  // V: transposed between [token][channel] and [channel][token] in LDS. The
  // tile holds 16-byte pieces (8 channels) of row (head, token); piece p of
  // token t sits at p ^ swizzle(t), so that lanes which differ in their
  // 8-token group reach different banks.
  const int tgs = BS / T;
  const int kv = k - half_tiles;
  const int h0 = (kv / tgs) * kHeads;
  const int t0 = (kv % tgs) * T;
  auto at = [](int hh, int t, int c) {      // element of the tile
    const int sw = (t >> 3) * (8 / kGroups);
    return (hh * T + t) * 128 + ((((c >> 3) ^ sw) << 3) | (c & 7));
  };
  int64_t nhd[4], att[4];
  int row_h[4], row_t[4], col_h[4], col_c[4], col_t[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int row = j * 16 + (tid >> 4);    // token-major side: 16 lanes per row
    row_t[j] = row / kHeads;
    row_h[j] = row % kHeads;
    nhd[j] = half_bytes + (int64_t(t0 + row_t[j]) * H + h0 + row_h[j]) * 256 + (tid & 15) * 16;
    const int item = j * 256 + tid;         // local side: kGroups lanes per channel
    col_t[j] = (item % kGroups) * 8;
    col_c[j] = (item / kGroups) % 128;
    col_h[j] = item / (kGroups * 128);
    att[j] = half_bytes + (int64_t((h0 + col_h[j]) * 128 + col_c[j]) * BS + t0 + col_t[j]) * 2;
  }
  if (d_local) {
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = ld16(sb + nhd[j]);
#pragma unroll
    for (int j = 0; j < 4; ++j)
      *reinterpret_cast<u32x4*>(&tile[at(row_h[j], row_t[j], (tid & 15) * 8)]) = v[j];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      uint32_t w[4];
#pragma unroll
      for (int q = 0; q < 4; ++q)
        w[q] = uint32_t(tile[at(col_h[j], col_t[j] + 2 * q, col_c[j])]) |
               (uint32_t(tile[at(col_h[j], col_t[j] + 2 * q + 1, col_c[j])]) << 16);
      st16(db + att[j], u32x4{w[0], w[1], w[2], w[3]});
    }
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = ld16(sb + att[j]);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t w[4] = {v[j].x, v[j].y, v[j].z, v[j].w};
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        tile[at(col_h[j], col_t[j] + 2 * q, col_c[j])] = uint16_t(w[q] & 0xffffu);
        tile[at(col_h[j], col_t[j] + 2 * q + 1, col_c[j])] = uint16_t(w[q] >> 16);
      }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 4; ++j)
      st16(db + nhd[j], *reinterpret_cast<const u32x4*>(&tile[at(row_h[j], row_t[j], (tid & 15) * 8)]));
  }
}

// Same-layout copy (both pools in the local layout): wave w of workgroup g
// moves piece g * kWaves + w -- xcd_item(g) * kWaves + w where blocks are Dealt
// to the XCDs -- 2 KiB of block src_ids[i], to the same offset of block
// dst_ids[i]. Out-of-range ids are skipped and counted once per block.
template <bool Dealt>
__global__ __launch_bounds__(256) void block_copy_same_kernel(PoolView pv, CopyIds ids,
                                                              int32_t n, int32_t* err_count,
                                                              TableRewrite rw, uint32_t xcd_run,
                                                              uint32_t xcd_limit) {
  if (int(blockIdx.x) < rw.n_groups) {
    rewrite_tables(rw, ids, blockIdx.x);
    return;
  }
  const int lane = threadIdx.x & 63;
  const uint32_t ppb = uint32_t(pv.block_bytes / kPieceBytes);
  // a launch has at most 2^25 wavefronts: pieces fit in 32 bits
  const uint32_t g = blockIdx.x - rw.n_groups;
  const uint32_t piece = (Dealt ? xcd_item(g, xcd_run, xcd_limit) : g) * kWaves + (threadIdx.x >> 6);
  if (piece >= uint32_t(n) * ppb) return;
  const int32_t i = int32_t(piece / ppb);
  const int k = int(piece - uint32_t(i) * ppb);
  int32_t s, d;
  copy_ids(ids, __builtin_amdgcn_readfirstlane(i), s, d);
  const int32_t n_total = pv.n_local + pv.n_slice;
  if (s < 0 || s >= n_total || d < 0 || d >= n_total) {
    if (k == 0 && lane == 0) atomicAdd(err_count, 1);
    return;
  }
  const char* sb = s < pv.n_local ? pv.local + int64_t(s) * pv.block_bytes
                                  : pv.slice + int64_t(s - pv.n_local) * pv.block_bytes;
  char* db = d < pv.n_local ? pv.local + int64_t(d) * pv.block_bytes
                            : pv.slice + int64_t(d - pv.n_local) * pv.block_bytes;
  const int64_t off = int64_t(k) * kPieceBytes + lane * 16;
  const u32x4 v0 = ld16(sb + off);
  const u32x4 v1 = ld16(sb + off + 1024);
  st16(db + off, v0);
  st16(db + off + 1024, v1);
}

// Same-layout copy of a list of scattered blocks, one wavefront per workgroup:
// workgroup (k, y, z) moves 2 KiB piece k of block z * kListRows + y. The grid
// gives piece and block, so nothing is divided, and the few arguments come in
// one load: a wavefront lives only for its ids, its two loads and its two
// stores, and how long it lives sets how many bytes a CU keeps in flight.
// Against the same with one more division and the general kernel's arguments, in
// us: 64 blocks of 64 KiB 3.49 / 3.31, 256 8.1 / 7.7, 1024 28.1 / 27.8, 9801 209.0 /
// 207.5 (6.19 TB/s); blocks of 8 KiB, 64 2.67 / 2.45, 1024 6.1 / 6.3, 10000 34.8 /
// 34.7. With four wavefronts to a workgroup 9801 go at 6.02 TB/s.
constexpr int kListRows = 32768;
__global__ __launch_bounds__(64) void block_copy_list_kernel(
    char* local, char* slice, const int32_t* __restrict__ src, const int32_t* __restrict__ dst,
    int64_t block_bytes, int32_t n_local, int32_t n_total, int32_t n, int32_t* err_count) {
  const int32_t i = int32_t(blockIdx.z) * kListRows + int32_t(blockIdx.y);
  if (i >= n) return;
  const int32_t s = src[i];
  const int32_t d = dst[i];
  const int lane = threadIdx.x;
  if (uint32_t(s) >= uint32_t(n_total) || uint32_t(d) >= uint32_t(n_total)) {
    if (blockIdx.x == 0 && lane == 0) atomicAdd(err_count, 1);
    return;
  }
  const int64_t off = int64_t(blockIdx.x) * kPieceBytes + lane * 16;
  const char* sp = (s < n_local ? local + int64_t(s) * block_bytes
                                : slice + int64_t(s - n_local) * block_bytes) + off;
  char* dp = (d < n_local ? local + int64_t(d) * block_bytes
                          : slice + int64_t(d - n_local) * block_bytes) + off;
  const u32x4 v0 = ld16(sp);
  const u32x4 v1 = ld16(sp + 1024);
  st16(dp, v0);
  st16(dp + 1024, v1);
}

// One workgroup per (sequence, KV head), one thread per channel: the K element
// goes to the token's row, the V element to the token's column of the
// transposed V rows.
__global__ __launch_bounds__(128) void kv_append_kernel(PoolView pv, const uint16_t* __restrict__ k_new,
                                                        const uint16_t* __restrict__ v_new,
                                                        const int32_t* __restrict__ table,
                                                        const int32_t* __restrict__ seq_lens,
                                                        int32_t max_blocks, int32_t* err_count) {
  const int b = blockIdx.x;
  const int h = blockIdx.y;
  const int d = threadIdx.x;
  const int H = pv.kv_heads;
  const int BS = pv.block_size;
  const int len = seq_lens[b];
  if (len <= 0) return;
  const int p = len - 1;
  const int j = p / BS;
  const int32_t id = j < max_blocks ? table[int64_t(b) * max_blocks + j] : -1;
  if (id < 0 || id >= pv.n_local) {
    if (h == 0 && d == 0) atomicAdd(err_count, 1);
    return;
  }
  const int r = p - j * BS;
  uint16_t* blk = reinterpret_cast<uint16_t*>(pv.local + int64_t(id) * pv.block_bytes);
  const int64_t src = (int64_t(b) * H + h) * 128 + d;
  blk[(int64_t(h) * BS + r) * 128 + d] = k_new[src];
  blk[int64_t(BS) * H * 128 + (int64_t(h) * 128 + d) * BS + r] = v_new[src];
}

}  // namespace

namespace {

hipError_t launch_copy(const PoolView& pv, CopyIds ids, int32_t n, int32_t* err_count,
                       hipStream_t stream, bool runs, const TableRewrite* rw) {
  TableRewrite rwl;
  if (rw && rw->n_entries > 0) {
    rwl = *rw;
    rwl.n_groups = int32_t((rw->n_entries + kRewriteEntries - 1) / kRewriteEntries);
  }
  if (n <= 0 && rwl.n_groups == 0) return hipSuccess;
  const bool same = pv.slice_layout == 0;
  // Tiles are min(BS, 64) tokens of whole groups of heads; block size 16 does
  // better in 4 KiB units.
  const bool tiled = !same && pv.block_size >= 32 && (pv.block_size >= 64 || pv.kv_heads % 2 == 0);
  const int64_t upb = pv.block_bytes / (same ? kPieceBytes : kUnitBytes);   // waves per block
  // scattered lists of blocks of up to 64 KiB, at most 2^22 pieces
  if (same && !runs && rwl.n_groups == 0 && ids.n_runs == 0 && ids.dst && pv.block_bytes <= 65536 &&
      int64_t(n) * upb <= (int64_t(1) << 22)) {
    const unsigned rows = unsigned(std::min(n, kListRows));
    hipLaunchKernelGGL(block_copy_list_kernel,
                       dim3(unsigned(upb), rows, unsigned((n + kListRows - 1) / kListRows)),
                       dim3(64), 0, stream, pv.local, pv.slice, ids.src, ids.dst, pv.block_bytes,
                       pv.n_local, pv.n_local + pv.n_slice, n, err_count);
    return hipGetLastError();
  }
  const size_t lds = same || tiled ? 0 : size_t(kWaves) * tile_elems(pv.block_size) * 2;
  // A launch stays below 2^32 work-items: at most 2^25 wavefronts. The table
  // rewrite rides on the first launch; lists are split, run plans always fit.
  const int64_t max_blocks = std::max<int64_t>(1, (int64_t(1) << 25) / upb);
  if (ids.n_runs > 0 && n > max_blocks) return hipErrorInvalidValue;
  int64_t b0 = 0;
  do {
    const int32_t m = int32_t(std::max<int64_t>(0, std::min<int64_t>(max_blocks, n - b0)));
    const int64_t grid = (int64_t(m) * upb + kWaves - 1) / kWaves + rwl.n_groups;
    CopyIds part = ids;
    if (ids.n_runs == 0) {
      part.src = m ? ids.src + b0 : nullptr;
      part.dst = m && ids.dst ? ids.dst + b0 : nullptr;
      part.dst_base = ids.dst ? 0 : int32_t(ids.dst_base + b0);
    }
    if (same) {
      // scattered large blocks: whole workgroups of a block, up to 256 KiB, to
      // an XCD; full rounds only
      const int64_t groups = int64_t(m) * upb / kWaves;
      const uint32_t run = uint32_t(std::min(upb, kXcdRunBytes / kPieceBytes) / kWaves);
      const uint32_t limit = uint32_t(groups / (8 * int64_t(run)) * (8 * int64_t(run)));
      const bool dealt = !runs && pv.block_bytes > 65536;
      hipLaunchKernelGGL(dealt ? block_copy_same_kernel<true> : block_copy_same_kernel<false>,
                         dim3(unsigned(grid)), dim3(256), 0, stream, pv, part, m, err_count, rwl,
                         run, limit);
    } else if (tiled) {
      hipLaunchKernelGGL(pv.block_size >= 64 ? block_relayout_kernel<64>
                                             : block_relayout_kernel<32>,
                         dim3(unsigned(grid)), dim3(256), 0, stream, pv, part, m, err_count,
                         rwl);
    } else {
      hipLaunchKernelGGL(block_copy_kernel, dim3(unsigned(grid)), dim3(256), lds, stream, pv,
                         part, m, err_count, rwl);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    rwl.n_groups = 0;
    b0 += m;
  } while (b0 < n);
  return hipSuccess;
}

}  // namespace

hipError_t launch_block_copy(const PoolView& pv, const int32_t* src, const int32_t* dst,
                             int32_t n, int32_t* err_count, hipStream_t stream, bool runs,
                             const TableRewrite* rw, int32_t dst_base) {
  CopyIds ids;
  ids.src = src;
  ids.dst = dst;
  ids.dst_base = dst_base;
  return launch_copy(pv, ids, n, err_count, stream, runs, rw);
}

hipError_t launch_block_copy_runs(const PoolView& pv, const int32_t* src_first,
                                  const int32_t* dst_first, const int32_t* len, int32_t n_runs,
                                  int32_t* err_count, hipStream_t stream,
                                  const TableRewrite* rw) {
  if (n_runs < 0 || n_runs > kArgRuns) return hipErrorInvalidValue;
  CopyIds ids;
  ids.n_runs = n_runs;
  int64_t n = 0;
  for (int32_t r = 0; r < n_runs; ++r) {
    ids.run_src[r] = src_first[r];
    ids.run_dst[r] = dst_first[r];
    ids.run_off[r] = int32_t(n);
    n += len[r];
  }
  ids.run_off[n_runs] = int32_t(n);
  if (n > INT32_MAX) return hipErrorInvalidValue;
  return launch_copy(pv, ids, int32_t(n), err_count, stream, true, rw);
}

hipError_t launch_kv_append(const PoolView& pv, const void* k_new, const void* v_new,
                            const int32_t* table, const int32_t* seq_lens, int32_t batch,
                            int32_t max_blocks, int32_t* err_count, hipStream_t stream) {
  if (batch <= 0) return hipSuccess;
  hipLaunchKernelGGL(kv_append_kernel, dim3(unsigned(batch), unsigned(pv.kv_heads)), dim3(128), 0,
                     stream, pv, static_cast<const uint16_t*>(k_new),
                     static_cast<const uint16_t*>(v_new), table, seq_lens, max_blocks, err_count);
  return hipGetLastError();
}

}  // namespace ema
