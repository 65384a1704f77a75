// Paged decode attention on the matrix cores (gfx950 MFMA 16x16x32).
//
// With grouped-query attention the G query heads that share a KV head turn
// decode into a small dense contraction per KV head: [G x 128] . [128 x T] for
// the scores and [G x T] . [T x 128] for the output. Both go to
// v_mfma_f32_16x16x32_{bf16,f16} (G <= 16 heads fill one 16-wide tile), which
// leaves the vector ALUs nearly idle and the kernel bound by HBM.
//
// Work is cut into 32-token tiles of one (sequence, KV head). Each wavefront
// streams tiles with an online softmax, the next tile's loads in flight while
// one is consumed:
//   scores   S^T[token][head] = K . Q^T   (A = 16 K rows straight from the
//            block, B = Q^T held in registers; two 16-token tiles whose rows
//            are chosen so that each lane ends up holding 8 consecutive
//            tokens of one head -- exactly the B-operand layout of the next
//            product, so no data moves between lanes)
//   output   O^T[channel][head] += V^T . P^T  (A = 16 channel rows of the
//            transposed V block, 8 consecutive tokens per lane, 16 B loads;
//            P is split into a 16-bit high part and a 16-bit remainder so the
//            probabilities keep ~16 significant bits)
// Scheduling is stream-K: the tiles of all (sequence, KV head) pairs, in that
// order, are split into equal contiguous ranges, one per wavefront, four
// wavefronts to a workgroup and one workgroup per CU, so every CU streams the
// same bytes whatever the length mix. A wavefront works alone until its range
// is done: a pair it covers whole it writes out itself, with no barrier; the
// pieces of pairs cut by range boundaries are merged at the end of the
// workgroup's range, in LDS within the workgroup, and by a small combine kernel
// where a pair crosses a workgroup boundary. Merging across workgroups inside
// this kernel costs more: partials must cross XCDs, whose L2s are not
// coherent, either behind device-scope fences (a whole-L2 write-back and
// invalidation per workgroup) or as written-through stores plus an arrival
// counter, and either way at the end of every workgroup's range.
//
// What bounds it: HBM. Scattered 4 KiB pieces (one head's K or V of a 16-token
// block at 8 KV heads) read at 6.65 TB/s on this GPU, contiguous memory at
// 6.9-7.2. Against workgroups whose four waves shared one range and met at a
// barrier after every pair (and staged each pair anew where a range did not
// fit its lists), in us a call: an 8B-shaped layer (64 sequences of 1024-4096
// tokens, 673 MB) 113.4 -> 109.5, 512 sequences of 17-1000 tokens (1.07 GB)
// 230 -> 177, a 70B share (211 MB) 43.7 -> 41.5, four of 20-120 thousand tokens
// 185.5 -> 180; 256 sequences of 17-300 tokens 72.4 -> 39.5. By timestamps in
// the 8B call: workgroups start over the first 2.3 us (XCDs one after another),
// have their plan after 0.75 us, the first tile after another 2.5; waves end
// between 97 and 108 us -- equal bytes at unequal rates, of which only a third
// repeats from call to call -- and the merge takes 1-1.6 us. Eight wavefronts
// to a workgroup: 8B +2 %, 70B share +9 %. A loop written so that every wait
// lets the next tile's loads stay in flight: 8B +2 %, long +2 %.
//
// Masked tokens (past the length, or in a block whose id is out of range) get
// -inf scores and zeroed V, so NaN in unused slots never leaks. Reduction
// orders depend only on the sequence lengths, not on block ids or the table's
// width.
#include "attn_store.h"
#include "kernels.h"

#include <algorithm>
#include <cmath>
#include <mutex>
#include <unordered_map>

namespace ema {
namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kD = 128;
constexpr int kWaves = 4;
constexpr int kThreads = kWaves * 64;
constexpr int kStreamWaves = 4;            // stream-K form
constexpr int kStreamThreads = kStreamWaves * 64;
constexpr int kShortRuns = 8;              // of a short pair
constexpr int kShortPair = -2;             // its combine record where each run left a partial
constexpr int kDirectWaves = kShortRuns;   // direct form
constexpr int kDirectThreads = kDirectWaves * 64;
constexpr int kCombineWaves = 4;           // stream-K form's combine
constexpr int kIt = 32;                    // tokens per tile (one wave iteration)
constexpr int kPieceTiles = 32;            // tiles whose block ids are staged in LDS at once
constexpr int kMaxIds = kPieceTiles * kIt / 16;
constexpr int kGridChunkTiles = 32;        // tiles per workgroup in the grid fallback
// Tokens of a short pair, in a batch of so many pairs (see attn_mfma_direct); 0:
// no pair counts as short.
__host__ __device__ constexpr int short_tokens(int64_t pairs) {
  return pairs <= 256 ? 2 * kShortRuns * kIt : pairs <= 512 ? kShortRuns * kIt : 0;
}
// Every pair a wave touches costs it about a tile's time beyond its tiles (the
// result goes through LDS, new queries and block ids arrive); the stream-K
// split counts it as kSegCost tiles. Measured, in us, for 0 / 1 / 2 / 3: an 8B
// layer 112.1 / 112.0 / 111.8 / 111.4, a 70B share 44.2 / 43.0 / 43.1 / 43.0,
// 512 sequences of 17-1000 tokens 204 / 181 / 180 / 182. At 16 query heads to
// each of 8 KV heads, whose partials are four times larger, for 1 / 2 / 4 / 8: 256
// sequences of 17-1000 tokens 109 / 102 / 104 / 108, 512 of them 210 / 201 / 205 /
// 215, 64 of 500-4000 104.2 / 103.6 / 105.2 / 105.1.
constexpr int kSegCost = 2;

__device__ __forceinline__ u32x4 ld16(const char* p) {
  return *reinterpret_cast<const u32x4*>(p);
}
// K/V are read exactly once per call: streaming loads keep them from
// displacing tables, queries and partials in L2 and the memory-side cache.
__device__ __forceinline__ u32x4 ld16_stream(const char* p) {
  return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
}
// But a line that a wave reads in two halves, tiles apart, has to stay in L2 in
// between, and a streamed one may not: from block size 64 on a tile's V rows
// are 64-byte pieces of rows of 128 bytes and more, the rest of which the next
// tile reads. Measured, us a call with K and V streamed / V kept / both kept: 64
// sequences of 1024-4096 tokens, 8 KV heads, block size 64 158 / 130 / 128, 256
// 157 / 131 / 127; streamed / K kept / both kept: block size 16 108.1 / 108.7 /
// 119, block size 32, one KV head, 128 sequences 44.1 / 44.6 / 48.5.
template <int BS>
__device__ __forceinline__ u32x4 ld16_kv(const char* p) {
  return BS >= 64 ? ld16(p) : ld16_stream(p);
}

template <bool BF16>
__device__ __forceinline__ f32x4 mfma(u32x4 a, u32x4 b, f32x4 c) {
  if constexpr (BF16)
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                   __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a),
                                                  __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}

// p -> (high, low) 16-bit parts with p ~= high + low, both rounded to nearest
// even: the remainder is exact, and the sum keeps 17 (bf16) or 22 bits of p. (A
// truncated high part leaves a bf16 remainder, and with it an error of the whole
// call, twice as large.)
template <bool BF16>
__device__ __forceinline__ void split16(float p, uint32_t& hi, uint32_t& lo) {
  if constexpr (BF16) {
    const uint32_t u = __builtin_bit_cast(uint32_t, p);
    hi = (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
    const float r = p - __builtin_bit_cast(float, hi << 16);
    const uint32_t v = __builtin_bit_cast(uint32_t, r);
    lo = (v + 0x7fffu + ((v >> 16) & 1u)) >> 16;
  } else {
    const _Float16 h = _Float16(p);
    const _Float16 l = _Float16(p - float(h));
    hi = __builtin_bit_cast(uint16_t, h);
    lo = __builtin_bit_cast(uint16_t, l);
  }
}

__device__ __forceinline__ int clamp_len(int len, const AttnArgs& a) {
  const int cap = a.max_blocks * a.block_size;
  return len < 0 ? 0 : (len > cap ? cap : len);
}

// One 32-token iteration's operands: K rows of the two score tiles and the
// eight V^T row tiles, plus how many of this lane's 8 tokens are valid.
struct Tile {
  u32x4 k[2][4];
  u32x4 v[8];
  int nv;
};

// Issues the loads of the tile starting at token t0 of the sequence. Every lane
// loads unconditionally (a lane whose token is masked reads block 0, which
// always exists), so the loads stay in straight-line code and the compiler can
// wait for this tile alone while the next one is in flight. K rows of masked
// tokens only reach scores that consume_tile sets to -inf; V of masked tokens
// is zeroed there before use.
template <int BS>
__device__ __forceinline__ void load_tile(Tile& T, int t0, int len, int blk0, const int32_t* s_ids,
                                          const char* pool, int64_t Bb, int kvh, int r16,
                                          int q4) {
  // K rows: tile t, row r16 -> token t0 + 8*(r16/4) + 4t + r16%4.
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int tok = t0 + 8 * (r16 >> 2) + 4 * t + (r16 & 3);
    const int id = s_ids[tok / BS - blk0];
    const bool ok = tok < len && id >= 0;
    const char* p = pool + (ok ? int64_t(id) * Bb + (int64_t(kvh * BS + tok % BS) * kD + q4 * 8) * 2
                               : int64_t(0));
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) T.k[t][kk] = ld16_stream(p + kk * 64);
  }
  // V^T rows: d-tile n, row 16n + r16, tokens t0 + 8q4 .. +8 (one block).
  const int vt = t0 + 8 * q4;
  const int vid = s_ids[vt / BS - blk0];
  const int vleft = len - vt;
  T.nv = vid < 0 ? 0 : (vleft < 0 ? 0 : (vleft > 8 ? 8 : vleft));
  const char* p = pool + (T.nv > 0 ? int64_t(vid) * Bb + Bb / 2 +
                                         (int64_t(kvh * kD + r16) * BS + vt % BS) * 2
                                   : int64_t(0));
#pragma unroll
  for (int n = 0; n < 8; ++n) T.v[n] = ld16_stream(p + int64_t(16 * n) * BS * 2);
}

// Scores, online softmax update and P.V for one loaded iteration.
// `issue_next` runs right after the score products are issued: loads of the
// next tile then queue behind this tile's V loads, so the in-order wait
// before P.V covers this tile only.
//
// A wave may add hundreds of tiles to one output, so what is rounded at the
// output's magnitude is kept to one multiplication and one addition a tile: the
// products of the high and the low parts are each summed from zero in the
// matrix cores (which round what they add to an accumulator after every few
// products, and the low parts against the larger sum) and then added. Relative
// error against 64 bits, of outputs accumulated in the matrix cores from tile to
// tile with P's high part truncated / as it is: 64 sequences of 1024-4096
// tokens, bf16 4.33e-6 / 2.17e-6, f16 3.87e-7 / 2.80e-7; 64 of 17-1000, f16
// 2.14e-7 / 1.91e-7; 120000 tokens, f16 4.28e-7 / 3.18e-7 (both parts into one
// sum from zero, the low one first: 5.23e-7). Multiplication and addition are
// not contracted: the fused form writes the product's registers, and the moves
// that follow from it spill (8B-shaped layer 109.5 -> 111 us, short calls
// +0.7 us). Four output rows at a time: all eight need 10 registers more.
template <bool BF16, typename Next>
__device__ __forceinline__ void consume_tile(Tile& T, const u32x4 (&qb)[4], float scale_log2,
                                             float& m, float& lsum, f32x4 (&o)[8],
                                             Next&& issue_next) {
#pragma clang fp contract(off)   // the same roundings wherever this is inlined
  const int nv = T.nv;
  // Scores for tokens 8q4 + 4t + i of head r16.
  f32x4 s[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    s[t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) s[t] = mfma<BF16>(T.k[t][kk], qb[kk], s[t]);
  }
  issue_next();
  float sv[8];
  float mx = -INFINITY;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    sv[j] = j < nv ? s[j >> 2][j & 3] * scale_log2 : -INFINITY;
    mx = fmaxf(mx, sv[j]);
  }
  mx = fmaxf(mx, __shfl_xor(mx, 16));
  mx = fmaxf(mx, __shfl_xor(mx, 32));
  const float m_new = fmaxf(m, mx);
  const float alpha = m_new == -INFINITY ? 1.0f : exp2f(m - m_new);
  uint32_t ph[4], pl[4];
  float ps = 0.0f;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const float p0 = m_new == -INFINITY ? 0.0f : exp2f(sv[2 * q] - m_new);
    const float p1 = m_new == -INFINITY ? 0.0f : exp2f(sv[2 * q + 1] - m_new);
    ps += p0 + p1;
    uint32_t h0, l0, h1, l1;
    split16<BF16>(p0, h0, l0);
    split16<BF16>(p1, h1, l1);
    ph[q] = h0 | (h1 << 16);
    pl[q] = l0 | (l1 << 16);
  }
  lsum = fmaf(lsum, alpha, ps);
  m = m_new;
#pragma unroll
  for (int q = 0; q < 4; ++q) {   // branch-free, so waits stay per tile
    const uint32_t keep = (2 * q < nv ? 0xffffu : 0u) | (2 * q + 1 < nv ? 0xffff0000u : 0u);
#pragma unroll
    for (int n = 0; n < 8; ++n) T.v[n][q] &= keep;
  }
  const u32x4 PH = {ph[0], ph[1], ph[2], ph[3]};
  const u32x4 PL = {pl[0], pl[1], pl[2], pl[3]};
  const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int n0 = 0; n0 < 8; n0 += 4) {
    f32x4 t[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
      t[i] = mfma<BF16>(T.v[n0 + i], PH, zero) + mfma<BF16>(T.v[n0 + i], PL, zero);
#pragma unroll
    for (int i = 0; i < 4; ++i) o[n0 + i] = o[n0 + i] * alpha + t[i];
  }
}

template <int G>
struct Smem {
  int32_t ids[kMaxIds];
  __attribute__((aligned(16))) float o[kWaves][G][kD];
  float m[kWaves][G];
  float l[kWaves][G];
};

// Attends tiles [j0, j1) of (sequence b, KV head kvh) with all four waves
// (wave w takes tiles j0 + w, j0 + w + 4, ...; two tiles in flight) and hands
// the merged (max, sum, unnormalised output) of each (head g, channel d) to
// emit(), with the (g, d) pairs spread over the workgroup's threads.
template <int G, int BS, bool BF16, typename Emit>
__device__ __forceinline__ void attend_segment(const AttnArgs& a, int b, int kvh, int len, int j0,
                                               int j1, Smem<G>& sm, Emit&& emit) {
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int r16 = lane & 15;
  const int q4 = lane >> 4;
  // Q^T as the B operand: lane (head r16, q4) holds channels 32kk + 8q4 .. +8.
  u32x4 qb[4];
  {
    const char* qrow = reinterpret_cast<const char*>(a.q) +
                       (int64_t(b) * a.q_heads + kvh * G + r16) * kD * 2 + q4 * 16;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
      qb[kk] = r16 < G ? ld16(qrow + kk * 64) : u32x4{0, 0, 0, 0};
  }
  const char* pool = a.local;
  const int64_t Bb = a.block_bytes;
  float m = -INFINITY;   // running max of this lane's head (log2 domain)
  float lsum = 0.0f;     // this lane's share of the running sum
  f32x4 o[8];
#pragma unroll
  for (int n = 0; n < 8; ++n) o[n] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

  for (int p0 = j0; p0 < j1; p0 += kPieceTiles) {
    const int p1 = min(j1, p0 + kPieceTiles);
    const int blk0 = p0 * kIt / BS;
    const int cnt = (p1 * kIt - 1) / BS - blk0 + 1;
    __syncthreads();                      // the previous piece's ids are no longer read
    if (tid < cnt) {
      const int j = blk0 + tid;
      int id = -1;
      if (j * BS < len) {
        id = a.table[int64_t(b) * a.max_blocks + j];
        if (id < 0 || id >= a.n_local) {
          atomicAdd(a.err_count, 1);
          id = -1;
        }
      }
      sm.ids[tid] = id;
    }
    __syncthreads();
    const int nt = p1 - p0;
    const int n_it = nt > wave ? (nt - wave + kWaves - 1) / kWaves : 0;
    auto load_at = [&](Tile& T, int k) {
      load_tile<BS>(T, (p0 + wave + k * kWaves) * kIt, len, blk0, sm.ids, pool, Bb, kvh, r16, q4);
    };
    Tile A, B;
    if (n_it > 0) load_at(A, 0);
    for (int it = 0; it < n_it; it += 2) {
      consume_tile<BF16>(A, qb, a.scale_log2, m, lsum, o, [&] {
        if (it + 1 < n_it) load_at(B, it + 1);
      });
      if (it + 1 >= n_it) break;
      consume_tile<BF16>(B, qb, a.scale_log2, m, lsum, o, [&] {
        if (it + 2 < n_it) load_at(A, it + 2);
      });
    }
  }

  // ---- merge the four waves ------------------------------------------------
  lsum += __shfl_xor(lsum, 16);
  lsum += __shfl_xor(lsum, 32);
  if (r16 < G) {
    if (q4 == 0) {
      sm.m[wave][r16] = m;
      sm.l[wave][r16] = lsum;
    }
#pragma unroll
    for (int n = 0; n < 8; ++n)
      *reinterpret_cast<f32x4*>(&sm.o[wave][r16][16 * n + 4 * q4]) = o[n];
  }
  __syncthreads();
  for (int e = tid; e < G * kD; e += kThreads) {
    const int g = e / kD;
    const int d = e % kD;
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) M = fmaxf(M, sm.m[w][g]);
    float L = 0.0f, O = 0.0f;
    if (M != -INFINITY) {
#pragma unroll
      for (int w = 0; w < kWaves; ++w) {
        const float mw = sm.m[w][g];
        if (mw == -INFINITY) continue;
        const float f = exp2f(mw - M);
        L = fmaf(f, sm.l[w][g], L);
        O = fmaf(f, sm.o[w][g][d], O);
      }
    }
    emit(g, d, M, L, O);
  }
}

// Wave-uniform value kept in a scalar register.
__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }

// o / l, given inv = 1 / l, one correction step: within an ulp of the division
// at a fraction of its instructions (l is 1 or more: the row's largest
// probability is 1). Infinities pass through uncorrected.
__device__ __forceinline__ float div_by(float o, float l, float inv) {
  const float q = o * inv;
  const float c = fmaf(fmaf(-q, l, o), inv, q);
  return fabsf(q) < INFINITY ? c : q;
}

// ---- one wavefront's stream of tiles -------------------------------------------------
//
// A wavefront streams a list of groups: up to 64 consecutive blocks of one
// segment, whose ids it holds one per lane. A segment is a run of tiles
// [j0, j1) of one (sequence, KV head) pair. Everything in Group is uniform
// over the wave.
struct Group {
  int b, kvh, len;
  int nt;             // tiles of the pair
  int j0, j1;         // the segment
  int g0, g1;         // the group's tiles
  int blk;            // the group's first block
};

// Whether block g.blk + lane belongs to the group's tiles.
template <int BS>
__device__ __forceinline__ bool in_group(const Group& g, int lane) {
  return (g.blk + lane) * BS < min(g.len, g.g1 * kIt);
}

// Table entry of block g.blk + lane; lanes past the group read its first one.
// The value is not looked at here, so nothing waits for the load.
template <int BS>
__device__ __forceinline__ int32_t load_group_ids(const AttnArgs& a, const Group& g, int lane) {
  const int j = g.blk + (in_group<BS>(g, lane) ? lane : 0);
  return a.table[int64_t(g.b) * a.max_blocks + j];
}

// The group's ids: -1 past its tiles and for ids outside the local pool, which
// are counted.
template <int BS>
__device__ __forceinline__ int32_t check_group_ids(const AttnArgs& a, const Group& g, int lane,
                                                   int32_t id) {
  const bool in = in_group<BS>(g, lane);
  const bool ok = uint32_t(id) < uint32_t(a.n_local);
  if (in && !ok) atomicAdd(a.err_count, 1);
  return in && ok ? id : -1;
}

// Issues the loads of tile j of group g. Block ids come from lane registers,
// so a block's address is uniform and only the offset inside it is per lane.
// Lanes whose token lies past the length re-read the tile's first rows (they
// are masked in consume_tile); a block whose id is out of range reads block 0,
// which always exists, and is masked too.
template <int BS>
__device__ __forceinline__ void load_tile_ids(Tile& T, const AttnArgs& a, const Group& g, int32_t ids,
                                              int j, int r16, int q4) {
  const int t0 = j * kIt;
  const int lb = t0 / BS - g.blk;
  const int left = g.len - t0;
  const int id0 = __builtin_amdgcn_readlane(ids, lb);
  const int64_t Bb = a.block_bytes;
  const char* base0 = a.local + int64_t(id0 < 0 ? 0 : id0) * Bb;
  const char* base1 = base0;
  int id1 = id0;
  if constexpr (BS == 16) {
    id1 = __builtin_amdgcn_readlane(ids, lb + 1);
    base1 = a.local + int64_t(id1 < 0 ? 0 : id1) * Bb;
  }
  const int tb = BS > kIt ? t0 % BS : 0;         // the tile's first token in its block
  const int khead = (g.kvh * BS + tb) * kD * 2;
  // K rows: tile t, row r16 -> token t0 + 8*(r16/4) + 4t + r16%4.
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int tok = 8 * (r16 >> 2) + 4 * t + (r16 & 3);
    const bool in = tok < left;
    const int row = in ? (BS == 16 ? tok & 15 : tok) : 0;
    const char* base = (BS == 16 && in && tok >= 16) ? base1 : base0;
    const char* p = base + (khead + row * kD * 2 + q4 * 16);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) T.k[t][kk] = ld16_kv<BS>(p + kk * 64);
  }
  // V^T rows: d-tile n, row 16n + r16, tokens t0 + 8q4 .. +8 (one block).
  const int vt = 8 * q4;
  const bool vin = vt < left;
  const bool second = BS == 16 && vin && q4 >= 2;
  T.nv = !vin || (second ? id1 : id0) < 0 ? 0 : min(left - vt, 8);
  const int vrow = vin ? r16 * BS + (BS == 16 ? vt & 15 : vt) : 0;
  const int64_t vhead = Bb / 2 + (g.kvh * kD * BS + tb) * 2;
  const char* p = (second ? base1 : base0) + vhead + vrow * 2;
#pragma unroll
  for (int n = 0; n < 8; ++n) T.v[n] = ld16_kv<BS>(p + 16 * n * BS * 2);
}

// Q^T of one pair as the B operand: lane (head r16, q4) holds channels
// 32kk + 8q4 .. +8. Lanes past G read head 0 (mask_q zeroes them).
template <int G>
__device__ __forceinline__ void load_q(u32x4 (&qn)[4], const AttnArgs& a, int b, int kvh, int r16,
                                       int q4) {
  const char* row = reinterpret_cast<const char*>(a.q) +
                    (int64_t(b) * a.q_heads + kvh * G + (r16 < G ? r16 : 0)) * kD * 2 + q4 * 16;
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) qn[kk] = ld16(row + kk * 64);
}
template <int G>
__device__ __forceinline__ void mask_q(u32x4 (&qb)[4], const u32x4 (&qn)[4], int r16) {
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) qb[kk] = r16 < G ? qn[kk] : u32x4{0, 0, 0, 0};
}

// Streams the wave's groups, first `g`, then whatever `next` makes of it
// (next(Group&) -> false when there is no further group), with one tile in
// flight while another is consumed and the block ids one group ahead. Neither
// segment ends nor id lists interrupt the loads: the first tile of the next
// segment and its queries are on their way before the current one is
// finished. finish(group, flags, m, lsum, o) gets each segment's result
// (running max and this lane's share of the sum).
template <int G, int BS, bool BF16, typename Next, typename Finish>
__device__ __forceinline__ void stream_wave(const AttnArgs& a, Group L, Next&& next,
                                            Finish&& finish) {
  const int lane = threadIdx.x & 63;
  const int r16 = lane & 15;
  const int q4 = lane >> 4;
  Group N = L;
  int32_t idn = load_group_ids<BS>(a, L, lane);
  u32x4 qb[4];
  Tile A, B;
  load_q<G>(B.k[0], a, L.b, L.kvh, r16, q4);
  int32_t ids = check_group_ids<BS>(a, L, lane, idn);
  int j = L.g0;
  load_tile_ids<BS>(A, a, L, ids, j, r16, q4);
  mask_q<G>(qb, B.k[0], r16);
  bool have_next = next(N);
  idn = load_group_ids<BS>(a, have_next ? N : L, lane);

  float m = -INFINITY;   // running max of this lane's head (log2 domain)
  float lsum = 0.0f;     // this lane's share of the running sum
  f32x4 o[8];
#pragma unroll
  for (int n = 0; n < 8; ++n) o[n] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

  // Consumes tile X (tile j of group L) while the following one loads into Y.
  bool more = true;
  auto turn = [&](Tile& X, Tile& Y) {
    const Group C = L;
    const bool last = j + 1 == L.j1;
    consume_tile<BF16>(X, qb, a.scale_log2, m, lsum, o, [&] {
      if (++j == L.g1) {
        more = have_next;
        if (more) {
          // into X's K registers, whose rows have been used
          if (last) load_q<G>(X.k[0], a, N.b, N.kvh, r16, q4);
          ids = check_group_ids<BS>(a, N, lane, idn);
          L = N;
          j = L.g0;
          have_next = next(N);
          idn = load_group_ids<BS>(a, have_next ? N : L, lane);
        }
      }
      if (more) load_tile_ids<BS>(Y, a, L, ids, j, r16, q4);
    });
    if (last) {
      finish(C, m, lsum, o);
      m = -INFINITY;
      lsum = 0.0f;
#pragma unroll
      for (int n = 0; n < 8; ++n) o[n] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
      mask_q<G>(qb, X.k[0], r16);
    }
  };
  for (;;) {
    turn(A, B);
    if (!more) break;
    turn(B, A);
    if (!more) break;
  }
}

// The segment [j0, j1) of a pair as its first group.
template <int BS>
__device__ __forceinline__ void first_group(Group& g) {
  g.g0 = g.j0;
  g.blk = g.g0 * kIt / BS;
  g.g1 = min(g.j1, (g.blk + 64) * BS / kIt);
}

// The next group of the same segment; false when the segment is done.
template <int BS>
__device__ __forceinline__ bool next_in_segment(Group& g) {
  if (g.g1 >= g.j1) return false;
  g.g0 = g.g1;
  g.blk = g.g0 * kIt / BS;
  g.g1 = min(g.j1, (g.blk + 64) * BS / kIt);
  return true;
}

// One partial result (of one segment) in LDS.
template <int G>
struct Part {
  __attribute__((aligned(16))) float o[G][kD];
  float m[G];
  float l[G];
};

template <int G>
__device__ __forceinline__ void put_part(Part<G>& p, float m, float lsum, const f32x4 (&o)[8],
                                         int r16, int q4) {
  lsum += __shfl_xor(lsum, 16);
  lsum += __shfl_xor(lsum, 32);
  if (r16 >= G) return;
  if (q4 == 0) {
    p.m[r16] = m;
    p.l[r16] = lsum;
  }
#pragma unroll
  for (int n = 0; n < 8; ++n) *reinterpret_cast<f32x4*>(&p.o[r16][16 * n + 4 * q4]) = o[n];
}

// Writes channels [4 * d4, 4 * d4 + 4) of output row `row` (sequence and query
// head) from the merged sum L and unnormalised output O.
__device__ __forceinline__ void write_row4(const AttnArgs& a, int64_t row, int d4, float L,
                                           const f32x4& O) {
  const float inv = 1.0f / L;
  f32x4 r;
#pragma unroll
  for (int k = 0; k < 4; ++k) r[k] = L > 0.0f ? div_by(O[k], L, inv) : 0.0f;
  store_out4(a, row * kD + 4 * d4, r);
}

// Writes a whole pair's output from the wave's own partial: the wave reads it
// back with all 64 lanes (in registers only the lanes of the G heads hold
// output, and would divide and store it 32 values a lane).
template <int G>
__device__ __forceinline__ void write_pair(const AttnArgs& a, int b, int kvh, const Part<G>& p,
                                           int lane) {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  const int64_t row = int64_t(b) * a.q_heads + kvh * G;
  // nothing of the stores is to be computed ahead and kept through the tile loop
  asm volatile("" : "+v"(lane));
#pragma unroll 1
  for (int e = lane; e < G * (kD / 4); e += 64) {
    const int g = e / (kD / 4), d4 = e % (kD / 4);
    write_row4(a, row + g, d4, p.l[g], *reinterpret_cast<const f32x4*>(&p.o[g][4 * d4]));
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

// Merges channels [4 * d4, 4 * d4 + 4) of head g over parts first, second,
// second + Step, ... (n <= K in all), read in one LDS round trip (indices past n
// repeat the last part and are given weight 0).
template <int G, int K, int Step>
__device__ __forceinline__ void merge_parts(const Part<G>* p, int first, int second, int n, int g,
                                            int d4, float& M, float& L, f32x4& O) {
  float mm[K], ll[K];
  f32x4 oo[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int i = min(k, n - 1);
    const Part<G>& q = p[i == 0 ? first : second + Step * (i - 1)];
    mm[k] = q.m[g];
    ll[k] = q.l[g];
    oo[k] = *reinterpret_cast<const f32x4*>(&q.o[g][4 * d4]);
  }
  M = -INFINITY;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    if (k >= n) mm[k] = -INFINITY;
    M = fmaxf(M, mm[k]);
  }
  L = 0.0f;
  O = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int k = 0; k < K; ++k) {
    if (mm[k] == -INFINITY) continue;
    const float f = exp2f(mm[k] - M);
    L = fmaf(f, ll[k], L);
#pragma unroll
    for (int c = 0; c < 4; ++c) O[c] = fmaf(f, oo[k][c], O[c]);
  }
}

// Leaves a merged partial in global memory.
template <int G>
__device__ __forceinline__ void write_partial4(const AttnArgs& a, int slot, int g, int d4, float M,
                                               float L, const f32x4& O) {
  const int64_t row = int64_t(slot) * G + g;
  *reinterpret_cast<f32x4*>(&a.part_o[row * kD + 4 * d4]) = O;
  if (d4 == 0) {
    a.part_ml[row * 2] = M;
    a.part_ml[row * 2 + 1] = L;
  }
}

__device__ __forceinline__ void write_zeros(const AttnArgs& a, int b, int threads) {
  for (int e = threadIdx.x; e < a.q_heads * kD; e += threads)
    store_out(a, int64_t(b) * a.q_heads * kD + e, 0.0f);
}

// Inclusive prefix sum over the wave's 64 lanes, by DPP moves: within rows of
// 16 lanes, then the row totals carried over.
__device__ __forceinline__ int wave_inclusive_sum(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, true);    // row_shr 1, 2, 4, 8
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);   // lane 15 of rows 0, 2 to rows 1, 3
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);   // lane 31 to rows 2, 3
  return x;
}

// Short pairs are cut into kShortRuns equal runs of one or two tiles whatever
// else is in the batch, whose partials are merged in one go, in order. The direct
// form and the stream-K form both take them this way, so that a batch's result
// does not depend on which of the two it gets.
struct ShortCut {
  int per, n;         // tiles of a run, runs
  __device__ __forceinline__ explicit ShortCut(int nt)
      : per((nt + kShortRuns - 1) / kShortRuns), n((nt + per - 1) / per) {}
};

// Run `run` of the pair in g (b, kvh, len and nt are set) by one wavefront; its
// partial goes to sink(m, lsum, o).
template <int G, int BS, bool BF16, typename Sink>
__device__ __forceinline__ void attend_run(const AttnArgs& a, Group g, const ShortCut& cut, int run,
                                           int lane, Sink&& sink) {
  static_assert(short_tokens(1) <= 2 * kShortRuns * kIt, "a run is one or two tiles");
  const int r16 = lane & 15, q4 = lane >> 4;
  g.j0 = run * cut.per;
  g.j1 = min(g.nt, g.j0 + cut.per);
  first_group<BS>(g);
  const int32_t got = load_group_ids<BS>(a, g, lane);
  u32x4 qb[4];
  load_q<G>(qb, a, g.b, g.kvh, r16, q4);
  const int32_t ids = check_group_ids<BS>(a, g, lane, got);
  Tile A, B;
  load_tile_ids<BS>(A, a, g, ids, g.j0, r16, q4);
  mask_q<G>(qb, qb, r16);
  float m = -INFINITY, lsum = 0.0f;
  f32x4 o[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) o[i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  const bool two = g.j1 - g.j0 == 2;
  consume_tile<BF16>(A, qb, a.scale_log2, m, lsum, o, [&] {
    if (two) load_tile_ids<BS>(B, a, g, ids, g.j0 + 1, r16, q4);
  });
  if (two) consume_tile<BF16>(B, qb, a.scale_log2, m, lsum, o, [] {});
  sink(m, lsum, o);
}

// A short pair by one workgroup of Waves wavefronts, merged in LDS.
template <int G, int BS, bool BF16, int Waves>
__device__ __forceinline__ void attend_short(const AttnArgs& a, int b, int kvh, int len,
                                             Part<G>* parts) {
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));             // as in write_pair: not kept from pair to pair
  const int lane = tid & 63;
  const int64_t row = int64_t(b) * a.q_heads + kvh * G;
  constexpr int kItems = G * (kD / 4);
  if (len == 0) {
    for (int e = tid; e < kItems; e += Waves * 64)
      store_out4(a, row * kD + 4 * e, out_f32x4{0.0f, 0.0f, 0.0f, 0.0f});
    return;
  }
  Group g;
  g.b = b;
  g.kvh = kvh;
  g.len = len;
  g.nt = (len + kIt - 1) / kIt;
  const ShortCut cut(g.nt);
  for (int run = uniform(tid >> 6); run < cut.n; run += Waves)
    attend_run<G, BS, BF16>(a, g, cut, run, lane, [&](float m, float lsum, const f32x4 (&o)[8]) {
      put_part<G>(parts[run], m, lsum, o, lane & 15, lane >> 4);
    });
  __syncthreads();
  for (int e = tid; e < kItems; e += Waves * 64) {
    const int h = e / (kD / 4), d4 = e % (kD / 4);
    float M, L;
    f32x4 O;
    merge_parts<G, kShortRuns, 1>(parts, 0, 1, cut.n, h, d4, M, L, O);
    write_row4(a, row + h, d4, L, O);
  }
}

// Run `run` of a short pair by one wavefront of the stream-K form: its partial
// goes to slot kShortRuns * pair + run, and the first run's wavefront leaves the
// pair's record (kShortPair, number of runs).
template <int G, int BS, bool BF16>
__device__ __forceinline__ void attend_short_run(const AttnArgs& a, int pair, int run, int b, int kvh,
                                                 int len, Part<G>& part, int lane) {
  constexpr int kItems = G * (kD / 4);
  if (len == 0) {
    if (run == 0) {
      for (int e = lane; e < kItems; e += 64)
        store_out4(a, (int64_t(b) * a.q_heads + kvh * G) * kD + 4 * e,
                   out_f32x4{0.0f, 0.0f, 0.0f, 0.0f});
      if (lane == 0) a.info[2 * pair] = -1;
    }
    return;
  }
  Group g;
  g.b = b;
  g.kvh = kvh;
  g.len = len;
  g.nt = (len + kIt - 1) / kIt;
  const ShortCut cut(g.nt);
  if (run == 0 && lane == 0) {
    a.info[2 * pair] = kShortPair;
    a.info[2 * pair + 1] = cut.n;
  }
  if (run >= cut.n) return;
  attend_run<G, BS, BF16>(a, g, cut, run, lane, [&](float m, float lsum, const f32x4 (&o)[8]) {
    put_part<G>(part, m, lsum, o, lane & 15, lane >> 4);
  });
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  for (int e = lane; e < kItems; e += 64) {
    const int h = e / (kD / 4), d4 = e % (kD / 4);
    write_partial4<G>(a, kShortRuns * pair + run, h, d4, part.m[h], part.l[h],
                      *reinterpret_cast<const f32x4*>(&part.o[h][4 * d4]));
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

// Combine records of the stream-K form: one per workgroup (the pair that begins
// there and goes on past it, its last workgroup), or one per pair (its first and
// last workgroup) where there are no more pairs than workgroups, so that few
// pairs take a combine of few workgroups (3 sequences of 100-900 tokens at 8
// heads to each of 8 KV heads: 12.2 -> 11.4 us a call). First value -1: nothing
// to combine. kShortPair (by pair only): the second is the number of the pair's
// runs, whose partials are in slots kShortRuns * pair on.
__host__ __device__ __forceinline__ bool records_by_pair(const AttnArgs& a, int64_t grid) {
  return int64_t(a.batch) * a.kv_heads <= grid;
}

// Stream-K form. The units of all (sequence, KV head) pairs, in that order --
// each pair's kSegCost cost units (no tiles), then its tiles -- are cut into
// equal contiguous ranges, one per wavefront. A pair that lies within one
// wave's range is written by that wave; a wave leaves a partial in LDS for a
// pair it enters in its middle (its head) and for one it leaves unfinished
// (its tail). One barrier at the end of the workgroup's range, then all four
// waves merge these: a pair that began and ended within the workgroup is
// written, one that crosses a workgroup boundary leaves one partial in global
// memory -- slot 2w for the pair workgroup w entered in its middle, 2w + 1 for
// the one that begins there and goes on -- and a record, written by the
// workgroup it begins in, for the combine. Batches that the direct form would
// take, were their table no wider than they need, are cut as it cuts them.
template <int G, int BS, bool BF16>
// Compiled as if two workgroups shared a CU (at most 256 registers a lane),
// although one per CU is launched: under the looser bound the compiler's
// schedule (which then also used accumulation registers) ran every call
// 11-12 % slower.
__global__ __launch_bounds__(kStreamThreads, 2) void attn_mfma_streamk(AttnArgs a) {
  __shared__ int32_t s_len[streamk_max_batch(G)];
  __shared__ int2 s_total[kStreamWaves];          // units of the wave's sequences, any of them long
  __shared__ int32_t s_start[kStreamWaves][2];   // first sequence of each wave's range, units into it
  __shared__ Part<G> s_part[kStreamWaves][2];    // head, tail
  __shared__ int4 s_open[kStreamWaves];   // head pair (-1: none), whether it ends in this
                                          // wave; tail pair (-1: none), last workgroup it is in
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = uniform(tid >> 6);
  const int r16 = lane & 15;
  const int q4 = lane >> 4;
  const int B = a.batch;
  const int H = a.kv_heads;
  const bool by_pair = records_by_pair(a, gridDim.x);

  // Every workgroup reads all lengths: thread t takes per_t consecutive
  // sequences, loaded four at a time (one round trip up to 1024 sequences).
  const int per_t = (B + kStreamThreads - 1) / kStreamThreads;
  const int b0 = min(B, tid * per_t);
  const int b1 = min(B, b0 + per_t);
  auto units_of = [&](int len) {
    const int nt = (len + kIt - 1) / kIt;
    return nt > 0 ? (nt + kSegCost) * H : 0;
  };
  int total = 0;
  const int at_most = short_tokens(int64_t(B) * H);
  bool longer = at_most == 0;
  for (int c = b0; c < b1; c += 4) {
    int raw[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) raw[i] = a.seq_lens[min(c + i, b1 - 1)];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (c + i >= b1) break;
      const int len = clamp_len(raw[i], a);
      if (blockIdx.x == 0 && len != raw[i] && raw[i] > 0) atomicAdd(a.err_count, 1);
      s_len[c + i] = len;
      longer |= len > at_most;
      total += units_of(len);
    }
  }
  const int incl = wave_inclusive_sum(total);
  const bool any_longer = __ballot(longer) != 0;
  if (lane == 63) s_total[wave] = int2{incl, any_longer};
  if (tid < kStreamWaves) s_start[tid][0] = -1;
  __syncthreads();
  const int n_waves = int(gridDim.x) * kStreamWaves;
  int before = incl - total, U = 0, long_ones = 0;
#pragma unroll
  for (int w = 0; w < kStreamWaves; ++w) {
    const int2 t = s_total[w];
    if (w < wave) before += t.x;
    U += t.x;
    long_ones |= t.y;
  }
  if (uniform(long_ones) == 0) {   // few short pairs, in a table too wide for the direct form
    if (2 * B * H <= int(gridDim.x) && B * H * kShortRuns <= part_slots(G, int(gridDim.x))) {
      // a slot for each run, the runs spread over all workgroups
      for (int id = wave * int(gridDim.x) + int(blockIdx.x); id < B * H * kShortRuns;
           id += n_waves) {
        const int pair = id / kShortRuns, b = pair / H;
        attend_short_run<G, BS, BF16>(a, pair, id % kShortRuns, b, pair - b * H, uniform(s_len[b]),
                                      s_part[wave][0], lane);
      }
      return;
    }
    for (int p = blockIdx.x; p < B * H; p += gridDim.x) {
      const int b = p / H;
      attend_short<G, BS, BF16, kStreamWaves>(a, b, p - b * H, uniform(s_len[b]), &s_part[0][0]);
      __syncthreads();
      if (by_pair && tid == 0) a.info[2 * p] = -1;
    }
    if (!by_pair && tid == 0) a.info[2 * blockIdx.x] = -1;
    return;
  }
  const int per = (U + n_waves - 1) / n_waves;
  const int first_wave = int(blockIdx.x) * kStreamWaves;
  // the thread whose sequences hold a wave's first unit says so
  for (int b = b0, at = before; b < b1; ++b) {
    const int n = units_of(s_len[b]);
#pragma unroll
    for (int w = 0; w < kStreamWaves; ++w) {
      const int u = (first_wave + w) * per;
      if (u >= at && u < at + n) {
        s_start[w][0] = b;
        s_start[w][1] = u - at;
      }
    }
    at += n;
  }
  __syncthreads();

  int head = -1, head_ends = 0, tail = -1, tail_wg = 0;
  const int b_first = uniform(s_start[wave][0]);
  if (b_first >= 0) {
    const int u0 = (first_wave + wave) * per;
    const int u1 = min(U, u0 + per);
    int left = u1 - u0;               // units of the range not yet handed out
    // The segment starting at unit r of the pair in g (cost units first);
    // false when the range ends before a tile.
    auto take = [&](Group& g, int r) {
      const int cost = max(0, kSegCost - r);
      if (left <= cost) return false;
      left -= cost;
      g.j0 = max(0, r - kSegCost);
      g.j1 = min(g.nt, g.j0 + left);
      left -= g.j1 - g.j0;
      first_group<BS>(g);
      return true;
    };
    auto next_pair = [&](Group& g) {
      if (left <= kSegCost) return false;
      if (++g.kvh == H) {
        g.kvh = 0;
        do {
          if (++g.b >= B) return false;
          g.len = uniform(s_len[g.b]);
        } while (g.len == 0);
        g.nt = (g.len + kIt - 1) / kIt;
      }
      return take(g, 0);
    };
    auto next = [&](Group& g) { return next_in_segment<BS>(g) || next_pair(g); };
    Group g;
    g.b = b_first;
    g.len = uniform(s_len[g.b]);
    g.nt = (g.len + kIt - 1) / kIt;
    const int into = uniform(s_start[wave][1]);
    g.kvh = into / (g.nt + kSegCost);
    if (take(g, into - g.kvh * (g.nt + kSegCost)))
      stream_wave<G, BS, BF16>(a, g, next, [&](const Group& c, float m, float lsum,
                                               const f32x4 (&o)[8]) {
        const bool begins = c.j0 == 0, ends = c.j1 == c.nt;
        // the tail's place is free until the range's last segment
        Part<G>& p = s_part[wave][begins ? 1 : 0];
        put_part<G>(p, m, lsum, o, r16, q4);
        if (begins && ends) {
          write_pair<G>(a, c.b, c.kvh, p, lane);
          if (by_pair && lane == 0) a.info[2 * (c.b * H + c.kvh)] = -1;
          return;
        }
        if (begins) {
          tail = c.b * H + c.kvh;
          tail_wg = (u1 + (c.nt - c.j1) - 1) / (per * kStreamWaves);   // the range ends with this segment
        } else {
          head = c.b * H + c.kvh;
          head_ends = ends;
        }
      });
  }
  if (lane == 0) s_open[wave] = int4{head, head_ends, tail, tail_wg};
  __syncthreads();

  // Chains of LDS partials. All waves together merge the pair that began in an
  // earlier workgroup, from wave 0's head on; each wave merges the pair that
  // begins as its tail. A chain goes on through the heads of the following
  // waves until its pair ends.
  const int4 mine = s_open[lane % kStreamWaves];
  const uint32_t ends = uint32_t(__ballot(lane < kStreamWaves && mine.x >= 0 && mine.y != 0));
  const Part<G>* parts = &s_part[0][0];
  constexpr int kItems = G * (kD / 4);
  if (uniform(mine.x) >= 0) {                       // lane 0: wave 0's head
    const int n = ends ? __builtin_ctz(ends) + 1 : kStreamWaves;
    for (int e = tid; e < kItems; e += kStreamThreads) {
      const int g = e / (kD / 4), d4 = e % (kD / 4);
      float M, L;
      f32x4 O;
      merge_parts<G, kStreamWaves, 2>(parts, 0, 2, n, g, d4, M, L, O);
      write_partial4<G>(a, 2 * blockIdx.x, g, d4, M, L, O);
    }
  }
  if (tail >= 0) {
    const uint32_t after = ends >> (wave + 1);
    const int n = 1 + (after ? __builtin_ctz(after) + 1 : kStreamWaves - 1 - wave);
    const int b = tail / H;
    const int64_t row = int64_t(b) * a.q_heads + (tail - b * H) * G;
    for (int e = lane; e < kItems; e += 64) {
      const int g = e / (kD / 4), d4 = e % (kD / 4);
      float M, L;
      f32x4 O;
      merge_parts<G, kStreamWaves, 2>(parts, 2 * wave + 1, 2 * wave + 2, n, g, d4, M, L, O);
      if (after)
        write_row4(a, row + g, d4, L, O);
      else
        write_partial4<G>(a, 2 * blockIdx.x + 1, g, d4, M, L, O);
    }
    if (by_pair && lane == 0) {
      a.info[2 * tail] = after ? -1 : int(blockIdx.x);
      a.info[2 * tail + 1] = tail_wg;
    }
  }
  if (!by_pair && tid < 64) {
    // the last tail of the workgroup goes on past it if no later head ends
    const uint64_t tails = __ballot(lane < kStreamWaves && mine.z >= 0);
    const int w = tails ? 63 - __builtin_clzll(tails) : 0;
    const bool open = tails && (ends >> (w + 1)) == 0;
    if (lane == w) {
      a.info[2 * blockIdx.x] = open ? mine.z : -1;
      a.info[2 * blockIdx.x + 1] = mine.w;
    }
  }
  for (int b = blockIdx.x; b < B; b += gridDim.x)
    if (s_len[b] == 0) {
      write_zeros(a, b, kStreamThreads);
      if (by_pair)
        for (int h = tid; h < H; h += kStreamThreads) a.info[2 * (b * H + h)] = -1;
    }
}

// Direct form, for few pairs that are short by the table's width: one
// workgroup of eight wavefronts per (sequence, KV head), a run of the pair's
// tiles each, merged in LDS. No plan over all lengths and no combine: one
// launch, and what it takes is the chain length - block id - tile - merge.
// Against stream-K, 4 query heads to each of 8 KV heads, block size 16, us a
// call: 8 pairs of up to 256 tokens 9.6 / 6.2, up to 512 9.4 / 8.9, up to 1024
// 10.2 / 10.3; 256 pairs 13.5 / 8.7, 17.9 / 13.7, 21.4 / 19.3; 512 pairs 17.5 /
// 15.3, 24.1 / 24.0, 33.9 / 35.0; 1024 pairs of up to 256 24.1 / 24.7. At 1, 2 and
// 8 heads the same within 5 %, at 16 more for the direct form (256 pairs 17.9 /
// 9.9, 21.8 / 14.8). Block size 64, 32 pairs 9.9 / 7.3, up to 512 tokens 10.6 /
// 11.1, 256 pairs of up to 512 18.8 / 13.7, 512 pairs 18.1 / 14.3 and 24.4 / 25.3.
// Short pairs that come to the stream-K form take a plan and, where their runs
// are spread over the workgroups, the combine, but are cut the same way. Then, 4
// heads, block size 16, stream-K's own ranges / one workgroup to a pair / the runs
// spread: 8 pairs of up to 128 tokens 9.6 / 7.2 / 8.0, 256 9.6 / 9.2 / 8.1, 512 9.4
// / 12.8 / 9.3; 64 pairs 10.6 / 7.9 / 8.7, 10.7 / 10.6 / 9.0, 11.3 / 14.8 / 10.7; 256
// pairs 12.5 / 8.2 / 13.4, 13.5 / 11.4 / 14.5, 17.9 / 16.4 / 19.1; 512 pairs 15.1 /
// 12.5, 17.5 / 18.7 and 24.1 / 28.1 -- hence one or two tiles a run up to 256 pairs
// and one tile up to 512, runs spread up to one pair to two workgroups. At block
// size 64 a batch of up to 64 pairs of 257-512 tokens does best with its runs
// spread (8 pairs 9.2 / - / 8.3, 64 pairs 11.0 / - / 10.9; direct 9.0 and 12.0; all
// of 470 tokens 10.1 / - / 8.4 and 13.3 / - / 11.4, direct 11.0 and 11.8), so it
// does not take the direct form.
template <int G, int BS, bool BF16>
__global__ __launch_bounds__(kDirectThreads, 2) void attn_mfma_direct(AttnArgs a) {
  __shared__ Part<G> s_part[kShortRuns];
  const int kvh = blockIdx.x;
  const int b = blockIdx.y;
  const int raw = a.seq_lens[b];
  const int len = clamp_len(raw, a);
  if (kvh == 0 && threadIdx.x == 0 && len != raw && raw > 0) atomicAdd(a.err_count, 1);
  attend_short<G, BS, BF16, kDirectWaves>(a, b, kvh, len, s_part);
}

// Grid form for batches too large for the LDS work list: grid (chunk of
// kGridChunkTiles tiles, KV head, sequence); partials go to row
// (sequence, query head, chunk) and the split-K combine merges them.
template <int G, int BS, bool BF16>
__global__ __launch_bounds__(kThreads, 2) void attn_mfma_grid(AttnArgs a) {
  __shared__ Smem<G> sm;
  const int split = blockIdx.x;
  const int kvh = blockIdx.y;
  const int b = blockIdx.z;
  const int raw = a.seq_lens[b];
  const int len = clamp_len(raw, a);
  if (split == 0 && kvh == 0 && threadIdx.x == 0 && len != raw && raw > 0)
    atomicAdd(a.err_count, 1);
  if (len == 0) {
    if (split == 0 && kvh == 0) write_zeros(a, b, kThreads);
    return;
  }
  const int nt = (len + kIt - 1) / kIt;
  const int j0 = split * kGridChunkTiles;
  if (j0 >= nt) return;
  const int j1 = min(nt, j0 + kGridChunkTiles);
  attend_segment<G, BS, BF16>(a, b, kvh, len, j0, j1, sm,
                              [&](int g, int d, float M, float L, float O) {
    const int hq = kvh * G + g;
    if (j0 == 0 && j1 == nt) {
      store_out(a, (int64_t(b) * a.q_heads + hq) * kD + d, L > 0.0f ? O / L : 0.0f);
    } else {
      const int64_t row = (int64_t(b) * a.q_heads + hq) * a.n_split + split;
      a.part_o[row * kD + d] = O;
      if (d == 0) {
        a.part_ml[row * 2] = M;
        a.part_ml[row * 2 + 1] = L;
      }
    }
  });
}

// Up to K partials of one pair's head g, channels [4 * d4, 4 * d4 + 4), loaded
// in one memory round trip: the i0-th on, held by workgroups w0 + i0, ... (the
// pair's first partial is in its workgroup's slot 2w + 1, the others in 2w).
template <int G, int K>
struct Partials {
  float m[K], l[K];
  f32x4 o[K];
  __device__ __forceinline__ void load(const AttnArgs& a, int w0, int i0, int w_max, int g, int d4) {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      get(k, a, 2 * int64_t(min(w0 + i0 + k, w_max)) + (i0 + k == 0 ? 1 : 0), g, d4);
    }
  }
  // The first n <= K of a short pair's: slot, slot + 1, ...
  __device__ __forceinline__ void load_short(const AttnArgs& a, int slot, int n, int g, int d4) {
#pragma unroll
    for (int k = 0; k < K; ++k) get(k, a, slot + min(k, n - 1), g, d4);
  }
  __device__ __forceinline__ void get(int k, const AttnArgs& a, int64_t slot, int g, int d4) {
    m[k] = a.part_ml[(slot * G + g) * 2];
    l[k] = a.part_ml[(slot * G + g) * 2 + 1];
    o[k] = *reinterpret_cast<const f32x4*>(&a.part_o[(slot * G + g) * kD + 4 * d4]);
  }
  // Merges the first n of them into the running (M, L, O).
  __device__ __forceinline__ void merge(int n, float& M, float& L, f32x4& O) {
    float Mb = M;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      if (k >= n) m[k] = -INFINITY;
      Mb = fmaxf(Mb, m[k]);
    }
    if (Mb == -INFINITY) return;
    const float f_old = M == -INFINITY ? 0.0f : exp2f(M - Mb);
    L *= f_old;
#pragma unroll
    for (int c = 0; c < 4; ++c) O[c] *= f_old;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      if (m[k] == -INFINITY) continue;
      const float f = exp2f(m[k] - Mb);
      L = fmaf(f, l[k], L);
#pragma unroll
      for (int c = 0; c < 4; ++c) O[c] = fmaf(f, o[k][c], O[c]);
    }
    M = Mb;
  }
};

// Merges the partials of every pair that crosses a stream-K workgroup
// boundary: grid (record, heads by two), one lane per four channels of a head.
// The record, then one wavefront merges up to 4 partials, read in one round
// trip; more are shared out over the workgroup's kCombineWaves wavefronts
// (consecutive ones to each, up to 16 a round trip), whose results one of them
// merges. What bounds it is that chain of round trips, about 2 us each. One
// wavefront for all partials / four / eight, us a call: one sequence of 30000
// tokens over 235 workgroups, 16 heads 43.7 / 19.6 / 17.0, two of 20-60
// thousand, 8 heads 32.3 / 21.1 / 20.6; 512 sequences of 17-1000 tokens, 16
// heads 38.0 / 38.4 / 39.8. Of these the record by pair is 30.2 -> 19.6 and
// 27.7 -> 21.1. Loading the first partials along with the record costs more
// than it saves: most workgroups have no pair to merge, and a call with 16
// pairs of 8 heads took 21.2 us instead of 19.6.
template <int G>
__global__ __launch_bounds__(kCombineWaves * 64) void attn_combine_streamk(AttnArgs a, bool by_pair) {
  __shared__ __attribute__((aligned(16))) f32x4 s_o[kCombineWaves][64];
  __shared__ float s_ml[kCombineWaves][64][2];
  const int rec = a.info[2 * blockIdx.x], last_wg = a.info[2 * blockIdx.x + 1];
  const int w0 = by_pair ? rec : int(blockIdx.x);
  const int pair = by_pair ? int(blockIdx.x) : rec;
  const int wave = uniform(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const bool whole_runs = by_pair && rec == kShortPair;   // of a short pair
  const int n = whole_runs ? 1 : last_wg - w0 + 1;
  if ((rec < 0 && !whole_runs) || (wave > 0 && n <= 4)) return;
  // G = 1: the upper half of the lanes repeats the lower half's work
  const int e = (blockIdx.y * 64 + lane) % (G * (kD / 4));
  const int g = e / (kD / 4), d4 = e % (kD / 4);
  float M = -INFINITY, L = 0.0f;
  f32x4 O = {0.0f, 0.0f, 0.0f, 0.0f};
  const int per = n <= 4 ? n : (n + kCombineWaves - 1) / kCombineWaves;
  const int i1 = min(n, (wave + 1) * per);
  if (whole_runs) {
    Partials<G, kShortRuns> p;
    p.load_short(a, kShortRuns * pair, last_wg, g, d4);
    p.merge(last_wg, M, L, O);
  } else if (per <= 4) {
    Partials<G, 4> p;
    p.load(a, w0, min(wave * per, n - 1), last_wg, g, d4);
    p.merge(i1 - wave * per, M, L, O);
  } else {
    for (int i0 = wave * per; i0 < i1; i0 += 16) {
      Partials<G, 16> p;
      p.load(a, w0, i0, last_wg, g, d4);
      p.merge(i1 - i0, M, L, O);
    }
  }
  if (n > 4) {
    s_ml[wave][lane][0] = M;
    s_ml[wave][lane][1] = L;
    s_o[wave][lane] = O;
    __syncthreads();
    if (wave > 0) return;
    float Mw = M;
#pragma unroll
    for (int w = 1; w < kCombineWaves; ++w) Mw = fmaxf(Mw, s_ml[w][lane][0]);
    L = 0.0f;
    O = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int w = 0; w < kCombineWaves; ++w) {
      const float m = s_ml[w][lane][0];
      if (m == -INFINITY) continue;
      const float f = exp2f(m - Mw);
      L = fmaf(f, s_ml[w][lane][1], L);
#pragma unroll
      for (int c = 0; c < 4; ++c) O[c] = fmaf(f, s_o[w][lane][c], O[c]);
    }
  }
  if (G == 1 && lane >= 32) return;
  const int H = a.kv_heads;
  const int b = pair / H;
  write_row4(a, int64_t(b) * a.q_heads + (pair - b * H) * G + g, d4, L, O);
}

template <int G, int BS, bool BF16>
hipError_t launch_typed(const AttnArgs& a, hipStream_t stream) {
  const int64_t pairs = int64_t(a.batch) * a.kv_heads;
  const int64_t width = int64_t(a.max_blocks) * BS;
  if (a.stream_k && short_tokens(pairs) > 0 && width <= short_tokens(pairs) &&
      (BS < 64 || width <= kShortRuns * kIt || pairs > 64)) {
    hipLaunchKernelGGL((attn_mfma_direct<G, BS, BF16>), dim3(a.kv_heads, a.batch),
                       dim3(kDirectThreads), 0, stream, a);
    return hipGetLastError();
  }
  if (a.stream_k) {
    const int grid = attn_streamk_grid();
    hipLaunchKernelGGL((attn_mfma_streamk<G, BS, BF16>), dim3(grid), dim3(kStreamThreads), 0,
                       stream, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const bool by_pair = records_by_pair(a, grid);
    hipLaunchKernelGGL(attn_combine_streamk<G>,
                       dim3(by_pair ? a.batch * a.kv_heads : grid, (G + 1) / 2),
                       dim3(kCombineWaves * 64), 0, stream, a, by_pair);
    return hipGetLastError();
  }
  hipLaunchKernelGGL((attn_mfma_grid<G, BS, BF16>), dim3(a.n_split, a.kv_heads, a.batch),
                     dim3(kThreads), 0, stream, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || a.n_split <= 1) return e;
  return launch_attn_combine(a, stream);
}

template <int G, int BS>
hipError_t launch_g_bs(const AttnArgs& a, hipStream_t stream) {
  return a.dtype == 1 ? launch_typed<G, BS, true>(a, stream) : launch_typed<G, BS, false>(a, stream);
}

template <int G>
hipError_t launch_g(const AttnArgs& a, hipStream_t stream) {
  switch (a.block_size) {
    case 16: return launch_g_bs<G, 16>(a, stream);
    case 32: return launch_g_bs<G, 32>(a, stream);
    case 64: return launch_g_bs<G, 64>(a, stream);
    case 128: return launch_g_bs<G, 128>(a, stream);
    case 256: return launch_g_bs<G, 256>(a, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

// Stream-K grid: one workgroup per CU. A second resident workgroup per CU
// adds no bandwidth (the two share the CU's memory path, the second running
// about 20 % slower) but doubles the cut pairs and their partials.
int attn_streamk_grid() {
  static const int grid = [] {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        cus <= 0)
      return 256;
    return std::min(cus, kMaxStreamGrid);
  }();
  return grid;
}

// The fixed workspace of the no-allocation entry point. Host code never uses
// this name as an address: it takes the per-device address from
// noalloc_workspace().
__device__ __align__(256) unsigned char scratch[kNoAllocBytes];

hipError_t noalloc_workspace(void** ptr) {
  static std::mutex mu;
  static std::unordered_map<int, void*> addr;   // device -> address of `scratch` there
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  std::lock_guard<std::mutex> lock(mu);
  auto it = addr.find(dev);
  if (it == addr.end()) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (p == nullptr) return hipErrorInvalidSymbol;
    it = addr.emplace(dev, p).first;
  }
  *ptr = it->second;
  return hipSuccess;
}

hipError_t launch_paged_attention_mfma(const AttnArgs& a, hipStream_t stream) {
  if (a.batch == 0) return hipSuccess;
  switch (a.q_heads / a.kv_heads) {
    case 1: return launch_g<1>(a, stream);
    case 2: return launch_g<2>(a, stream);
    case 4: return launch_g<4>(a, stream);
    case 8: return launch_g<8>(a, stream);
    case 16: return launch_g<16>(a, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace ema
