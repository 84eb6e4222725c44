// What the attention kernels share: the piece plan of a call's keys, derived
// on the device from ctx_lens, the ancestor words of a packed tree, and the
// fp32 path's log-sum-exp.
#pragma once

#include "glance_internal.h"

namespace glance {
namespace {

// Wave reductions by DPP, all lanes active: butterflies within 16-lane rows,
// then row_bcast:15 / row_bcast:31 fold the rows into lane 63 (a lane that a
// row mask leaves out reads the neutral value).  Every step is one vector
// instruction; shuffles through LDS cost a round trip each, and the plan's
// reductions all precede the kernel's first tile load.
template <int CTRL, int ROWS, int NEUTRAL>
__device__ __forceinline__ int plan_dpp(int v) {
  return __builtin_amdgcn_update_dpp(NEUTRAL, v, CTRL, ROWS, 0xf, false);
}
__device__ __forceinline__ int wave_sum(int v) {
  v += plan_dpp<0xb1, 0xf, 0>(v);   // quad_perm [1,0,3,2]
  v += plan_dpp<0x4e, 0xf, 0>(v);   // quad_perm [2,3,0,1]
  v += plan_dpp<0x141, 0xf, 0>(v);  // row_half_mirror
  v += plan_dpp<0x140, 0xf, 0>(v);  // row_mirror
  v += plan_dpp<0x142, 0xa, 0>(v);  // row_bcast:15
  v += plan_dpp<0x143, 0xc, 0>(v);  // row_bcast:31
  return __builtin_amdgcn_readlane(v, 63);
}
__device__ __forceinline__ int wave_max(int v) {  // v >= 0
  v = max(v, plan_dpp<0xb1, 0xf, 0>(v));
  v = max(v, plan_dpp<0x4e, 0xf, 0>(v));
  v = max(v, plan_dpp<0x141, 0xf, 0>(v));
  v = max(v, plan_dpp<0x140, 0xf, 0>(v));
  v = max(v, plan_dpp<0x142, 0xa, 0>(v));
  v = max(v, plan_dpp<0x143, 0xc, 0>(v));
  return __builtin_amdgcn_readlane(v, 63);
}
// Inclusive prefix sum over the wave: row shifts within the rows, then the
// broadcasts into the rows after them.
__device__ __forceinline__ int wave_incl_sum(int v) {
  v += plan_dpp<0x111, 0xf, 0>(v);  // row_shr:1
  v += plan_dpp<0x112, 0xf, 0>(v);  // row_shr:2
  v += plan_dpp<0x114, 0xf, 0>(v);  // row_shr:4
  v += plan_dpp<0x118, 0xf, 0>(v);  // row_shr:8
  v += plan_dpp<0x142, 0xa, 0>(v);  // row_bcast:15
  v += plan_dpp<0x143, 0xc, 0>(v);  // row_bcast:31
  return v;
}

__device__ __forceinline__ int clamp_ctx(int ctx, int cap) { return ctx < 0 ? 0 : (ctx > cap ? cap : ctx); }
// tiles of a sequence: its context tiles, then the tile of new keys
__device__ __forceinline__ int seq_tiles(int ctx) { return (ctx + 63) / 64 + 1; }

struct Piece {
  int b;        // sequence
  int first;    // piece slot of the sequence's first piece (within the KV head)
  int count;    // pieces of the sequence
  int index;    // this piece's index among them
  int t_begin;  // first tile (of the sequence's tile list)
  int n_tiles;  // tiles of the piece, >= 1
  int ctx;      // context keys of the sequence
};

// ln(2^M sum) of the fp32 path.  The reference M need not be the row maximum,
// so log2(sum) may be as large as the result and its rounding as coarse: the
// logarithm is taken of the sum's fraction and every larger term enters by a
// fused multiply-add, which leaves little more than the result's own rounding.
__device__ __forceinline__ float log_sum(float M, float sum) {
  constexpr float ln2 = 0.6931471805599453f;
  const float frac = log2f(__builtin_amdgcn_frexp_mantf(sum)) * ln2;
  return fmaf((float)__builtin_amdgcn_frexp_expf(sum), ln2, fmaf(M, ln2, frac));
}

// The smallest piece, in tiles, for a longest sequence of `longest` tiles: the
// merge pass takes up to 24 pieces in one chunk of loads, and a further chunk
// costs it more than another tile costs the attention, up to pieces of seven
// tiles (four where more than four row tiles make a tile dearer).  Calls with
// few KV heads, whose pieces are the smallest, with a least piece of 3 tiles,
// 4, and by this rule: 336 tiles x 2, 4 rows of 4/1 heads of 64: 21.4, 19.5,
// 16.7 us; 124 x 1, 16 rows of 6/3 heads of 64: 14.4, 13.5, 12.9; 173 x 3, 44
// rows of 8/1 heads of 128: 25.1, 25.1, 25.1 (26.2 with pieces of seven).
__host__ __device__ __forceinline__ int least_piece(const AttnParams& p, int longest) {
  const int most = p.tiles_rg > 4 ? 4 : 7;
  const int t = (longest + 23) / 24;
  const int least = t < most ? t : most;
  return least > p.min_tiles ? least : p.min_tiles;
}

// The piece plan (identical in every wave of every workgroup): T is the
// smallest piece size, at least least_piece(), with sum_b ceil(len_b / T) <=
// slots; piece slot ps then names piece ps - first_b of the sequence b with
// first_b <= ps < first_b + n_b.  Returns false if the slot is unused.  The
// lengths are read once (sequences lane + 64 k, k < kPlanCache, held in
// registers; larger batches re-read the rest), since every memory round trip
// here delays the first tile load.  ONE: at most 64 sequences, one per lane.
//
// Bound by latency, and all of it precedes the kernel's first tile load: with
// shuffles through LDS and a chunk loop for every batch, a draft of one
// sequence of 2048 keys took 15.1 us, with DPP reductions and the one-chunk
// form 14.3 us.
constexpr int kPlanCache = 4;
template <bool ONE>
__device__ __forceinline__ bool find_piece_in(const AttnParams& p, int ps, int lane, Piece& out) {
  constexpr int CACHE = ONE ? 1 : kPlanCache;
  int ctx_c[CACHE];
#pragma unroll
  for (int k = 0; k < CACHE; ++k) {
    const int b = lane + 64 * k;
    ctx_c[k] = b < p.batch ? clamp_ctx(p.ctx_lens[b], p.cap) : -1;
  }
  auto ctx_of = [&](int k) __attribute__((always_inline)) {  // -1 past the batch
    if (ONE || k < CACHE) return ctx_c[ONE ? 0 : k];
    return lane + 64 * k < p.batch ? clamp_ctx(p.ctx_lens[lane + 64 * k], p.cap) : -1;
  };
  auto len_of = [&](int k) __attribute__((always_inline)) {
    const int ctx = ctx_of(k);
    return ctx < 0 ? 0 : seq_tiles(ctx);
  };
  const int chunks = ONE ? 1 : (p.batch + 63) / 64;
  int total = 0, longest = 0;
  for (int k = 0; k < chunks; ++k) {
    const int len = len_of(k);
    total += len;
    longest = max(longest, len);
  }
  total = wave_sum(total);
  longest = wave_max(longest);
  const int slots = p.slots_per_g;
  auto count = [&](int T) __attribute__((always_inline)) {
    int cnt = 0;
    for (int k = 0; k < chunks; ++k) cnt += (len_of(k) + T - 1) / T;
    return wave_sum(cnt);
  };
  int lo = max(least_piece(p, longest), (total + slots - 1) / slots);
  if (count(lo) > slots) {  // not for equal lengths
    // With T = longest every sequence is one piece (slots >= batch), and with
    // T >= total / (slots - batch) the sum stays below total / T + batch.
    int hi = max(lo, longest);
    if (slots > p.batch) hi = max(lo, min(hi, (total + slots - p.batch - 1) / (slots - p.batch)));
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (count(mid) <= slots) hi = mid;
      else lo = mid + 1;
    }
  }
  const int T = lo;
  int base = 0;
  for (int k = 0; k < chunks; ++k) {
    const int ctx = ctx_of(k);
    const int len = len_of(k);
    const int nb = (len + T - 1) / T;
    const int incl = wave_incl_sum(nb) + base;
    const int excl = incl - nb;
    const unsigned long long hit = __ballot(excl <= ps && ps < incl);
    if (hit) {
      const int src = (int)__builtin_ctzll(hit);
      out.b = 64 * k + src;
      out.first = __builtin_amdgcn_readlane(excl, src);
      out.count = __builtin_amdgcn_readlane(nb, src);
      out.ctx = __builtin_amdgcn_readlane(ctx, src);
      const int slen = __builtin_amdgcn_readlane(len, src);
      out.index = ps - out.first;
      out.t_begin = out.index * slen / out.count;
      out.n_tiles = (out.index + 1) * slen / out.count - out.t_begin;
      return true;
    }
    base = __builtin_amdgcn_readlane(incl, 63);
  }
  return false;
}
__device__ __forceinline__ bool find_piece(const AttnParams& p, int ps, int lane, Piece& out) {
  return p.batch <= 64 ? find_piece_in<true>(p, ps, lane, out) : find_piece_in<false>(p, ps, lane, out);
}

// Ancestor words of a packed tree, anc[i] = {i} u anc[parent(i)], lane i's in
// lane i (par: the lane's parent, -1 for none), by pointer doubling: after r
// rounds lane i holds its root path from i up to (excluding) its 2^r-th
// ancestor.  A parent outside [0, i) ends the chain.
__device__ __forceinline__ unsigned long long ancestor_word(int par, int lane) {
  int up = (par >= 0 && par < lane) ? par : -1;
  unsigned long long anc = 1ull << lane;
#pragma unroll
  for (int r = 0; r < 6; ++r) {
    const int src = up < 0 ? lane : up;
    const unsigned lo = __shfl((unsigned)anc, src);
    const unsigned hi = __shfl((unsigned)(anc >> 32), src);
    const int up2 = __shfl(up, src);
    if (up >= 0) {
      anc |= ((unsigned long long)hi << 32) | lo;
      up = up2;
    }
  }
  return anc;
}

}  // namespace
}  // namespace glance
