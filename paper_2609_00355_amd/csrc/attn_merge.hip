// Second pass of split-KV attention: combine the per-split partial results.
//
// Each split s of a row left (m_s, l_s, O_s) with m_s a reference near the
// split's largest scaled score in log2 units, l_s = sum exp2(score - m_s) and
// O_s = sum exp2(score - m_s) v, or all three scaled alike (see
// attn_merge_pieces).  With M = max_s m_s and L = sum_s 2^(m_s - M) l_s:
//   out = sum_s 2^(m_s - M) O_s / L,   lse = (M + log2 L) ln 2
//
// attn_merge_kernel (fp32 attention): D/4 lanes serve one output row, four
// dims (16 bytes) each, so a wave merges 64/(D/4) rows.  The row index is the
// output's own (b, new row, query head) index, so writes are contiguous.  The
// (m, l) pairs and the O partials of up to kChunk splits are loaded together,
// before any of them is needed, so a row with at most kChunk splits costs one
// memory round trip; longer rows take further chunks, rescaled online like
// the attention itself.
//
// attn_merge_pieces (bf16 attention): the partials are the pieces' MFMA
// register tiles in fp16, O_s / l_s scaled by a power of two that the row's
// (max, sum) pair carries (lane l of a 32-row tile holds row l % 32 and, in
// quad k, dims 32 (k / 4) + 8 (k % 4) + 4 (l / 32) .. +3).  A thread owns one
// (row, four dims) and reads that quad of every piece of its sequence, in
// piece order, a chunk of pieces at a time; consecutive threads read
// consecutive lanes, 512 bytes per wave-wide load.  Sequences with one piece
// were written by the attention kernel and are skipped.  Bound by latency.
// The plan's read is one memory round trip; the only sequence of a batch of
// one starts at slot 0, so its first chunk's loads go out beside it, before
// the piece count is known.  A chunk costs more than one round trip: its loads
// depend on the piece count and so become a branch a piece, between the first
// of which the compiler puts a wait for the loads before (seen in the
// assembly after the first two pieces; 16 and 24 pieces also spill 23 and 79
// scalar registers).
#include "attn_plan.h"

namespace glance {
namespace {

constexpr float kLn2 = 0.6931471805599453f;
constexpr int kMergeWaves = 2;
typedef __attribute__((ext_vector_type(4))) _Float16 f16x4;

template <int D>
__global__ __launch_bounds__(64 * kMergeWaves) void attn_merge_kernel(AttnParams p) {
  constexpr int LPR = D / 4;     // lanes per row
  constexpr int RPW = 64 / LPR;  // rows per wave
  constexpr int kChunk = 16;     // splits in flight per lane
  static_assert(kChunk <= LPR, "one (m, l) pair per lane and chunk");
  const int lane = threadIdx.x & 63;
  const int q = lane % LPR;
  const int lead = lane - q;  // first lane of this row
  // row counts are far below 2^31 (batch * new rows * query heads), so 32-bit index math
  const int total = p.batch * p.n * p.hq;
  const int row_raw = ((int)blockIdx.x * kMergeWaves + (int)(threadIdx.x >> 6)) * RPW + lane / LPR;
  const bool live = row_raw < total;
  const int row = live ? row_raw : total - 1;  // dead lanes shadow the last row, store nothing
  const int h = (unsigned)row % (unsigned)p.hq;
  const int bi = (unsigned)row / (unsigned)p.hq;
  const int i = (unsigned)bi % (unsigned)p.n;
  const int b = (unsigned)bi / (unsigned)p.n;
  const int g = h / p.group;
  const int r = i * p.group + (h - g * p.group);

  int ctx = p.ctx_lens[b];
  ctx = ctx < 0 ? 0 : (ctx > p.cap ? p.cap : ctx);
  const int nsb = ctx > 0 ? (ctx + p.split_keys - 1) / p.split_keys : 1;

  const size_t base = ((size_t)b * p.hkv + g) * p.nsplit * p.rows_pad + r;
  const float4* po = reinterpret_cast<const float4*>(p.part_o) + base * (D / 4) + q;
  const size_t sstride = (size_t)p.rows_pad * (D / 4);  // float4s from one split to the next

  float M = -__builtin_inff();
  float lsum = 0.f;  // this lane's share of the denominator
  float4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int s0 = 0; s0 < nsb; s0 += kChunk) {
    const int cnt = min(kChunk, nsb - s0);
    float2 ml = {-__builtin_inff(), 0.f};
    if (q < cnt) ml = p.part_ml[base + (size_t)(s0 + q) * p.rows_pad];
    float4 v[kChunk];
#pragma unroll
    for (int u = 0; u < kChunk; ++u)
      v[u] = u < cnt ? po[(size_t)(s0 + u) * sstride] : float4{0.f, 0.f, 0.f, 0.f};
    float mc = ml.x;
#pragma unroll
    for (int off = LPR / 2; off >= 1; off >>= 1) mc = fmaxf(mc, __shfl_xor(mc, off));
    const float Mn = fmaxf(M, mc);
    const float sc = M == -__builtin_inff() ? 0.f : exp2f(M - Mn);
    const float w = q < cnt ? exp2f(ml.x - Mn) : 0.f;
    lsum = fmaf(w, ml.y, lsum * sc);
    acc.x *= sc; acc.y *= sc; acc.z *= sc; acc.w *= sc;
#pragma unroll
    for (int u = 0; u < kChunk; ++u) {
      const float wu = __shfl(w, lead + u);  // 0 past the last split
      acc.x = fmaf(wu, v[u].x, acc.x);
      acc.y = fmaf(wu, v[u].y, acc.y);
      acc.z = fmaf(wu, v[u].z, acc.z);
      acc.w = fmaf(wu, v[u].w, acc.w);
    }
    M = Mn;
  }
#pragma unroll
  for (int off = LPR / 2; off >= 1; off >>= 1) lsum += __shfl_xor(lsum, off);
  if (!live || nsb == 1) return;  // one split: written by the attention kernel
  const float inv = 1.f / lsum;
  *reinterpret_cast<float4*>(static_cast<float*>(p.out) + (size_t)row * D + 4 * q) =
      float4{acc.x * inv, acc.y * inv, acc.z * inv, acc.w * inv};
  if (p.lse && q == 0) p.lse[row] = log_sum(M, lsum);
}

template <int D, int kChunk>
__global__ __launch_bounds__(256) void attn_merge_pieces(AttnParams p) {
  constexpr int KQ = D / 8;    // quads of values per lane of a tile (OV / 4)
  constexpr int WG_K = 4;      // quad slots per workgroup (one per wave)
  const int lane = threadIdx.x & 63;
  const int k = (blockIdx.x % (KQ / WG_K)) * WG_K + (threadIdx.x >> 6);
  int unit = blockIdx.x / (KQ / WG_K);  // ((b * hkv + g) * row_groups + rgi) * tiles_rg + w
  const int w = unit % p.tiles_rg;
  unit /= p.tiles_rg;
  const int rgi = unit % p.row_groups;
  unit /= p.row_groups;
  const int g = unit % p.hkv;
  const int b = unit / p.hkv;
  const int2 pl = p.plan[b];  // (pieces, first slot)
  const int r32 = lane & 31, h = lane >> 5;
  const int row = 32 * (rgi * p.tiles_rg + w) + r32;
  const bool live = row < p.rows;
  const size_t o_stride = (size_t)p.row_groups * p.tiles_rg * KQ * 64;  // fp16 quads between pieces
  const size_t ml_stride = (size_t)p.row_groups * p.rows_rg;

  float M = -__builtin_inff(), lsum = 0.f;
  float4 acc = {0.f, 0.f, 0.f, 0.f};
  float2 ml[kChunk];
  f16x4 v[kChunk];
  // the (max, sum) pairs and output quads of up to `cnt` pieces from slot
  // `slot` on
  auto load = [&](int slot, int cnt) __attribute__((always_inline)) {
    const size_t ws = ((size_t)g * p.slots_per_g + slot) * p.row_groups + rgi;  // piece u: ws + u * row_groups
    const f16x4* po = reinterpret_cast<const f16x4*>(p.part_o) + (ws * p.tiles_rg + w) * KQ * 64 + k * 64 + lane;
    const float2* pm = p.part_ml + ws * p.rows_rg + 32 * w + r32;
#pragma unroll
    for (int u = 0; u < kChunk; ++u) {
      ml[u] = u < cnt ? pm[(size_t)u * ml_stride] : make_float2(-__builtin_inff(), 0.f);
      v[u] = u < cnt ? po[(size_t)u * o_stride] : f16x4{};
    }
  };
  auto combine = [&](int cnt) __attribute__((always_inline)) {
    float mc = M;
#pragma unroll
    for (int u = 0; u < kChunk; ++u) mc = fmaxf(mc, u < cnt ? ml[u].x : -__builtin_inff());
    const float sc = M == -__builtin_inff() ? 0.f : exp2f(M - mc);
    lsum *= sc;
    acc.x *= sc; acc.y *= sc; acc.z *= sc; acc.w *= sc;
#pragma unroll
    for (int u = 0; u < kChunk; ++u) {
      const bool in = u < cnt;  // a slot past the pieces may hold anything
      const float wu = in ? exp2f(ml[u].x - mc) : 0.f;
      const f16x4 x = in ? v[u] : f16x4{};
      lsum = fmaf(wu, in ? ml[u].y : 0.f, lsum);
      acc.x = fmaf(wu, (float)x[0], acc.x);
      acc.y = fmaf(wu, (float)x[1], acc.y);
      acc.z = fmaf(wu, (float)x[2], acc.z);
      acc.w = fmaf(wu, (float)x[3], acc.w);
    }
    M = mc;
  };
  if (p.batch == 1) load(0, min(kChunk, p.slots_per_g));
  const int count = __builtin_amdgcn_readfirstlane(pl.x), first = __builtin_amdgcn_readfirstlane(pl.y);
  if (count <= 1) return;
  if (p.batch != 1) load(first, min(kChunk, count));
  combine(min(kChunk, count));
  for (int q0 = kChunk; q0 < count; q0 += kChunk) {
    const int cnt = min(kChunk, count - q0);
    load(first + q0, cnt);
    combine(cnt);
  }
  if (!live) return;
  const int node = row / p.group;
  const size_t out_row = ((size_t)b * p.n + node) * p.hq + (size_t)g * p.group + (row - node * p.group);
  const int d0 = 32 * (k >> 2) + 8 * (k & 3) + 4 * h;
  const float inv = 1.f / lsum;
  typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
  const bf16x4 o = {(__bf16)(acc.x * inv), (__bf16)(acc.y * inv), (__bf16)(acc.z * inv), (__bf16)(acc.w * inv)};
  *reinterpret_cast<bf16x4*>(static_cast<__bf16*>(p.out) + out_row * D + d0) = o;
  if (p.lse && k == 0 && h == 0) p.lse[out_row] = (M + log2f(lsum)) * kLn2;
}

}  // namespace

// Pieces in a chunk of loads: enough for every piece of a sequence
// where the plan gives at most 24 to sequences that fill the capacity, and no
// more, since a thread's registers bound the loads in flight on the chip.
// Calls of the attention at 28/4 heads: 64 rows over 4096 keys of 128 dims, 22
// pieces: 20.0 us with 16, 18.8 with 24, 20.0 with 32; 37 rows of 64 dims,
// about 10 pieces: 24.8 with 16, 25.3 with 24 and 32.
static int merge_chunk(const AttnParams& p) {
  const long tiles = ((long)p.cap + 63) / 64 + 1;
  long t = (tiles * p.batch + p.slots_per_g - 1) / p.slots_per_g;
  const long least = least_piece(p, (int)tiles);
  if (t < least) t = least;
  const long pieces = (tiles + t - 1) / t;
  return pieces <= 8 ? 8 : pieces <= 16 || pieces > 24 ? 16 : 24;
}

template <int D>
static void launch_pieces(const AttnParams& p, dim3 grid, dim3 block, hipStream_t s) {
  switch (merge_chunk(p)) {
    case 8: hipLaunchKernelGGL((attn_merge_pieces<D, 8>), grid, block, 0, s, p); break;
    case 24: hipLaunchKernelGGL((attn_merge_pieces<D, 24>), grid, block, 0, s, p); break;
    default: hipLaunchKernelGGL((attn_merge_pieces<D, 16>), grid, block, 0, s, p); break;
  }
}

hipError_t launch_attn_merge_pieces(const AttnParams& p, hipStream_t s) {
  const long units = (long)p.batch * p.hkv * p.row_groups * p.tiles_rg;
  const dim3 grid((unsigned)(units * (p.d / 8) / 4)), block(256);
  if (p.d == 128) launch_pieces<128>(p, grid, block, s);
  else launch_pieces<64>(p, grid, block, s);
  return hipGetLastError();
}

hipError_t launch_attn_merge(const AttnParams& p, hipStream_t s) {
  const long total = (long)p.batch * p.n * p.hq;
  const long rows_per_wg = (long)kMergeWaves * 64 / (p.d / 4);
  const dim3 grid((unsigned)((total + rows_per_wg - 1) / rows_per_wg)), block(64 * kMergeWaves);
  if (p.d == 128) hipLaunchKernelGGL(attn_merge_kernel<128>, grid, block, 0, s, p);
  else hipLaunchKernelGGL(attn_merge_kernel<64>, grid, block, 0, s, p);
  return hipGetLastError();
}

}  // namespace glance
