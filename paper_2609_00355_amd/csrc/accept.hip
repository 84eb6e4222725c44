// Greedy acceptance: the target-greedy token of every verified row and the
// walk of Algorithm 1 (App. B) over the packed tree.
//
// argmax_partial  grid (row, vocabulary chunk): each workgroup streams one
//                 chunk of one row with 16-byte loads and reduces it to a
//                 packed (order key, ~index) word, so that the maximum word
//                 is the largest value at the lowest index.  With the root
//                 entropy asked for, the first workgroups compute it.
// accept_walk     one wave per sequence: lane v merges the chunk words of row
//                 v, then the wave walks the tree from the root, finding the
//                 child that carries the current row's argmax token with one
//                 ballot per step.
//
// Rows of any vocabulary take the same vector loads: a row whose length is no
// multiple of 16 bytes only makes them unaligned, which the memory pipeline
// serves (at most one more cache line per wave-wide load); the values past a
// row's last whole vector are loaded one by one, beside the vectors.
// 2 x 33 x 50257 bf16, with entropy: 13.6 us with one load per value, 7.6 us
// with these.  Short chunks are latency and little else, so they take what
// costs least of it: up to 256 values one a thread, bf16 chunks of up to 2048
// one vector a thread with exact keys.  Graph-timed acceptances, with the long
// chunks' eight loads and barrier and with these: 61 x 48 x 250 8.7 and 6.0
// us, 61 x 48 x 1003 9.4 and 6.7, 4 x 64 x 1000 5.4 and 4.6, 200 x 64 x 2001
// 30.9 and 17.7 (one load per value: 6.1, 6.9, 5.3 with vectors, 29.0).
//
// sample_partial  the sampling walk's row draws (temperature T > 0): the same
//                 grid and packed reduction as argmax_partial over
//                 z / T + g instead of z, with Gumbel noise g = -ln(-ln u);
//                 accept_walk then walks the draws.  u comes from
//                 Philox4x32-10 (Salmon et al., SC'11) with key (seed) and
//                 counter (w / 4, node, sequence, round), word w % 4, mapped
//                 to ((x >> 9) + 0.5) 2^-23; both logarithms use one fixed
//                 fp32 recipe (exponent, then 2 atanh(s) with
//                 s = (m - 1) / (m + 1) as an odd series to s^9) with fused
//                 multiply-add disabled, so every draw is reproducible bit for
//                 bit off the GPU.  Tokens that provably cannot win skip the
//                 logarithms (see sample_partial).
//
// Root entropy (optional): the target's next-token entropy at the round root,
// H = -sum_w p(w) log p(w) over row 0 of each sequence (the scalar of the
// paper's entropy law, Sec. 4).  Workgroups of their own, the first of the
// grid, read a chunk of a root row once each and leave, relative to its
// maximum m, S = sum e^(z - m) and T = sum e^(z - m) (z - m); the walk merges
// them to H = log S - T / S.
//
// Order key of a float (fp32 bits, or bf16 bits shifted up 16): the sign-
// magnitude encoding mapped to two's complement, so +0 and -0 both map to 0
// (they tie, and the lowest index wins), and every NaN maps to INT32_MAX (a
// NaN is larger than every number; the first NaN wins).
#include "glance_internal.h"

namespace glance {
namespace {

typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
typedef u32x4 u32x4_any __attribute__((aligned(2)));  // at any bf16 or fp32 element

__device__ __forceinline__ int order_key(unsigned int bits) {
  const int neg = (int)(0x80000000u - bits);  // -(magnitude) for a negative value
  int k = ((int)bits < 0) ? neg : (int)bits;
  // a NaN: magnitude above +inf; positive NaN already exceeds +inf, negative NaN does not
  k = ((bits & 0x7fffffffu) > 0x7f800000u) ? 0x7fffffff : k;
  return k;
}

__device__ __forceinline__ unsigned long long pack(int key, int idx) {
  return ((unsigned long long)((unsigned int)key ^ 0x80000000u) << 32) |
         (unsigned long long)(0xffffffffu - (unsigned int)idx);
}

__device__ __forceinline__ unsigned long long umax64(unsigned long long a, unsigned long long b) {
  return a > b ? a : b;
}

__device__ __forceinline__ unsigned long long wave_max64(unsigned long long v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    const unsigned int lo = __shfl_xor((unsigned int)v, off);
    const unsigned int hi = __shfl_xor((unsigned int)(v >> 32), off);
    v = umax64(v, ((unsigned long long)hi << 32) | lo);
  }
  return v;
}

__device__ __forceinline__ float as_f32(unsigned u) { return __builtin_bit_cast(float, u); }

// IEEE 754-2019 maximum (v_maximum3_f32): a NaN operand gives NaN, and -0 < +0.
__device__ __forceinline__ float fmaximum(float a, float b) { return __builtin_elementwise_maximum(a, b); }
__device__ __forceinline__ float fmaximum3(float a, float b, float c) { return fmaximum(fmaximum(a, b), c); }

// bf16 rows, whole vectors of 8 values.  A 32-bit word w holds two bf16 values:
// the high one read as fp32 is w itself (the low value only adds mantissa
// bits below the bf16 precision, so the order of distinct bf16 values is
// kept), the low one is w << 16.  Per 8 values the thread takes one fp32
// maximum, masks it back to bf16 precision and keeps the first 8-value vector
// that reached its running best, together with that vector itself, so the
// lowest index holding the best value is found at the end without a second
// read.  The maximum propagates NaN, so a chunk holding a NaN (or an infinity,
// which the extra mantissa bits can turn into a NaN) shows up as a NaN running
// maximum; such chunks, and chunks whose best value is +0 or -0 (which must
// tie), are redone by the exact scalar scan.
__device__ __forceinline__ void argmax_bf16_fast(const unsigned short* x, int c0, int c1, int tid,
                                                 int& best_key, int& best_idx) {
  constexpr int kUnroll = 8;
  constexpr unsigned kPad = 0xff7fff7fu;  // two finite -3.39e38 values, never selected
  float bk = -__builtin_inff();
  float run = -__builtin_inff();
  int bpos = -1;
  u32x4 bv = {0u, 0u, 0u, 0u};
  for (int e0 = c0 + 8 * tid; e0 < c1; e0 += 8 * 256 * kUnroll) {
    u32x4 v[kUnroll];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const int e = e0 + u * 8 * 256;
      v[u] = e < c1 ? (u32x4)__builtin_nontemporal_load(reinterpret_cast<const u32x4_any*>(x + e))
                    : u32x4{kPad, kPad, kPad, kPad};
    }
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const int e = e0 + u * 8 * 256;
      const float a = fmaximum3(as_f32(v[u][0]), as_f32(v[u][1]), as_f32(v[u][2]));
      const float b = fmaximum3(as_f32(v[u][3]), as_f32(v[u][0] << 16), as_f32(v[u][1] << 16));
      const float m = fmaximum3(as_f32(v[u][2] << 16), as_f32(v[u][3] << 16), fmaximum(a, b));
      run = fmaximum(run, m);
      const float vm = as_f32(__builtin_bit_cast(unsigned, m) & 0xffff0000u);
      if ((vm > bk || bpos < 0) && e < c1) { bk = vm; bpos = e; bv = v[u]; }
    }
  }
  const bool redo = run != run || bk == 0.f;
  if (__syncthreads_or(redo)) {  // exact path: NaN is the largest value, the first one wins
    for (int e = c0 + tid; e < c1; e += 256) {
      const int k = order_key((unsigned int)x[e] << 16);
      if (k > best_key) { best_key = k; best_idx = e; }
    }
    return;
  }
  if (bpos < 0) return;
  unsigned bits = 0;
#pragma unroll
  for (int w = 3; w >= 0; --w) {  // backwards, so the lowest index overwrites last
    if (as_f32(bv[w] & 0xffff0000u) == bk) { best_idx = bpos + 2 * w + 1; bits = bv[w] >> 16; }
    if (as_f32(bv[w] << 16) == bk) { best_idx = bpos + 2 * w; bits = bv[w] & 0xffffu; }
  }
  best_key = order_key(bits << 16);
}

// (S, T) relative to maximum m, moved to the maximum M >= m:
// e^(z-M) (z-M) = e^(m-M) e^(z-m) ((z-m) + (m-M)).  Values so far below M that
// e^(m-M) is zero leave nothing: masked tokens may hold the type's lowest
// value, with which (m-M) S overflows.
__device__ __forceinline__ void entropy_rebase(float m, float M, float& S, float& T) {
  if (S == 0.f) return;  // no mass yet (m may be -inf)
  const float f = __builtin_amdgcn_exp2f((m - M) * 1.4426950408889634f);
  T = f == 0.f ? 0.f : (T + (m - M) * S) * f;
  S *= f;
}

// Entropy statistics of values [chunk ent_len, +ent_len) of a sequence's row
// 0: kEntropyStep values at a time in registers, their maximum first, then
// both sums, each thread relative to its own running maximum.  Bound by the
// load and 32 exponentials a thread and step, within the time the other
// workgroups stream their chunks.  The whole acceptance at 4 x 64 x 152064
// bf16: 54.8 us when the root rows' own argmax workgroups (8 of 512) read
// their chunks a second time value by value, 17.5 us with these (76 more).
// Rows of up to 2048 values take a step of that size (4 x 64 x 1150: the
// 8192-value step's padding cost 0.4 of 7.5 us).
template <bool BF16, int STEP>
__device__ __forceinline__ void entropy_chunk(const AcceptParams& p, int b, int chunk) {
  constexpr int V = BF16 ? 8 : 4;  // values per 16-byte load
  constexpr int LOADS = STEP / (256 * V);
  __shared__ float red_m[4], red_s[4], red_t[4];
  const int tid = threadIdx.x;
  const char* rowp = static_cast<const char*>(p.logits) + (size_t)b * p.n_nodes * p.vocab * (BF16 ? 2 : 4);
  const int begin = chunk * p.ent_len;
  const int end = min(p.vocab, begin + p.ent_len);
  float m = -__builtin_inff(), S = 0.f, T = 0.f;
  for (int c0 = begin; c0 < end; c0 += STEP) {
    const int c1 = min(end, c0 + STEP);
    u32x4 w[LOADS];
#pragma unroll
    for (int l = 0; l < LOADS; ++l) {
      const int e = c0 + (l * 256 + tid) * V;
      w[l] = BF16 ? u32x4{0xff80ff80u, 0xff80ff80u, 0xff80ff80u, 0xff80ff80u}
                  : u32x4{0xff800000u, 0xff800000u, 0xff800000u, 0xff800000u};  // -inf
      if (e + V <= c1) w[l] = *reinterpret_cast<const u32x4_any*>(rowp + (size_t)e * (BF16 ? 2 : 4));
    }
    const int cv = c0 + (c1 - c0) / V * V + tid;  // a value past the last whole vector
    float rest = -__builtin_inff();
    if (cv < c1)
      rest = BF16 ? as_f32((unsigned)reinterpret_cast<const unsigned short*>(rowp)[cv] << 16)
                  : reinterpret_cast<const float*>(rowp)[cv];
    auto each = [&](auto f) __attribute__((always_inline)) {
#pragma unroll
      for (int l = 0; l < LOADS; ++l)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          if (BF16) {
            f(as_f32(w[l][i] << 16));
            f(as_f32(w[l][i] & 0xffff0000u));
          } else {
            f(as_f32(w[l][i]));
          }
        }
      f(rest);
    };
    float mc = m;
    each([&](float z) __attribute__((always_inline)) { mc = fmaxf(mc, z); });
    entropy_rebase(m, mc, S, T);
    m = mc;
    each([&](float z) __attribute__((always_inline)) {
      // finite, so that x d is zero with x: z - m is -inf for z = -inf (and may
      // be for the lowest value), NaN while every value is -inf
      const float d = fmaxf(z - m, -3.4028234663852886e38f);
      const float x = __builtin_amdgcn_exp2f(d * 1.4426950408889634f);
      S += x;
      T += x * d;
    });
  }
  float M = m;
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) M = fmaxf(M, __shfl_xor(M, off));
  if ((tid & 63) == 0) red_m[tid >> 6] = M;
  __syncthreads();
  M = fmaxf(fmaxf(red_m[0], red_m[1]), fmaxf(red_m[2], red_m[3]));
  entropy_rebase(m, M, S, T);
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    S += __shfl_xor(S, off);
    T += __shfl_xor(T, off);
  }
  if ((tid & 63) == 0) {
    red_s[tid >> 6] = S;
    red_t[tid >> 6] = T;
  }
  __syncthreads();
  if (tid == 0)
    p.ent_part[(size_t)b * p.ent_chunks + chunk] =
        make_float4(M, (red_s[0] + red_s[1]) + (red_s[2] + red_s[3]), (red_t[0] + red_t[1]) + (red_t[2] + red_t[3]), 0.f);
}

// ENT: with the root entropy's workgroups, which come first, so that they end
// with the others.
template <bool BF16, bool ENT>
__global__ __launch_bounds__(256) void argmax_partial(AcceptParams p) {
  __shared__ unsigned long long red[4];
  const int ent_blocks = ENT ? p.batch * p.ent_chunks : 0;
  if (ENT && (int)blockIdx.x < ent_blocks) {
    const int b = blockIdx.x / p.ent_chunks, c = blockIdx.x % p.ent_chunks;
    if (p.vocab <= 2048) entropy_chunk<BF16, 2048>(p, b, c);
    else entropy_chunk<BF16, kEntropyStep>(p, b, c);
    return;
  }
  const int block = blockIdx.x - ent_blocks;
  const int chunk = block % p.chunks;
  const long row = block / p.chunks;
  const int c0 = chunk * p.chunk_len;
  const int c1 = min(p.vocab, c0 + p.chunk_len);
  constexpr int V = BF16 ? 8 : 4;          // values per 16-byte load
  // end of the whole vectors (none in chunks of a value a thread at most)
  const int cv = c1 - c0 <= 256 ? c0 : c0 + (c1 - c0) / V * V;
  const int tid = threadIdx.x;
  int best_key = (int)0x80000000;
  int best_idx = 0x7fffffff;
  unsigned rest = 0u;  // a value past them, one a thread, used after the scan
  if (BF16) {
    const unsigned short* x = static_cast<const unsigned short*>(p.logits) + row * (long)p.vocab;
    if (cv + tid < c1) rest = x[cv + tid];
    if (c1 - c0 <= 256 * V) {
      // a vector a thread at most: eight exact keys instead of the long
      // chunks' eight loads and their barrier
      const int e = c0 + V * tid;
      if (e < cv) {
        const u32x4 v = *reinterpret_cast<const u32x4_any*>(x + e);
#pragma unroll
        for (int w = 0; w < V; ++w) {
          const int k = order_key(w & 1 ? v[w / 2] & 0xffff0000u : v[w / 2] << 16);
          if (k > best_key) { best_key = k; best_idx = e + w; }
        }
      }
    } else {
      argmax_bf16_fast(x, c0, cv, tid, best_key, best_idx);
    }
    rest <<= 16;
  } else {
    const unsigned int* x = static_cast<const unsigned int*>(p.logits) + row * (long)p.vocab;
    if (cv + tid < c1) rest = x[cv + tid];
    constexpr int kUnroll = 4;
    for (int e0 = c0 + 4 * tid; e0 < cv; e0 += 4 * 256 * kUnroll) {
      u32x4 v[kUnroll];
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        const int e = e0 + u * 4 * 256;
        v[u] = e < cv ? (u32x4)*reinterpret_cast<const u32x4_any*>(x + e) : u32x4{0u, 0u, 0u, 0u};
      }
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        const int e = e0 + u * 4 * 256;
        if (e >= cv) break;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const int k = order_key(v[u][w]);
          if (k > best_key) { best_key = k; best_idx = e + w; }
        }
      }
    }
  }
  // threads that saw no element keep the smallest possible word
  unsigned long long w = (best_idx == 0x7fffffff) ? 0ull : pack(best_key, best_idx);
  if (cv + tid < c1) w = umax64(w, pack(order_key(rest), cv + tid));
  w = wave_max64(w);
  if ((tid & 63) == 0) red[tid >> 6] = w;
  __syncthreads();
  if (tid == 0) p.part[row * p.chunks + chunk] = umax64(umax64(red[0], red[1]), umax64(red[2], red[3]));
}

// Philox4x32-10: ten rounds of two 32x32 -> 64-bit multiplies and a
// counter shuffle, the key advanced by the Weyl constants between rounds.
// c[0]'s product of the first round comes in as p0: the caller's counters are
// an arithmetic sequence, so that it is an addition there.
constexpr unsigned kPhiloxM0 = 0xD2511F53u, kPhiloxM1 = 0xCD9E8D57u;
__device__ __forceinline__ void philox4x32_10(unsigned long long p0, unsigned (&c)[4], unsigned k0, unsigned k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r > 0) {
      k0 += 0x9E3779B9u;
      k1 += 0xBB67AE85u;
      p0 = (unsigned long long)kPhiloxM0 * c[0];
    }
    const unsigned long long p1 = (unsigned long long)kPhiloxM1 * c[2];
    // three-input XOR in one v_bitop3_b32 (truth table 0x96)
    const unsigned n0 = __builtin_amdgcn_bitop3_b32((unsigned)(p1 >> 32), c[1], k0, 0x96);
    const unsigned n2 = __builtin_amdgcn_bitop3_b32((unsigned)(p0 >> 32), c[3], k1, 0x96);
    c[0] = n0;
    c[1] = (unsigned)p1;
    c[2] = n2;
    c[3] = (unsigned)p0;
  }
}

// ln t for a positive normal t by the fixed recipe: t = m 2^e with m in
// [sqrt(1/2), sqrt(2)) (so m - 1 is exact and t near 1 keeps e = 0), then
// e ln 2 + 2 atanh(s), s = (m - 1) / (m + 1), atanh(s) / s as the series
// 1 + s^2/3 + ... + s^8/9.  IEEE-rounded operations, no fused multiply-add.
__device__ __forceinline__ float ln_fixed(float t) {
#pragma clang fp contract(off)
  const unsigned bits = __builtin_bit_cast(unsigned, t);
  const unsigned mant = bits & 0x007FFFFFu;
  const bool high = mant > 0x3504F3u;  // m >= sqrt(2): halve it
  const int e = (int)((bits >> 23) & 0xFFu) - 127 + (high ? 1 : 0);
  const float m = __builtin_bit_cast(float, mant | (high ? 0x3F000000u : 0x3F800000u));
  const float s = (m - 1.0f) / (m + 1.0f);
  const float s2 = s * s;
  float acc = (float)(1.0 / 9.0);
  acc = acc * s2 + (float)(1.0 / 7.0);
  acc = acc * s2 + (float)(1.0 / 5.0);
  acc = acc * s2 + (float)(1.0 / 3.0);
  acc = acc * s2 + 1.0f;
  const float at2 = 2.0f * (s * acc);
  return (float)e * (float)0.6931471805599453 + at2;
}

// The perturbed logit z / T + g of one token, g = -ln(-ln u), exactly as the
// definition rounds it.
__device__ __forceinline__ float gumbel_logit(float z, float temperature, unsigned x) {
#pragma clang fp contract(off)
  const float u = ((float)(x >> 9) + 0.5f) * 0x1p-23f;
  const float g = -ln_fixed(-ln_fixed(u));
  return z / temperature + g;
}

// Monotone map between floats and signed integers (its own inverse): larger
// numbers give larger keys; a positive NaN maps above +inf.
__device__ __forceinline__ int float_order(int bits) { return bits ^ ((bits >> 31) & 0x7fffffff); }

// Wave maximum of integer keys, broadcast; every lane must be active.
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp_i(int v) {  // lanes a row mask leaves out read INT_MIN
  return __builtin_amdgcn_update_dpp((int)0x80000000, v, CTRL, ROWS, 0xf, false);
}
__device__ __forceinline__ int wave_max_key(int v) {
  v = max(v, dpp_i<0xb1, 0xf>(v));
  v = max(v, dpp_i<0x4e, 0xf>(v));
  v = max(v, dpp_i<0x141, 0xf>(v));
  v = max(v, dpp_i<0x140, 0xf>(v));
  v = max(v, dpp_i<0x142, 0xa>(v));
  v = max(v, dpp_i<0x143, 0xc>(v));
  return __builtin_amdgcn_readlane(v, 63);
}

// One group of four tokens as raw words (bf16 pairs, or fp32 bits), loaded a
// loop iteration ahead and unpacked when used; any element alignment.
typedef __attribute__((ext_vector_type(2))) unsigned int u32x2;
typedef u32x2 u32x2_any __attribute__((aligned(2)));
template <bool BF16>
__device__ __forceinline__ void load_group(const void* rowp, int e4, unsigned (&w)[4]) {
  if (BF16) {
    const u32x2 v = *reinterpret_cast<const u32x2_any*>(static_cast<const unsigned short*>(rowp) + e4);
    w[0] = v[0];
    w[1] = v[1];
  } else {
    const u32x4 v = *reinterpret_cast<const u32x4_any*>(static_cast<const unsigned*>(rowp) + e4);
#pragma unroll
    for (int j = 0; j < 4; ++j) w[j] = v[j];
  }
}

template <bool BF16>
__device__ __forceinline__ void unpack_group(const unsigned (&w)[4], float (&z)[4]) {
  if (BF16) {
    z[0] = __builtin_bit_cast(float, w[0] << 16);
    z[1] = __builtin_bit_cast(float, w[0] & 0xffff0000u);
    z[2] = __builtin_bit_cast(float, w[1] << 16);
    z[3] = __builtin_bit_cast(float, w[1] & 0xffff0000u);
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) z[j] = __builtin_bit_cast(float, w[j]);
  }
}

// Row draws of the sampling walk.  Evaluating both logarithms for every token
// would cost about a hundred instructions a token, so each group of four is
// first tested against the wave's running best y* (the largest z / T + g found
// so far by any lane of the wave).  Let m be the group's largest z / T and x
// = m - y* plus an allowance for every rounding involved (2^-17 relative,
// 2^-12 absolute).  A token can only win if its noise g >= -x; with
// u = (k + 0.5) 2^-23, r = 2^23 - 1 - k and c the generator word (k = c >> 9),
// g <= -ln(1 - u) and 1 - u > r 2^-23, so it takes r <= R = 2^23 e^x, that is
// ~c <= 512 R + 511.  So one exponential per group gives a threshold T (a
// thousandth and 512 larger, for the roundings), and the group is skipped if
// the largest of its four words is below ~T: then a strictly larger value
// exists and none of its tokens is the draw.  With x < -24 ln 2 no word can
// pass, and the group skips the generator too.  In a group that passes, each
// token is tested with its own z / T and the bound log2 r >= F 2^-23 - 127, F
// the fp32 bits of float(r) (exponent plus mantissa fraction, since
// log2(1 + f) >= f on [0, 1]); survivors take the exact definition.  NaN or
// infinite operands give a T that every word passes, and a NaN bound takes the
// exact path: slower, never wrong.  -inf logits are clamped to -FLT_MAX for
// the group test, so fully masked groups are skipped once y* is finite.
//
// Bound by instruction issue: 107 vector instructions a group on average, 81 %
// of the kernel's cycles at four a wave and instruction (the generator's 17
// 64-bit multiply-adds among them issue like any other).  4 x 64 x 152064
// bf16, T = 1: 33.7 us with a bound per token (11 instructions each), 30.3 us
// with one per group.
struct SampleState {
  int best_key, best_idx;
  float lane_best;  // y of the lane's best token
};

// One group of four tokens of one lane.  FIRST (the wave's first full
// group, no running best yet): the wave first takes the largest lower bound
// on z / T + g over its 256 tokens as y*, from the integer alone: for
// u >= 1/2, -ln u <= (1 - u) / u gives g >= -ln(1 - u) - 2 (1 - u), bounded
// below through the fp32 bits of float(r + 1) (within about 0.05 of the
// noise in its upper tail); g >= -2.82 for u < 1/2; less the same rounding
// allowance.  Every value is at most some token's exact z / T + g, and the
// token reaching it is never skipped, so the exact draw is kept.
template <bool TAIL, bool FIRST>
__device__ __forceinline__ void sample_group(const AcceptParams& p, const float (&z)[4], int e4, int c1,
                                             unsigned long long m0c, unsigned node, unsigned seq, unsigned rnd,
                                             float& wbest, SampleState& st) {
  constexpr float kLn2 = 0.6931472f;
  constexpr float kLog2e = 1.442695041f;
  const float inv_t = p.inv_temperature;
  const float m = __builtin_elementwise_maximum(__builtin_elementwise_maximum(z[0], z[1]),
                                                __builtin_elementwise_maximum(z[2], z[3]));
  const float mt = __builtin_elementwise_maximum(m * inv_t, -3.4028234663852886e38f);
  const float mt_hi = fmaf(fabsf(mt), 0x1p-17f, mt);
  if (!FIRST) {
    const bool beaten = mt_hi + (fmaf(fabsf(wbest), 0x1p-17f, 0x1p-12f) - wbest) < -24.f * kLn2;
    if (beaten || (TAIL && e4 >= c1)) return;
  }
  unsigned c[4] = {(unsigned)e4 >> 2, node, seq, rnd};
  philox4x32_10(m0c, c, p.seed_lo, p.seed_hi);
  if (FIRST) {
    int lo_key = (int)0x80000000;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float zt = z[j] * inv_t;
      const float zt_lo = zt * (zt >= 0.f ? 1.0f - 0x1p-17f : 1.0f + 0x1p-17f);
      // r + 1 = 2^23 - k; log2(r + 1) <= F 2^-23 - 127 + 0.0861 for F the bits of float(r + 1)
      const float r1 = (float)(0x800000u - (c[j] >> 9));
      const float lg1 = (float)__builtin_bit_cast(unsigned, r1) * 0x1p-23f - 127.f;
      const float g_lo = (int)c[j] < 0 ? (22.9138f - lg1) * kLn2 - 2.f * (r1 * 0x1p-23f) : -2.82f;
      lo_key = max(lo_key, float_order(__builtin_bit_cast(int, zt_lo + g_lo - 0x1p-12f)));
    }
    wbest = __builtin_bit_cast(float, float_order(wave_max_key(lo_key)));
  }
  const float slack = fmaf(fabsf(wbest), 0x1p-17f, 0x1p-12f);
  // T = 512 R (1 + 2^-10) + 1024, saturating; a NaN x passes everything (the
  // minimum takes the other operand)
  const float x = mt_hi + (slack - wbest);
  const float t = __builtin_amdgcn_exp2f(fmaf(fminf(x, 0.f), kLog2e, 32.00141f)) + 1024.f;
  unsigned T;
  asm("v_cvt_u32_f32 %0, %1" : "=v"(T) : "v"(t));  // saturates, unlike a cast
  if (max(max(c[0], c[1]), max(c[2], c[3])) < ~T) return;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if (TAIL && e4 + j >= c1) break;
    const float zt = z[j] * inv_t;
    // the noise's upper bound from its own word (r = 0: 150 ln 2)
    const unsigned r = 0x7FFFFFu - (c[j] >> 9);
    const float lg2r = (float)__builtin_bit_cast(unsigned, (float)r) * 0x1p-23f - 127.f;
    const float bound = fmaf(23.f - lg2r, kLn2, fmaf(fabsf(zt), 0x1p-17f, zt) + slack);
    if (!(bound < wbest)) {
      const float y = gumbel_logit(z[j], p.temperature, c[j]);
      const int k = order_key(__builtin_bit_cast(unsigned, y));
      if (k > st.best_key) {
        st.best_key = k;
        st.best_idx = e4 + j;
        st.lane_best = y;
      }
    }
  }
}

template <bool BF16>
__global__ __launch_bounds__(256) void sample_partial(AcceptParams p) {
  __shared__ unsigned long long red[4];
  __shared__ __align__(16) float s_best[4];  // each wave's running best, shared without barriers
  const int chunk = blockIdx.x % p.chunks;
  const long row = blockIdx.x / p.chunks;
  const unsigned node = (unsigned)(row % p.n_nodes), seq = (unsigned)(row / p.n_nodes);
  const int c0 = chunk * p.chunk_len;  // a multiple of 8: groups of four never straddle chunks
  const int c1 = min(p.vocab, c0 + p.chunk_len);
  const int full_end = c0 + (c1 - c0) / 1024 * 1024;  // iterations where every lane has four tokens
  const int tid = threadIdx.x, wave = tid >> 6;
  const char* rowp = static_cast<const char*>(p.logits) + row * (long)p.vocab * (BF16 ? 2 : 4);
  // the round number: the argument, plus the device counter when one is given
  // (the walk kernel, later on the stream, advances it)
  const unsigned rnd = p.round + (p.round_counter ? __hip_atomic_load(p.round_counter, __ATOMIC_RELAXED,
                                                                      __HIP_MEMORY_SCOPE_AGENT)
                                                  : 0u);
  SampleState st = {(int)0x80000000, 0x7fffffff, -__builtin_inff()};
  float wbest = -__builtin_inff();  // a value some token of the workgroup reaches
  if ((tid & 63) == 0) s_best[wave] = -__builtin_inff();
  __syncthreads();
  // A wave publishes its running best to its slot and takes the maximum of
  // the four slots.  Reads may see another wave's older value: every value a
  // slot ever holds is reached by some token, so a stale one only skips less.
  auto share = [&]() __attribute__((always_inline)) {
    const float wm = __builtin_bit_cast(float, float_order(wave_max_key(float_order(__builtin_bit_cast(int, st.lane_best)))));
    wbest = wm > wbest ? wm : wbest;  // a NaN maximum leaves wbest as it is
    if ((tid & 63) == 0) __hip_atomic_store(&s_best[wave], wbest, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    float o = -__builtin_inff();
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float x = __hip_atomic_load(&s_best[w], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      o = x > o ? x : o;
    }
    o = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, o)));
    wbest = o > wbest ? o : wbest;
  };
  unsigned wn[4] = {0u, 0u, 0u, 0u};
  // the generator's first product, M0 times the counter, of the lane's group
  unsigned long long m0c = (unsigned long long)kPhiloxM0 * (unsigned)((c0 >> 2) + tid);
  if (c0 < full_end) {
    load_group<BF16>(rowp, c0 + 4 * tid, wn);
    float z[4];
    unpack_group<BF16>(wn, z);
    if (c0 + 1024 < full_end) load_group<BF16>(rowp, c0 + 1024 + 4 * tid, wn);
    sample_group<false, true>(p, z, c0 + 4 * tid, c1, m0c, node, seq, rnd, wbest, st);
    share();
  }
  // the running best is exchanged every iteration while it still climbs fast,
  // then every fourth (a uniform condition: the exchange needs every lane)
  int it = 0;
  for (int base = c0 + 1024; base < full_end; base += 1024) {  // the same trip count for every lane
    float z[4];
    unpack_group<BF16>(wn, z);
    if (base + 1024 < full_end) load_group<BF16>(rowp, base + 1024 + 4 * tid, wn);
    m0c += (unsigned long long)kPhiloxM0 * 256u;  // 1024 tokens on
    sample_group<false, false>(p, z, base + 4 * tid, c1, m0c, node, seq, rnd, wbest, st);
    ++it;
    if (it <= 4 || (it & 3) == 0) share();
  }
  if (full_end < c1) {  // the ragged tail: per-token bounds checks
    const int e4 = full_end + 4 * tid;
    float z[4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
      z[j] = e4 + j < c1 ? (BF16 ? __builtin_bit_cast(float, (unsigned)reinterpret_cast<const unsigned short*>(rowp)[e4 + j] << 16)
                                 : reinterpret_cast<const float*>(rowp)[e4 + j])
                         : -__builtin_inff();
    sample_group<true, false>(p, z, e4, c1, (unsigned long long)kPhiloxM0 * ((unsigned)e4 >> 2), node, seq, rnd, wbest, st);
  }
  unsigned long long w = (st.best_idx == 0x7fffffff) ? 0ull : pack(st.best_key, st.best_idx);
  w = wave_max64(w);
  if ((tid & 63) == 0) red[tid >> 6] = w;
  __syncthreads();
  if (tid == 0) p.part[row * p.chunks + chunk] = umax64(umax64(red[0], red[1]), umax64(red[2], red[3]));
}

// Lane v holds row v's token, its node's parent and the edge token, so a step
// of the walk is a readlane and a ballot, with no memory access; lane k keeps
// path entry k.
template <bool ENT>
__global__ __launch_bounds__(64) void accept_walk(AcceptParams p) {
  const int b = blockIdx.x;
  const int lane = threadIdx.x;
  const int n = p.n_nodes;
  const long rb = (long)b * n;

  int am = 0;
  int par = -1;
  int tok = 0;
  // the entropy's chunk statistics go out with the other loads (a lane's first)
  const float4* ep = ENT ? p.ent_part + (long)b * p.ent_chunks : nullptr;
  float4 e0 = {-__builtin_inff(), 0.f, 0.f, 0.f};
  if (ENT && lane < p.ent_chunks) e0 = ep[lane];
  if (lane < n) {
    // the tree and the chunk words are all loaded before any is used (one
    // memory round trip; the argmax store below could alias the tree inputs,
    // so the compiler would not hoist their loads over it)
    par = p.parents[rb + lane];
    tok = p.tokens[rb + lane];
    unsigned long long w = 0ull;
    const unsigned long long* src = p.part + (rb + lane) * p.chunks;
    for (int c0 = 0; c0 < p.chunks; c0 += 8) {
      unsigned long long v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = c0 + u < p.chunks ? src[c0 + u] : 0ull;
#pragma unroll
      for (int u = 0; u < 8; ++u) w = umax64(w, v[u]);
    }
    am = (int)(0xffffffffu - (unsigned int)(w & 0xffffffffull));
    p.argmax_out[rb + lane] = am;
  }

  // Walk: from node v, descend to the lowest-index child c > v of v whose token
  // is argmax(row v).  Node indices strictly increase, so at most n - 1 steps.
  int v = 0;
  int len = 0;
  int entry = lane == 0 ? 0 : -1;  // path entry of this lane
  for (int step = 0; step < n; ++step) {
    const int t = __builtin_amdgcn_readlane(am, v);
    const unsigned long long m = __ballot(lane < n && lane > v && par == v && tok == t);
    if (m == 0ull) break;
    v = (int)__builtin_ctzll(m);
    ++len;
    entry = lane == len ? v : entry;
  }
  const int bonus = __builtin_amdgcn_readlane(am, v);  // every lane still active
  int32_t* path = p.accept_path + (long)b * p.path_stride;
  for (int k = lane; k < p.path_stride; k += 64) path[k] = k < 64 ? entry : -1;
  if (lane == 0) {
    p.accept_len[b] = len;
    p.next_root[b] = bonus;
  }
  // sampling with a device round counter: every row draw of this call has
  // read it (the draws kernel ran earlier on the stream), so advance it once
  if (p.round_counter && b == 0 && lane == 0) {
    const unsigned r = __hip_atomic_load(p.round_counter, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(p.round_counter, r + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (ENT) {
    // merge the chunks relative to the row maximum M
    float M = e0.x;
    for (int c = lane + 64; c < p.ent_chunks; c += 64) M = fmaxf(M, ep[c].x);
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) M = fmaxf(M, __shfl_xor(M, off));
    float S = e0.y, T = e0.z;
    entropy_rebase(e0.x, M, S, T);
    for (int c = lane + 64; c < p.ent_chunks; c += 64) {
      float4 q = ep[c];
      entropy_rebase(q.x, M, q.y, q.z);
      S += q.y;
      T += q.z;
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
      S += __shfl_xor(S, off);
      T += __shfl_xor(T, off);
    }
    if (lane == 0) p.root_entropy[b] = __builtin_amdgcn_logf(S) * 0.6931471805599453f - T / S;
  }
}

}  // namespace

hipError_t launch_sample(const AcceptParams& p, bool bf16, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
  const long rows = (long)p.batch * p.n_nodes;
  const dim3 grid((unsigned)(rows * p.chunks)), block(256);
  if (ev0) (void)hipEventRecord(ev0, s);
  if (bf16) hipLaunchKernelGGL(sample_partial<true>, grid, block, 0, s, p);
  else hipLaunchKernelGGL(sample_partial<false>, grid, block, 0, s, p);
  hipError_t e = hipGetLastError();
  if (ev1) (void)hipEventRecord(ev1, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(accept_walk<false>, dim3(p.batch), dim3(64), 0, s, p);
  return hipGetLastError();
}

hipError_t launch_accept(const AcceptParams& p, bool bf16, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
  const long rows = (long)p.batch * p.n_nodes;
  const bool ent = p.root_entropy != nullptr;
  const long ent_blocks = ent ? (long)p.batch * p.ent_chunks : 0;
  auto launch = [&](bool with_ent, long blocks) {
    const dim3 grid((unsigned)blocks), block(256);
    if (bf16 && with_ent) hipLaunchKernelGGL((argmax_partial<true, true>), grid, block, 0, s, p);
    else if (bf16) hipLaunchKernelGGL((argmax_partial<true, false>), grid, block, 0, s, p);
    else if (with_ent) hipLaunchKernelGGL((argmax_partial<false, true>), grid, block, 0, s, p);
    else hipLaunchKernelGGL((argmax_partial<false, false>), grid, block, 0, s, p);
  };
  if (ev0) (void)hipEventRecord(ev0, s);
  if (ent_blocks + rows * p.chunks < (1l << 24)) {
    launch(ent, ent_blocks + rows * p.chunks);
  } else {  // a launch holds fewer than 2^32 threads: the entropy on its own
    if (ent) launch(true, ent_blocks);
    launch(false, rows * p.chunks);
  }
  hipError_t e = hipGetLastError();
  if (ev1) (void)hipEventRecord(ev1, s);
  if (e != hipSuccess) return e;
  if (ent) hipLaunchKernelGGL(accept_walk<true>, dim3(p.batch), dim3(64), 0, s, p);
  else hipLaunchKernelGGL(accept_walk<false>, dim3(p.batch), dim3(64), 0, s, p);
  return hipGetLastError();
}

}  // namespace glance
