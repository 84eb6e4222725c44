// Split-KV attention for the block draft and the ancestor-masked tree verify,
// fp32 in / fp32 out, on the fp32 matrix instructions (fp32 products and
// sums): the path in which exactness is decided (the paper audits losslessness
// in fp32, Sec. 3.3 and App. C).
//
// One workgroup of W waves owns (sequence b, KV head g, context split s, row
// tile of 16 R rows).  The split's keys are cut into blocks of 16, dealt to
// the waves in turn; every wave keeps its own online softmax over its blocks
// and the workgroup merges the W results through LDS at its end.  A wave's
// block is
//   S^T[key][row] = K[key][:] . Q[row][:]       (v_mfma_f32_16x16x4_f32, A = K, B = Q^T)
//   P = exp2(S c - m c)                          (online softmax, lazily rescaled)
//   O^T[dim][row] += V^T[dim][key] . P^T[key][row]   (A = V^T, B = P^T)
// Lane l holds row l % 16 of each 16-row part, keys 4 (l / 16) + i of S^T, so
// S^T's result registers are P^T's operands as they are, and K, V and Q come
// straight from global memory in operand order: 16 bytes a lane, the k and dim
// indices of a lane chosen so that its four consecutive floats feed four
// instructions.  No K/V staging in LDS: the matrix instructions take 256 cycles
// per kilobyte of K or V, far longer than its loads.  The next block's K is
// loaded while P.V runs, its V while Q.K^T runs.
//
// Bound by the fp32 matrix rate (about 150 TFLOP/s) where the chip is full: 28
// us of the 48 at 64 rows, 28/4 heads of 128 and 4096 keys (3.8 GFLOP); the
// rest is the start-up, the splits' ends and the merge.  Before, with scalar
// multiply-adds from LDS tiles: 251 us.  The same with two waves a SIMD
// instead of one (twice the splits, or eight waves a workgroup on 64 rows)
// takes 55 us, 42 with its loads taken out: they come in too slowly there;
// 64 rows a wave (one wave a SIMD, accumulators in AGPRs) takes 53 us.  The
// round of 4/1 heads of 64 over 256 keys (8 and 16 rows, a kernel each for
// draft, verify, argmax, walk and commit): 50 -> 27 us.
//
// Partial results (more than one split): O unnormalised, [row][dim], and
// (max * scale * log2 e, sum) per row, combined by attn_merge_kernel; a
// sequence with one split is written by its workgroup.
#include "attn_plan.h"

namespace glance {
namespace {

constexpr float kNegInf = -__builtin_inff();
constexpr float kSumLimit = 256.f;  // per-lane probability sum that forces a rescale

typedef __attribute__((ext_vector_type(4))) float f32x4;

template <int D, bool TREE, int R, int W>
__global__ __launch_bounds__(64 * W, 2) void attn_f32(AttnParams p) {
  constexpr int KC = D / 16;  // 16-byte chunks of K (and Q) per lane and key
  constexpr int DB = D / 16;  // output blocks; result row m of block 4 v + x is dim 64 v + 4 m + x
  constexpr int VC = DB / 4;  // 16-byte chunks of V per lane and key
  __shared__ f32x4 sO[W][R * 4 * VC][64];
  __shared__ float2 sML[W][16 * R];
  __shared__ unsigned long long sAnc[64];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int q = lane >> 4, m16 = lane & 15;

  // The work items (split-major, row tiles of one split side by side) are cut
  // into eight equal runs, one per XCD (block index mod 8): a split's row
  // tiles read its K/V through one L2, two at a run's ends, and no XCD gets
  // more than its eighth (whole splits per XCD would put 70 workgroups on an
  // XCD with room for 64 at 36 splits of 14 tiles: 68 us instead of 55).
  const int total = p.nsplit * p.batch * p.hkv * p.row_groups;
  const int item = (blockIdx.x & 7) * ((total + 7) / 8) + (blockIdx.x >> 3);
  if (item >= min(total, ((int)(blockIdx.x & 7) + 1) * ((total + 7) / 8))) return;
  const int rg = item % p.row_groups;
  const int grp = item / p.row_groups;
  const int g = grp % p.hkv;
  const int bs = grp / p.hkv;
  const int b = bs % p.batch;
  const int s = bs / p.batch;

  const int ctx = clamp_ctx(p.ctx_lens[b], p.cap);
  const int nsb = ctx > 0 ? (ctx + p.split_keys - 1) / p.split_keys : 1;
  if (s >= nsb) return;
  const int k_begin = s * p.split_keys;
  const int k_end = min(ctx, k_begin + p.split_keys);
  const bool has_new = s == nsb - 1;
  const int nb_ctx = k_end > k_begin ? (k_end - k_begin + 15) / 16 : 0;
  const int nb = nb_ctx + (has_new ? (p.n + 15) / 16 : 0);

  // this lane's query rows, dims 16 c + 4 q .. +3 (zeros for padding rows)
  f32x4 qf[R][KC];
  int node[R];
  size_t out_row[R];
  bool row_ok[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int row = (rg * R + r) * 16 + m16;
    row_ok[r] = row < p.rows;
    node[r] = row_ok[r] ? row / p.group : p.n;
    const int hl = row_ok[r] ? row - node[r] * p.group : 0;
    out_row[r] = ((size_t)b * p.n + node[r]) * p.hq + (size_t)g * p.group + hl;
    const float* qp = static_cast<const float*>(p.q) + out_row[r] * D + 4 * q;
#pragma unroll
    for (int c = 0; c < KC; ++c) qf[r][c] = row_ok[r] ? *reinterpret_cast<const f32x4*>(qp + 16 * c) : f32x4{};
  }
  const bool tree_words = TREE && has_new;
  int par = -1;
  if (tree_words && wave == 0 && lane < p.n) par = p.parents[(size_t)b * p.n + lane];

  // Block j of the split: its first key row, the rows' stride in floats and
  // the number of valid keys.  Rows past the valid ones re-read the last
  // valid row (their scores are masked).
  struct Block {
    const float* base;
    unsigned stride;
    int nv;
  };
  auto block = [&](int j, bool v_side) __attribute__((always_inline)) {
    Block o;
    if (j < nb_ctx) {
      const int key0 = k_begin + 16 * j;
      o.base = static_cast<const float*>(v_side ? p.v_ctx : p.k_ctx) + (((size_t)b * p.hkv + g) * p.cap + key0) * D;
      o.stride = D;
      o.nv = min(16, k_end - key0);
    } else {
      const int key0 = 16 * (j - nb_ctx);
      o.base = static_cast<const float*>(v_side ? p.v_new : p.k_new) + (((size_t)b * p.n + key0) * p.hkv + g) * D;
      o.stride = (unsigned)p.hkv * D;
      o.nv = min(16, p.n - key0);
    }
    return o;
  };
  f32x4 kr[KC], vr[4][VC];
  auto load_k = [&](int j) __attribute__((always_inline)) {
    const Block o = block(j, false);
    const float* a = o.base + (unsigned)min(m16, o.nv - 1) * o.stride + 4 * q;
#pragma unroll
    for (int c = 0; c < KC; ++c) kr[c] = *reinterpret_cast<const f32x4*>(a + 16 * c);
  };
  auto load_v = [&](int j) __attribute__((always_inline)) {
    const Block o = block(j, true);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float* a = o.base + (unsigned)min(4 * q + i, o.nv - 1) * o.stride + 4 * m16;
#pragma unroll
      for (int v = 0; v < VC; ++v) vr[i][v] = *reinterpret_cast<const f32x4*>(a + 64 * v);
    }
  };

  f32x4 O[R][DB];
  float m_run[R], l_run[R], nmc[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    m_run[r] = kNegInf;
    l_run[r] = 0.f;
    nmc[r] = 0.f;
#pragma unroll
    for (int d = 0; d < DB; ++d) O[r][d] = f32x4{};
  }
  const float c = p.scale_log2;

  if (wave < nb) {
    load_k(wave);
    load_v(wave);
  }
  if (tree_words) {
    if (wave == 0) {
      const unsigned long long anc = ancestor_word(par, lane);
      if (lane < p.n) sAnc[lane] = anc;
    }
    __syncthreads();
  }

  // MORE: the wave has another block, whose loads go out here.  (Peeled, not a
  // condition: a conditional load makes the compiler's waits for K also wait
  // for the V loads issued after it.)
  auto step = [&](int j, auto MORE_) __attribute__((always_inline)) {
    constexpr bool MORE = decltype(MORE_)::value;
    // Two accumulators per row part: chains half as long, which with one row
    // part a wave keep consecutive instructions from waiting for each other,
    // and with two halve the scores' error (outputs 3.9e-7 from 64 bits
    // instead of 5.0e-7 at 4096 keys; scalar multiply-adds had 4.5e-7).
    constexpr int CH = 2;
    f32x4 S[R][CH];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int h = 0; h < CH; ++h) S[r][h] = f32x4{};
#pragma unroll
    for (int k = 0; k < KC; ++k)
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int r = 0; r < R; ++r)
          S[r][u % CH] = __builtin_amdgcn_mfma_f32_16x16x4f32(kr[k][u], qf[r][k][u], S[r][u % CH], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
    if (MORE) load_k(j + W);

    // softmax of the block; key 4 q + i of a context block is visible if it
    // is valid, of a new-key block also if it is an ancestor-or-self
    const bool is_new = j >= nb_ctx;
    const int key0 = is_new ? 16 * (j - nb_ctx) : 0;
    const int nv = is_new ? min(16, p.n - key0) : min(16, k_end - k_begin - 16 * j);
    float e[R][4], l_new[R];
    bool redo = false;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      S[r][0] += S[r][1];
      if (nv < 16 || (TREE && is_new)) {
        unsigned long long anc = ~0ull;
        if (TREE && is_new && node[r] < p.n) anc = sAnc[node[r]];
        anc >>= key0 + 4 * q;
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (4 * q + i >= nv || !((anc >> i) & 1ull)) S[r][0][i] = kNegInf;
      }
      float sum = 0.f;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        e[r][i] = __builtin_amdgcn_exp2f(fmaf(S[r][0][i], c, nmc[r]));
        sum += e[r][i];
      }
      redo = redo || m_run[r] == kNegInf || !(sum <= kSumLimit);
      l_new[r] = l_run[r] + sum;
    }
    if (__builtin_amdgcn_ballot_w64(redo)) {
      // no reference yet, or one far below the scores: move it to the rows'
      // maximum, rescale, and take the block's probabilities again
#pragma unroll
      for (int r = 0; r < R; ++r) {
        float mx = fmaxf(fmaxf(S[r][0][0], S[r][0][1]), fmaxf(S[r][0][2], S[r][0][3]));
        mx = fmaxf(mx, __shfl_xor(mx, 16));
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        const float m_new = fmaxf(m_run[r], mx);
        const float m_use = m_new == kNegInf ? 0.f : m_new;
        const float alpha = __builtin_amdgcn_exp2f((m_run[r] - m_use) * c);
        m_run[r] = m_new;
        nmc[r] = -m_use * c;
        float sum = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          e[r][i] = __builtin_amdgcn_exp2f(fmaf(S[r][0][i], c, nmc[r]));
          sum += e[r][i];
        }
        l_new[r] = l_run[r] * alpha + sum;
#pragma unroll
        for (int d = 0; d < DB; ++d) O[r][d] *= alpha;
      }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) l_run[r] = l_new[r];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int d = 0; d < DB; ++d)
#pragma unroll
        for (int r = 0; r < R; ++r)
          O[r][d] = __builtin_amdgcn_mfma_f32_16x16x4f32(vr[i][d >> 2][d & 3], e[r][i], O[r][d], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
    if (MORE) load_v(j + W);
  };
  if (wave < nb) {
    int j = wave;
    for (; j + W < nb; j += W) step(j, std::true_type{});
    step(j, std::false_type{});
  }

  // Merge of the workgroup's waves: every wave scales its output to the common
  // maximum and leaves it in LDS; then each wave sums its share of the output.
#pragma unroll
  for (int r = 0; r < R; ++r) {
    l_run[r] += __shfl_xor(l_run[r], 16);
    l_run[r] += __shfl_xor(l_run[r], 32);
    if (q == 0) sML[wave][16 * r + m16] = make_float2(m_run[r] == kNegInf ? kNegInf : m_run[r] * c, l_run[r]);
  }
  __syncthreads();
  float M[R], lsum[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    float2 ml[W];
    M[r] = kNegInf;
#pragma unroll
    for (int w = 0; w < W; ++w) {
      ml[w] = sML[w][16 * r + m16];
      M[r] = fmaxf(M[r], ml[w].x);
    }
    lsum[r] = 0.f;
    float mine = 0.f;
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const float f = ml[w].x == kNegInf ? 0.f : __builtin_amdgcn_exp2f(ml[w].x - M[r]);
      lsum[r] = fmaf(f, ml[w].y, lsum[r]);
      mine = w == wave ? f : mine;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int v = 0; v < VC; ++v)
        sO[wave][(r * 4 + i) * VC + v][lane] = f32x4{O[r][4 * v][i] * mine, O[r][4 * v + 1][i] * mine,
                                                     O[r][4 * v + 2][i] * mine, O[r][4 * v + 3][i] * mine};
  }
  __syncthreads();
  const bool split = nsb > 1;
  const size_t pr0 = (((size_t)b * p.hkv + g) * p.nsplit + s) * p.rows_pad + (size_t)rg * R * 16 + m16;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const float inv = split ? 1.f : 1.f / lsum[r];
    float* dst = split ? p.part_o + (pr0 + 16 * r) * D : static_cast<float*>(p.out) + out_row[r] * D;
#pragma unroll
    for (int t = 0; t < 4 * VC; t += W) {  // slot t + wave: dims 64 v + 4 (4 q + i) .. +3
      const int slot = t + wave;
      if (4 * VC % W == 0 || slot < 4 * VC) {
        f32x4 acc = sO[0][r * 4 * VC + slot][lane];
#pragma unroll
        for (int w = 1; w < W; ++w) acc += sO[w][r * 4 * VC + slot][lane];
        const int i = slot / VC, v = slot % VC;
        if (split || row_ok[r]) *reinterpret_cast<f32x4*>(dst + 64 * v + 4 * (4 * q + i)) = acc * inv;
      }
    }
    if (wave == 0 && q == 0) {
      if (split) p.part_ml[pr0 + 16 * r] = make_float2(M[r], lsum[r]);
      else if (p.lse && row_ok[r]) p.lse[out_row[r]] = log_sum(M[r], lsum[r]);
    }
  }
}

template <int D, bool TREE>
void launch(const AttnParams& p, dim3 grid, hipStream_t s) {
  if (p.rows_rg == 16) hipLaunchKernelGGL((attn_f32<D, TREE, 1, 8>), grid, dim3(512), 0, s, p);
  else hipLaunchKernelGGL((attn_f32<D, TREE, 2, 4>), grid, dim3(256), 0, s, p);
}

}  // namespace

hipError_t launch_attn_f32(const AttnParams& p, bool tree, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
  const int items = p.nsplit * p.batch * p.hkv * p.row_groups;
  const dim3 grid((items + 7) / 8 * 8);
  if (ev0) (void)hipEventRecord(ev0, s);
  if (p.d == 128) {
    if (tree) launch<128, true>(p, grid, s);
    else launch<128, false>(p, grid, s);
  } else {
    if (tree) launch<64, true>(p, grid, s);
    else launch<64, false>(p, grid, s);
  }
  hipError_t e = hipGetLastError();
  if (ev1) (void)hipEventRecord(ev1, s);
  return e;
}

}  // namespace glance
