// Draft tree builder: the N strings of highest plug-in score
// sum_j log q_j(y_j), q_j the softmax of the drafter's logits at offset j
// (Assumption 1, Sec. 3.2), packed as a prefix-closed tree (Sec. 3.3;
// Algorithm 1, second step).
//
// Ranking, in fp32: the tokens of an offset by (logit desc, index asc); the
// strings by (score desc, length asc, rank vector lexicographic asc), each
// score summed from the first offset on.  Node 0 is the root, nodes 1..N the
// kept strings in ranking order, so parents[i] < i.  A kept string only ever
// uses the K = min(N, vocab) best-ranked tokens of each offset: swapping a
// token for a better-ranked one never moves a string back, so a string with a
// token of rank >= N would follow N others.
//
// tree_scan    grid (slice group, row), one 1024-value slice per wave, read
//              once: per slice (max, sum exp(x - max)) for the
//              log-normaliser, the maxima of `groups` disjoint lane groups
//              (the row's sketch), and the slice's candidates.  A slice
//              cannot see the row, so it keeps its values >= its own
//              threshold thr, the smallest of the maxima of its four 16-lane
//              rows: every value it leaves out lies below thr.  Candidates go
//              to the slice's own slots (no atomics).
// tree_rank    one workgroup per row: the log-normaliser from the slice
//              statistics; the row threshold tau, the K-th largest entry of the
//              sketch (its entries are maxima of disjoint lane groups, so at
//              least K values of the row are >= tau and the K best all are);
//              the candidates >= tau gathered and ranked by counting.  A slice
//              whose thr lies above tau may have left out values >= tau, and a
//              slice whose slots overflowed lost some: those slices are read
//              again.  Only if too many candidates are found is the K-th
//              largest key of the row found by radix selection over the whole
//              row.  The row's K best (log q, token) are written in rank order.
// tree_enum    one wave per sequence: the best-first enumeration.  Lane i is
//              node i; the frontier holds each emitted node's next unemitted
//              child (its children leave in rank order), kept in the node's
//              lane.  Each step takes the wave's best string by a
//              min-reduction, emits it as node k into lane k, which takes its
//              first child (rank 0 at the next offset), and moves the parent's
//              lane on to its next child (same prefix, next rank).  Each string
//              is generated by exactly one string ranked before it, so strings
//              leave the frontier in ranking order; N <= 63 nodes fit in 64
//              lanes.
//
// The passes hand data over through kernel boundaries only: no global
// atomics and no device-scope fences, which serialise across the chip.
//
// Candidates are packed as (order key << 32) | ~index, so the larger packed
// word is the larger logit, then the lower index: every word is distinct.
#include "glance_internal.h"

namespace glance {
namespace {

typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
typedef __attribute__((ext_vector_type(2))) unsigned int u32x2;
// at any bf16 or fp32 element: rows of any length take vector loads, which
// the memory pipeline serves unaligned
typedef u32x4 u32x4_any __attribute__((aligned(2)));
typedef u32x2 u32x2_any __attribute__((aligned(2)));
typedef unsigned long long u64;

constexpr int kThreads = 256;
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr float kInf = __builtin_inff();

__device__ __forceinline__ float as_f32(unsigned u) { return __builtin_bit_cast(float, u); }
__device__ __forceinline__ unsigned as_u32(float f) { return __builtin_bit_cast(unsigned, f); }

// Unsigned order key of a float: larger value, larger key; +0 and -0 share a
// key (they are equal logits and tie on the index).  NaN is outside the contract.
__device__ __forceinline__ unsigned order_key(float v) {
  const unsigned bits = as_u32(v);
  const unsigned k = (bits & 0x80000000u) ? 0x80000000u - bits : bits;
  return k ^ 0x80000000u;
}

__device__ __forceinline__ float key_value(unsigned key) {
  const unsigned k = key ^ 0x80000000u;
  return as_f32((int)k >= 0 ? k : 0x80000000u - k);
}

__device__ __forceinline__ u64 pack(float v, int idx) {
  return ((u64)order_key(v) << 32) | (u64)(0xffffffffu - (unsigned)idx);
}

template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) {  // lanes without a source keep their own value
  return as_f32((unsigned)__builtin_amdgcn_update_dpp((int)as_u32(v), (int)as_u32(v), CTRL, 0xf, 0xf, false));
}

// Max / min over the wave of a signed int, returned uniform: the row-level
// butterflies, then row_bcast:15 and row_bcast:31 fold the four rows into
// lane 63.  VALU and DPP only: no LDS round trip.  All 64 lanes must be
// active (DPP reads of inactive lanes are undefined), so callers reduce
// before any branch on a lane condition.
// Lanes a row mask leaves out read the operation's neutral element ID, which
// lets the compiler fuse each step into one v_max_i32_dpp / v_min_i32_dpp.
template <int CTRL, int ROWS, int ID>
__device__ __forceinline__ int dpp_i(int v) {
  return __builtin_amdgcn_update_dpp(ID, v, CTRL, ROWS, 0xf, false);
}
__device__ __forceinline__ int wave_max_i(int v) {
  constexpr int I = (int)0x80000000;
  v = max(v, dpp_i<0xb1, 0xf, I>(v));
  v = max(v, dpp_i<0x4e, 0xf, I>(v));
  v = max(v, dpp_i<0x141, 0xf, I>(v));
  v = max(v, dpp_i<0x140, 0xf, I>(v));
  v = max(v, dpp_i<0x142, 0xa, I>(v));
  v = max(v, dpp_i<0x143, 0xc, I>(v));
  return __builtin_amdgcn_readlane(v, 63);
}
__device__ __forceinline__ int wave_min_i(int v) {
  constexpr int I = 0x7fffffff;
  v = min(v, dpp_i<0xb1, 0xf, I>(v));
  v = min(v, dpp_i<0x4e, 0xf, I>(v));
  v = min(v, dpp_i<0x141, 0xf, I>(v));
  v = min(v, dpp_i<0x140, 0xf, I>(v));
  v = min(v, dpp_i<0x142, 0xa, I>(v));
  v = min(v, dpp_i<0x143, 0xc, I>(v));
  return __builtin_amdgcn_readlane(v, 63);
}

// Signed order key of a score: larger score, larger key; -0 folds onto +0.
__device__ __forceinline__ int score_key(float s) {
  const int b = (int)as_u32(s + 0.f);
  return b ^ ((b >> 31) & 0x7fffffff);
}

__device__ __forceinline__ float key_float(int k) { return as_f32((unsigned)(k ^ ((k >> 31) & 0x7fffffff))); }
__device__ __forceinline__ float wave_max_f(float v) { return key_float(wave_max_i(score_key(v))); }
__device__ __forceinline__ float wave_min_f(float v) { return key_float(wave_min_i(score_key(v))); }
__device__ __forceinline__ float wave_sum_f(float v) {  // rows not written by a broadcast add 0
  v += dpp_f<0xb1>(v);
  v += dpp_f<0x4e>(v);
  v += dpp_f<0x141>(v);
  v += dpp_f<0x140>(v);
  v += as_f32((unsigned)__builtin_amdgcn_update_dpp(0, (int)as_u32(v), 0x142, 0xa, 0xf, false));
  v += as_f32((unsigned)__builtin_amdgcn_update_dpp(0, (int)as_u32(v), 0x143, 0xc, 0xf, false));
  return as_f32((unsigned)__builtin_amdgcn_readlane((int)as_u32(v), 63));
}

__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ int lane_of(int v, int l) { return __builtin_amdgcn_readlane(v, l); }

template <bool BF16>
__device__ __forceinline__ float load_one(const char* rowp, int e) {
  if (BF16) return as_f32((unsigned)reinterpret_cast<const unsigned short*>(rowp)[e] << 16);
  return reinterpret_cast<const float*>(rowp)[e];
}

// Values per 16-byte load and loads per lane for the 16 values a lane holds.
template <bool BF16> struct SliceShape {
  static constexpr int kVpl = BF16 ? 8 : 4;
  static constexpr int kLoads = 16 / kVpl;
};

// Position in the row of value i (0..15) of `lane` in the slice at `base`:
// load l covers 64 consecutive 16-byte pieces, lane `lane` takes piece `lane`.
template <bool BF16>
__device__ __forceinline__ int slice_pos(int base, int lane, int i) {
  constexpr int V = SliceShape<BF16>::kVpl;
  return base + (i / V) * 64 * V + lane * V + (i % V);
}

// The 16 values of one lane in one slice; positions past the row read -inf.
template <bool BF16>
__device__ __forceinline__ void load_slice(const char* rowp, int base, int vocab, int lane, float (&v)[16]) {
  constexpr int V = SliceShape<BF16>::kVpl;
#pragma unroll
  for (int l = 0; l < SliceShape<BF16>::kLoads; ++l) {
    const int e0 = slice_pos<BF16>(base, lane, l * V);
    if (e0 + V <= vocab) {
      const u32x4 w = *reinterpret_cast<const u32x4_any*>(rowp + (size_t)e0 * (BF16 ? 2 : 4));
      if (BF16) {
        v[l * 8 + 0] = as_f32(w.x << 16);
        v[l * 8 + 1] = as_f32(w.x & 0xffff0000u);
        v[l * 8 + 2] = as_f32(w.y << 16);
        v[l * 8 + 3] = as_f32(w.y & 0xffff0000u);
        v[l * 8 + 4] = as_f32(w.z << 16);
        v[l * 8 + 5] = as_f32(w.z & 0xffff0000u);
        v[l * 8 + 6] = as_f32(w.w << 16);
        v[l * 8 + 7] = as_f32(w.w & 0xffff0000u);
      } else {
        v[l * 4 + 0] = as_f32(w.x);
        v[l * 4 + 1] = as_f32(w.y);
        v[l * 4 + 2] = as_f32(w.z);
        v[l * 4 + 3] = as_f32(w.w);
      }
    } else {
#pragma unroll
      for (int u = 0; u < V; ++u) v[l * V + u] = e0 + u < vocab ? load_one<BF16>(rowp, e0 + u) : -kInf;
    }
  }
}

// The same for a slice wholly inside the row: plain vector
// loads with no per-lane guard (a per-lane guard makes each load a branch of
// its own, waited on before the next is issued).  Issue first, convert after,
// so that all of a wave's loads are in flight together.
template <bool BF16>
__device__ __forceinline__ void issue_slice_full(const char* rowp, int base, int lane,
                                                 u32x4 (&w)[SliceShape<BF16>::kLoads]) {
  constexpr int V = SliceShape<BF16>::kVpl;
#pragma unroll
  for (int l = 0; l < SliceShape<BF16>::kLoads; ++l)
    w[l] = *reinterpret_cast<const u32x4_any*>(rowp + (size_t)slice_pos<BF16>(base, lane, l * V) * (BF16 ? 2 : 4));
}
template <bool BF16>
__device__ __forceinline__ void unpack_slice(const u32x4 (&w)[SliceShape<BF16>::kLoads], float (&v)[16]) {
#pragma unroll
  for (int l = 0; l < SliceShape<BF16>::kLoads; ++l) {
    if (BF16) {
      v[l * 8 + 0] = as_f32(w[l].x << 16);
      v[l * 8 + 1] = as_f32(w[l].x & 0xffff0000u);
      v[l * 8 + 2] = as_f32(w[l].y << 16);
      v[l * 8 + 3] = as_f32(w[l].y & 0xffff0000u);
      v[l * 8 + 4] = as_f32(w[l].z << 16);
      v[l * 8 + 5] = as_f32(w[l].z & 0xffff0000u);
      v[l * 8 + 6] = as_f32(w[l].w << 16);
      v[l * 8 + 7] = as_f32(w[l].w & 0xffff0000u);
    } else {
      v[l * 4 + 0] = as_f32(w[l].x);
      v[l * 4 + 1] = as_f32(w[l].y);
      v[l * 4 + 2] = as_f32(w[l].z);
      v[l * 4 + 3] = as_f32(w[l].w);
    }
  }
}

__device__ __forceinline__ const char* row_ptr(const TreeParams& p, int row, size_t esz) {
  const int b = row / p.horizon, j = row - b * p.horizon;
  return static_cast<const char*>(p.logits) + ((size_t)b * p.seq_stride + (size_t)j * p.vocab) * esz;
}

// Inclusive prefix sum over the wave: row shifts within each 16-lane row (a
// lane without a source adds 0), then lane 15 / lane 31 broadcast into the
// rows after them.
__device__ __forceinline__ int wave_incl_sum(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true);  // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true);  // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true);  // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true);  // row_shr:8
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // row_bcast:15
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);  // row_bcast:31
  return v;
}

// Maximum over each 16-lane row of the wave, in every lane of the row (the
// first four steps of wave_max_i).
__device__ __forceinline__ int row_max_i(int v) {
  constexpr int I = (int)0x80000000;
  v = max(v, dpp_i<0xb1, 0xf, I>(v));
  v = max(v, dpp_i<0x4e, 0xf, I>(v));
  v = max(v, dpp_i<0x141, 0xf, I>(v));
  v = max(v, dpp_i<0x140, 0xf, I>(v));
  return v;
}

// The statistics, sketch entries and candidates of one slice whose 16 values
// per lane are in v.  FULL: every position of the slice lies inside the row,
// so no position is checked.  Candidates are the values >= thr, taken value
// index by value index across the wave (one ballot each), so that a slot is
// the count before it in the wave and the count is a scalar sum; the order
// of a slice's candidates is immaterial to the ranking pass.
template <bool BF16, bool FULL>
__device__ __forceinline__ void scan_slice(const TreeParams& p, int row, int slice, int lane, const float (&v)[16]) {
  constexpr int V = SliceShape<BF16>::kVpl;
  const int base = slice * kTreeSlice;
  float lm = v[0];
#pragma unroll
  for (int i = 1; i < 16; ++i) lm = fmaxf(lm, v[i]);
  // row maxima -> slice maximum and the slice's threshold
  const int rk = row_max_i(score_key(lm));
  int mk = lane_of(rk, 0), tk = mk;
#pragma unroll
  for (int r = 1; r < 4; ++r) {
    const int x = lane_of(rk, 16 * r);
    mk = max(mk, x);
    // row r's first position is slice_pos(base, 16 r, 0)
    if (FULL || base + 16 * r * V < p.vocab) tk = min(tk, x);
  }
  const float m = key_float(mk), thr = key_float(tk);
  float sum = 0.f;
  if (m != -kInf) {
    // the maximum comes off before the scaling: masked tokens may hold the
    // type's lowest value, which times log2 e overflows
#pragma unroll
    for (int i = 0; i < 16; ++i) sum += __builtin_amdgcn_exp2f((v[i] - m) * kLog2e);
  }
  sum = wave_sum_f(sum);
  const size_t sl = (size_t)row * p.slices + slice;
  if (lane == 0) {
    p.stats[sl] = make_float2(m, sum);
    p.thr[sl] = thr;
  }
  const int gs = 64 / p.groups;  // lanes per sketch group
  if (gs == 64) {
    if (lane == 0) p.sketch[sl] = m;
  } else {
    float g = lm;
    for (int off = 1; off < gs; off <<= 1) g = fmaxf(g, __shfl_xor(g, off));
    if ((lane & (gs - 1)) == 0) p.sketch[sl * p.groups + lane / gs] = g;
  }
  // the values >= thr, packed, into the slice's own slots
  u64* dst = p.cand + sl * kTreeSliceCap;
  const int e_lane = base + lane * V;  // position of value 0 of this lane
  int n = 0;                            // uniform: candidates of value indexes before i
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int e = e_lane + (i / V) * 64 * V + (i % V);
    const bool keep = v[i] >= thr && (FULL || e < p.vocab);
    const u64 b = __builtin_amdgcn_ballot_w64(keep);
    if (b) {
      if (keep) {
        const int slot = n + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(b >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)b, 0u));
        if (slot < kTreeSliceCap) dst[slot] = pack(v[i], e);
      }
      n += __popcll(b);
    }
  }
  if (lane == 0) p.ccount[sl] = n;
}

// One read of the logits: per 1024-value slice the normaliser statistics, the
// sketch, and the candidates.  A slice cannot know the row's threshold, so it
// keeps the values >= its own threshold thr: the smallest of the maxima of its
// four 16-lane rows (rows holding no position of the slice left out), so at
// least one value per row, and every value it leaves out lies below thr.
template <bool BF16>
__global__ __launch_bounds__(64 * kTreeScanWaves) void tree_scan(TreeParams p) {
  const int row = blockIdx.y;
  const int lane = threadIdx.x & 63;
  const int s0 = (blockIdx.x * kTreeScanWaves + (threadIdx.x >> 6)) * kTreeSlicesPerWave;
  if (s0 >= p.slices) return;
  const char* rowp = row_ptr(p, row, BF16 ? 2 : 4);
  float v[kTreeSlicesPerWave][16];
  if ((long)(s0 + kTreeSlicesPerWave) * kTreeSlice <= p.vocab) {  // uniform: every slice full
    u32x4 w[kTreeSlicesPerWave][SliceShape<BF16>::kLoads];
#pragma unroll
    for (int u = 0; u < kTreeSlicesPerWave; ++u) issue_slice_full<BF16>(rowp, (s0 + u) * kTreeSlice, lane, w[u]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < kTreeSlicesPerWave; ++u) {
      unpack_slice<BF16>(w[u], v[u]);
      scan_slice<BF16, true>(p, row, s0 + u, lane, v[u]);
    }
  } else {
#pragma unroll
    for (int u = 0; u < kTreeSlicesPerWave; ++u)
      if (s0 + u < p.slices) load_slice<BF16>(rowp, (s0 + u) * kTreeSlice, p.vocab, lane, v[u]);
#pragma unroll
    for (int u = 0; u < kTreeSlicesPerWave; ++u)
      if (s0 + u < p.slices) scan_slice<BF16, false>(p, row, s0 + u, lane, v[u]);
  }
}

constexpr int kRescanCap = 64;  // slices re-read by the ranking pass before the exact fallback

struct RankShared {
  __attribute__((aligned(16))) u64 cand[kTreeCap + 32];
  __attribute__((aligned(16))) float ent[kThreads];  // the row's sketch
  __attribute__((aligned(16))) u64 top[64];          // the exact fallback's result
  int hist[256];
  float red[12];
  int n, digit, above;
  int nres;
  int res[kRescanCap];
  int part[kThreads];
};

// Exact top-K of a whole row when its candidates overflow the ranking: radix
// selection of the K-th largest packed word, 8 bits per pass from the top,
// then the K words >= it.  Reads the row nine times; only inputs with very
// many values tied near the top (or fewer than K finite values) come here.
template <bool BF16>
__device__ void radix_top(const TreeParams& p, const char* rowp, RankShared& sh) {
  const int tid = threadIdx.x;
  u64 prefix = 0, pmask = 0;
  int krem = p.k;
  for (int shift = 56; shift >= 0; shift -= 8) {
    sh.hist[tid] = 0;
    __syncthreads();
    for (int e = tid; e < p.vocab; e += kThreads) {
      const u64 key = pack(load_one<BF16>(rowp, e), e);
      if ((key & pmask) == prefix) atomicAdd(&sh.hist[(key >> shift) & 255], 1);
    }
    __syncthreads();
    if (tid == 0) {
      int cum = 0, d = 255;
      for (; d > 0; --d) {
        if (cum + sh.hist[d] >= krem) break;
        cum += sh.hist[d];
      }
      sh.digit = d;
      sh.above = cum;
    }
    __syncthreads();
    prefix |= (u64)sh.digit << shift;
    pmask |= (u64)0xff << shift;
    krem -= sh.above;
    __syncthreads();
  }
  if (tid == 0) sh.n = 0;
  __syncthreads();
  for (int e = tid; e < p.vocab; e += kThreads) {
    const u64 key = pack(load_one<BF16>(rowp, e), e);
    if (key >= prefix) {
      const int slot = atomicAdd(&sh.n, 1);
      if (slot < 64) sh.cand[slot] = key;
    }
  }
  __syncthreads();
  if (tid < p.k) {
    const u64 key = sh.cand[tid];
    int rank = 0;
    for (int i = 0; i < p.k; ++i) rank += sh.cand[i] > key;
    sh.top[rank] = key;
  }
}

// Best-first enumeration of one sequence's tree by one wave (see the header).
//
// Lane i is node i, node 0 the root.  The frontier holds at most one string
// per emitted node, its next unemitted child: a node's children leave in rank
// order and child r + 1 enters when child r leaves.  Lane i keeps that string
// as its key (the float bits of its score with the sign bit set: for the
// scores <= 0 here the smallest key is the best score, and +0 / -0 meet;
// INT_MAX once node i has no child left or is not emitted yet), a node word
// (length, pending rank, parent, own rank) and the node's score, and, from
// the offset tables in LDS, what the string hands over if it is taken next:
// its node word and its first child's key, and the key of the lane's next
// child.  A step takes the smallest key (lane P) and moves those values with
// one readlane / writelane pair each: the string becomes node k in lane k with
// its first child as lane k's pending string, and lane P moves on to its next
// child.  Tokens are looked up once at the end, from each node's offset and
// own rank.
struct EnumShared {
  uint2 ent[kTreeMaxHorizon + 1][64];  // (q_j(rank r + 1), token of rank r) at offset j
  float first[kTreeMaxHorizon + 2];    // q_j(rank 0)
};

// A lane's node word: node length (bits 0-3) | pending rank (4-9) | parent
// (10-15) | own rank (16-21).
__device__ __forceinline__ int node_len(int w) { return w & 15; }
__device__ __forceinline__ int node_pending(int w) { return (w >> 4) & 63; }
__device__ __forceinline__ int node_parent(int w) { return (w >> 10) & 63; }
__device__ __forceinline__ int node_rank(int w) { return w >> 16; }

// Rank-vector order of the pending strings of lanes x != y, which have the
// same length: walk both nodes up to their lowest common ancestor; its two
// children on the paths hold the first differing rank.  Only exact score ties
// come here, so plain readlanes.
__device__ __forceinline__ bool lex_before(int x, int y, int node) {
  int rx = 0, ry = 0;
  while (x != y) {
    const int wx = lane_of(node, x), wy = lane_of(node, y);
    rx = node_rank(wx);
    ry = node_rank(wy);
    x = node_parent(wx);
    y = node_parent(wy);
  }
  return rx < ry;
}

// Among frontier lanes tied on the score: the shortest pending string, then
// the smallest rank vector.  Ties are few lanes at a time: a scalar pass over
// them.  Equal lengths mean distinct nodes of one depth, whose paths differ,
// so the node paths decide before the pending ranks would.
__device__ __forceinline__ int tie_break(u64 tied, int node) {
  int best = __builtin_ctzll(tied), lb = node_len(lane_of(node, best));
  tied &= tied - 1;
  while (tied) {
    const int x = __builtin_ctzll(tied), lx = node_len(lane_of(node, x));
    tied &= tied - 1;
    if (lx < lb || (lx == lb && lex_before(x, best, node))) {
      best = x;
      lb = lx;
    }
  }
  return best;
}

// v_writelane: `v` in lane `l`, the other lanes keep `old` (uniform v and l).
extern "C" __device__ int glance_writelane_i32(int v, int l, int old) __asm("llvm.amdgcn.writelane.i32");
__device__ __forceinline__ int put_lane(int v, int l, int old) { return glance_writelane_i32(v, l, old); }

__device__ void enumerate(const TreeParams& p, int b, int lane) {
  __shared__ EnumShared es;
  const int N = p.budget, L = p.horizon, K = p.k;
  constexpr int kEmpty = 0x7fffffff;
  // all table loads in flight at once, then the LDS layout (the ranking pass
  // wrote slot r as (log q of rank r + 1, token of rank r), slot 63 the log q
  // of rank 0)
  float q[kTreeMaxHorizon];
  int t[kTreeMaxHorizon];
#pragma unroll
  for (int j = 0; j < kTreeMaxHorizon; ++j) {
    // plain loads of every slot (rows past the horizon repeat the last): a
    // condition would make a branch of each
    const size_t at = ((size_t)b * L + min(j, L - 1)) * 64 + lane;
    q[j] = p.lq[at];
    t[j] = p.tok[at];
  }
#pragma unroll
  for (int j = 0; j < kTreeMaxHorizon; ++j) {
    const bool in = j < L && lane < K;
    es.ent[j][lane] = make_uint2(as_u32(in ? q[j] : -kInf), (unsigned)t[j]);
    if (lane == 63) es.first[j] = j < L ? q[j] : -kInf;
  }
  es.ent[kTreeMaxHorizon][lane] = make_uint2(as_u32(-kInf), 0u);
  if (lane < 2) es.first[kTreeMaxHorizon + lane] = -kInf;
  __syncthreads();
  int key = lane == 0 && L > 0 ? (int)(as_u32(es.first[0]) | 0x80000000u) : kEmpty;
  int node = 0;  // node word
  int nsc = 0;   // the node's score (float bits)
  // What each lane's pending string hands over if it is taken next: its node
  // word and its first child's key, and the key of the lane's next child
  // (lane-local, recomputed after every step; only lanes k and P change).
  // The table reads are issued after a step's updates and used after the
  // next step's reduction, which hides their latency.
  int c_key, c_node, s_key;
  float e_next, qc;
  auto issue = [&]() {
    const int len = node_len(node);
    e_next = as_f32(es.ent[len][node_pending(node)].x);
    qc = es.first[len + 1];
  };
  auto finish = [&]() {
    const int len = node_len(node), r = node_pending(node);
    const int ck = (int)(as_u32(as_f32((unsigned)key) + qc) | 0x80000000u);
    const int sk = (int)(as_u32(as_f32((unsigned)nsc) + e_next) | 0x80000000u);
    c_key = len + 1 < L ? ck : kEmpty;
    s_key = r + 1 < K ? sk : kEmpty;
    c_node = (len + 1) | (lane << 10) | (r << 16);
  };
  // The host's budget check guarantees N strings, so the frontier never
  // empties before node N (an empty one would only repeat an in-range lane).
  // Node k = lane P's pending string, recorded in lane k.
  auto pick = [&](int m) {
    const u64 tied = __ballot(key == m);
    return (tied & (tied - 1)) ? uniform(tie_break(tied, node)) : (int)__builtin_ctzll(tied);
  };
  issue();
  for (int k = 1; k < N; ++k) {
    const int m = wave_min_i(key);
    finish();
    const int P = pick(m);
    // lane k takes node k with its first child; lane P moves on to its next child
    node = put_lane(lane_of(c_node, P), k, node);
    nsc = put_lane(m, k, nsc);
    key = put_lane(lane_of(c_key, P), k, key);
    const bool me = lane == P;
    key = me ? s_key : key;
    node = me ? node + 16 : node;
    issue();
  }
  {
    const int m = wave_min_i(key);
    finish();
    const int P = pick(m);
    node = put_lane(lane_of(c_node, P), N, node);
    nsc = put_lane(m, N, nsc);
  }
  // node i's token: rank node_rank at offset node_len - 1
  int32_t* par_out = p.parents + (size_t)b * (N + 1);
  int32_t* tok_out = p.tokens + (size_t)b * (N + 1);
  if (lane <= N) {
    const int len = node_len(node);
    par_out[lane] = lane == 0 ? -1 : node_parent(node);
    tok_out[lane] = lane == 0 ? p.roots[b] : (int)es.ent[len > 0 ? len - 1 : 0][node_rank(node)].y;
    if (p.scores) p.scores[(size_t)b * (N + 1) + lane] = as_f32((unsigned)nsc);
  }
}

template <bool BF16>
__global__ __launch_bounds__(kThreads) void tree_rank(TreeParams p) {
  __shared__ RankShared sh;
  const int row = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const char* rowp = row_ptr(p, row, BF16 ? 2 : 4);
  if (tid == 0) {
    sh.n = 0;
    sh.nres = 0;
  }
  const float2* st = p.stats + (size_t)row * p.slices;
  const float* th = p.thr + (size_t)row * p.slices;
  const int* cnt = p.ccount + (size_t)row * p.slices;
  const int S = p.slices * p.groups;
  const float* sk = p.sketch + (size_t)row * S;
  const bool counted = S <= kThreads;

  // Every first read in flight at once, one slice per thread (further slices
  // of very long rows in the loops below): the slice's statistics, threshold,
  // candidate count and first 16 candidate slots (slots past the count stay
  // inside the slice's slots and are ignored), and the thread's sketch entry.
  const bool in0 = tid < p.slices;
  const float2 st0 = in0 ? st[tid] : make_float2(-kInf, 0.f);
  const float th0 = in0 ? th[tid] : -kInf;
  const int c0 = in0 ? cnt[tid] : 0;
  const float ent0 = counted && tid < S ? sk[tid] : -kInf;
  u64 ka[16], kb[16];  // slots 0..15 and 16..31 (a slice holds 8.5 candidates on average)
  auto load16 = [&](u64 (&kk)[16], int sl, int j0) {
    const u64* src = p.cand + ((size_t)row * p.slices + sl) * kTreeSliceCap + j0;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const ulonglong2 w = reinterpret_cast<const ulonglong2*>(src)[u];
      kk[2 * u] = w.x;
      kk[2 * u + 1] = w.y;
    }
  };
  load16(ka, in0 ? tid : 0, 0);

  // The row's maximum M and threshold tau: at least K values of the row are >=
  // tau and the K best all are, since the sketch entries are maxima of
  // disjoint lane groups.  Up to 256 entries: tau is their K-th largest, the
  // smallest entry with fewer than K larger ones, each thread counting the
  // entries above its own.  More (rows past 262144 values): lane l < B = ceil(K / 4)
  // of wave 0 keeps the four largest entries of bucket l (entries l, l + B, ...:
  // 16 at least, as K <= 63) and tau is the smallest of the buckets' fourth
  // largest ones.
  float M, tau_part = kInf;
  if (counted) {
    sh.ent[tid] = ent0;
    if (c0 > 16 && c0 <= kTreeSliceCap) load16(kb, tid, 16);  // in flight through the counting
    __syncthreads();
    M = -kInf;
    int above = 0;
    for (int i = 0; i < (S + 3) / 4; ++i) {  // entries past S are -inf
      const float4 x = reinterpret_cast<const float4*>(sh.ent)[i];
      M = fmaxf(fmaxf(fmaxf(x.x, x.y), fmaxf(x.z, x.w)), M);
      above += (x.x > ent0 ? 1 : 0) + (x.y > ent0 ? 1 : 0) + (x.z > ent0 ? 1 : 0) + (x.w > ent0 ? 1 : 0);
    }
    if (tid < S && above < p.k) tau_part = ent0;
  } else {
    if (c0 > 16 && c0 <= kTreeSliceCap) load16(kb, tid, 16);
    M = st0.x;
    for (int i = tid + kThreads; i < p.slices; i += kThreads) M = fmaxf(M, st[i].x);
    M = wave_max_f(M);
    if (lane == 0) sh.red[wave] = M;
    if (wave == 0) {
      const int buckets = (p.k + 3) / 4;
      float t0 = -kInf, t1 = -kInf, t2 = -kInf, t3 = -kInf;
      if (tid < buckets) {
        for (int i = tid; i < S; i += buckets) {
          float x = sk[i], h;
          h = fmaxf(t0, x); x = fminf(t0, x); t0 = h;
          h = fmaxf(t1, x); x = fminf(t1, x); t1 = h;
          h = fmaxf(t2, x); x = fminf(t2, x); t2 = h;
          t3 = fmaxf(t3, x);
        }
      }
      if (tid < buckets) tau_part = t3;
    }
    __syncthreads();
    M = fmaxf(fmaxf(sh.red[0], sh.red[1]), fmaxf(sh.red[2], sh.red[3]));
  }
  float Z = 0.f;
  if (M != -kInf) {
    if (st0.x != -kInf) Z = st0.y * __builtin_amdgcn_exp2f((st0.x - M) * kLog2e);
    for (int i = tid + kThreads; i < p.slices; i += kThreads) {
      const float2 s2 = st[i];
      if (s2.x != -kInf) Z += s2.y * __builtin_amdgcn_exp2f((s2.x - M) * kLog2e);
    }
  }
  Z = wave_sum_f(Z);
  tau_part = wave_min_f(tau_part);
  if (lane == 0) {
    sh.red[4 + wave] = Z;
    sh.red[8 + wave] = tau_part;
  }
  __syncthreads();
  Z = (sh.red[4] + sh.red[5]) + (sh.red[6] + sh.red[7]);
  const float tau = fminf(fminf(sh.red[8], sh.red[9]), fminf(sh.red[10], sh.red[11]));
  // The sum holds the maximum's own term exp(0) = 1, so log Z >= 0; keeping
  // that under rounding keeps every log q <= 0 and scores non-increasing
  // along each path.
  const float lse = M == -kInf ? -kInf : M + fmaxf(__builtin_amdgcn_logf(Z), 0.f) * kLn2;

  // The slices' candidates >= tau, in any order (they are ranked by
  // counting); one LDS atomic per wave and round, the wave's prefix sum
  // placing each lane's keys.  A slice left out only values below its own
  // threshold, so it is whole unless that lies above tau (about one slice in
  // 3500 here) or its slots overflowed: those are read again.
  const unsigned tkey = order_key(tau);
  auto emit = [&](const u64 (&kk)[16], int j0, int c) {
    unsigned pm = 0;
#pragma unroll
    for (int u = 0; u < 16; ++u) pm |= (j0 + u < c && (unsigned)(kk[u] >> 32) >= tkey) ? 1u << u : 0u;
    const int np = __popc(pm);
    const int incl = wave_incl_sum(np);
    int base = 0;
    if (lane == 63) base = atomicAdd(&sh.n, incl);
    int at = lane_of(base, 63) + incl - np;
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      if ((pm >> u) & 1) {
        if (at < kTreeCap) sh.cand[at] = kk[u];
        ++at;
      }
    }
  };
  for (int s0 = 0; s0 < p.slices; s0 += kThreads) {
    const int sl = s0 + tid;
    const bool in = sl < p.slices;
    int c = c0;
    float t = th0, m = st0.x;
    if (s0 > 0) {
      c = in ? cnt[sl] : 0;
      t = in ? th[sl] : -kInf;
      m = in ? st[sl].x : -kInf;
      load16(ka, in ? sl : 0, 0);
      if (c > 16 && c <= kTreeSliceCap) load16(kb, sl, 16);
    }
    const bool has = in && order_key(m) >= tkey;
    if (has && (c > kTreeSliceCap || order_key(t) > tkey)) {
      const int at = atomicAdd(&sh.nres, 1);
      if (at < kRescanCap) sh.res[at] = sl;
    }
    if (!has || c > kTreeSliceCap) c = 0;
    const int most = wave_max_i(c);
    if (most > 0) emit(ka, 0, c);
    if (most > 16) emit(kb, 16, c);
    for (int j0 = 32; j0 < most; j0 += 16) {
      load16(ka, in ? sl : 0, j0);
      emit(ka, j0, c);
    }
  }
  __syncthreads();
  const int nres = sh.nres;
  if (nres > 0 && nres <= kRescanCap) {  // the same in every thread: nres no longer changes (sh.n does)
    // four consecutive values per thread and slice: those >= tau that are
    // below the slice's threshold (all of them where the slots overflowed)
    constexpr int kPer = kTreeSlice / kThreads;
    for (int i = 0; i < nres; ++i) {
      const int sl = sh.res[i];
      const bool whole = cnt[sl] > kTreeSliceCap;
      const unsigned hkey = order_key(th[sl]);
      const int e0 = sl * kTreeSlice + kPer * tid;
      float v[kPer];
      if (e0 + kPer <= p.vocab) {
        if (BF16) {
          const u32x2 w = *reinterpret_cast<const u32x2_any*>(rowp + (size_t)e0 * 2);
          v[0] = as_f32(w.x << 16);
          v[1] = as_f32(w.x & 0xffff0000u);
          v[2] = as_f32(w.y << 16);
          v[3] = as_f32(w.y & 0xffff0000u);
        } else {
          const u32x4 w = *reinterpret_cast<const u32x4_any*>(rowp + (size_t)e0 * 4);
          v[0] = as_f32(w.x);
          v[1] = as_f32(w.y);
          v[2] = as_f32(w.z);
          v[3] = as_f32(w.w);
        }
      } else {
#pragma unroll
        for (int u = 0; u < kPer; ++u) v[u] = e0 + u < p.vocab ? load_one<BF16>(rowp, e0 + u) : -kInf;
      }
#pragma unroll
      for (int u = 0; u < kPer; ++u) {
        const unsigned k32 = order_key(v[u]);
        if (e0 + u < p.vocab && k32 >= tkey && (whole || k32 < hkey)) {
          const int at = atomicAdd(&sh.n, 1);
          if (at < kTreeCap) sh.cand[at] = pack(v[u], e0 + u);
        }
      }
    }
    __syncthreads();
  }
  // The K best in rank order, in the layout the enumeration reads: slot r
  // holds the token of rank r and the log q of rank r + 1 (-inf past the
  // K-th), slot 63 the log q of rank 0.
  auto write = [&](int rank, u64 key) {
    const float lq = lse == -kInf ? -kInf : key_value((unsigned)(key >> 32)) - lse;
    p.tok[(size_t)row * 64 + rank] = (int)(0xffffffffu - (unsigned)key);
    p.lq[(size_t)row * 64 + (rank == 0 ? 63 : rank - 1)] = lq;
    if (rank == p.k - 1) p.lq[(size_t)row * 64 + rank] = -kInf;
  };
  const int n = sh.n;
  if (n < p.k || n > kTreeCap || nres > kRescanCap) {
    radix_top<BF16>(p, rowp, sh);
    __syncthreads();
    if (tid < p.k) write(tid, sh.top[tid]);
    return;
  }
  // Ranking by counting: the rank of a key is the number of larger keys.
  // sh.cand is padded with zeros (below every key) to a multiple of 64 and
  // read 16 bytes at a time; up to 128 keys, two threads share a key.
  const int n64 = (n + 63) & ~63;
  for (int i = n + tid; i < n64; i += kThreads) sh.cand[i] = 0;
  __syncthreads();
  auto count_above = [&](u64 key, int i0, int i1) {
    int r = 0;
    for (int i = i0; i < i1; i += 32) {
#pragma unroll
      for (int u = 0; u < 32; u += 2) {
        const ulonglong2 w = *reinterpret_cast<const ulonglong2*>(&sh.cand[i + u]);
        r += (w.x > key ? 1 : 0) + (w.y > key ? 1 : 0);
      }
    }
    return r;
  };
  if (n <= 128) {
    const int at = tid & 127, half = tid >> 7;
    const u64 key = sh.cand[at < n ? at : 0];
    const int mine = count_above(key, half * (n64 / 2), (half + 1) * (n64 / 2));
    if (half) sh.part[at] = mine;
    __syncthreads();
    const int rank = mine + sh.part[at];
    if (!half && at < n && rank < p.k) write(rank, key);
    return;
  }
  for (int t = tid; t < n; t += kThreads) {
    const u64 key = sh.cand[t];
    const int rank = count_above(key, 0, n64);
    if (rank < p.k) write(rank, key);
  }
}

__global__ __launch_bounds__(64) void tree_enum(TreeParams p) { enumerate(p, blockIdx.x, threadIdx.x); }

}  // namespace

hipError_t launch_tree(const TreeParams& p, bool bf16, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
  const unsigned rows = (unsigned)(p.batch * p.horizon);
  const dim3 grid((unsigned)p.wgs_per_row, rows), sblock(64 * kTreeScanWaves), block(kThreads);
  if (ev0) (void)hipEventRecord(ev0, s);
  if (bf16) {
    hipLaunchKernelGGL(tree_scan<true>, grid, sblock, 0, s, p);
    hipLaunchKernelGGL(tree_rank<true>, dim3(rows), block, 0, s, p);
  } else {
    hipLaunchKernelGGL(tree_scan<false>, grid, sblock, 0, s, p);
    hipLaunchKernelGGL(tree_rank<false>, dim3(rows), block, 0, s, p);
  }
  hipLaunchKernelGGL(tree_enum, dim3((unsigned)p.batch), dim3(64), 0, s, p);
  const hipError_t e = hipGetLastError();
  if (ev1) (void)hipEventRecord(ev1, s);
  return e;
}

}  // namespace glance
