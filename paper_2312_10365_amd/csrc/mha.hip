// Sparse multi-head attention of SPT (section 4.1: Eq. 6, Algorithm 1; section 5.1: Algorithms 2
// and 3, CSR with a fixed row length) for gfx950.
//
// Codes and index lists are integer work; the attention products over the kept keys run as dense
// tiles on the matrix cores (mha_dense.hip) unless very few of many keys are kept.  For those shapes
// every query gathers its own 128/256-byte rows through its index list here: coalesced rows, LDS
// residency and the 64-lane wavefront.
//
//   pq_assign_kernel        a matrix-core product per 16 vectors and codebook, fused argmin; near ties measured exactly
//   topl_lane_kernel        Algorithm 3 bit-sliced, two or four LANES per query: inverted code table in LDS,
//                           carry-save score planes for 32 keys at a time, rows staged in LDS
//   seq_dots_kernel         one workgroup per sequence, gathered tensor resident in LDS: logits +
//                           softmax (forward) or dA + softmax Jacobian (backward)
//   seq_accum_kernel        same residency: weighted sums of gathered rows (Y, dQ through the index
//                           lists; dV, dK through the transposed lists), rows held as fp16
//   transpose_lists_kernel  one workgroup per sequence: the index lists regrouped by key, each
//                           key's entries in ascending query order (bit matrix in LDS, popcount ranks)
//   attn_row_kernel, attn_kv_kernel   the dots + accumulate pair with rows read from L2 (one
//                           wavefront per query / per key), for sequences too large for LDS; the query
//                           one also in front of the dense key side where few of more than 512 keys are kept
#include <math.h>

#include <type_traits>
#include <utility>

#include "mha_host.hpp"
#include "profile.hpp"
#include "spt_device.hpp"

namespace spt {
namespace {

constexpr int kDp = 8;          // dimensions per codeword (section 5.1)
constexpr int kMaxE = 16;       // codewords per codebook

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float dot2(uint32_t a, uint32_t b, float c) {
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, a), __builtin_bit_cast(bf16x2, b), c, false);
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
  return v;
}
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// ---------------------------------------------------------------- Algorithm 2, lines 2-3
// The nearest codeword is the one with the largest x . c - |c|^2 / 2.  For 16 vectors and the 16 codewords of a codebook that
// is three MFMAs, one per bf16 part of the fp32 codeword (x is bf16 as it comes, so every product is exact), with
// codewords as rows, vectors as columns and the accumulator starting at -|c|^2 / 2.  K holds the sub-vectors of four codebooks, as
// the lane groups load them; the codeword's part stands in its own codebook's quarter and zeros in the others.
// A score's last four bits give way to the codeword's index, so a maximum carries it along.  What is lost with them, the
// rounding of the scores and that of the distances they stand for are below kPqTie (|x|^2 + max |c|^2): 32 additions of
// 2^-23 of at most (|x|^2 + 2 |c|^2) / 2 on either side, 2^-19 of that for the index, 10 of 2^-24 of a distance of at most
// 2 (|x|^2 + |c|^2): together 2^-16.3 of |x|^2 + |c|^2.  The products, sums, squares and parts of a codeword that fall below the
// smallest normal number may be lost whole: 56 of up to 2^-126, eight of them times max(1, |x|, |c|).  kPqFloor, added to the bound,
// is 2^20 times that for |x|, |c| up to 1, and beyond 1 the bound grows faster.  A vector whose second best is nearer than the
// two -- or with anything infinite or NaN about it, which makes the test fail -- is measured again as Algorithm 2 has it: the
// distances in fp32, the lower index on a tie.  So the codes are those of the distances, bit for bit.
// us, distances measured one by one (256 instructions of the vector units per wavefront of them) -> this: S 512, n 512, E 16:
// 20.1 -> 15.9 (8 codebooks), 37.5 -> 28.4 (16); S 96, n 1100 25.0 -> 17.6; S 8, n 130 7.6 -> 5.6; S 64, n 777, E 8 7.7 -> 7.9.  What
// is left is reading X (15 us of the 28), preparing the codebooks, and the wait for both.  (One MFMA per codebook, its sub-vector in
// all lane groups: 71, bound by 20 loads of 16 lines each per 16 vectors.)
constexpr float kPqTie = 1.52587890625e-5f;   // 2^-16
constexpr float kPqFloor = 0x1p-100f;
constexpr int kPqWaves = 8, kPqVectors = 16 * kPqWaves;   // vectors of a workgroup at a time

__device__ __forceinline__ float hw_max(float a, float b) {   // (fmaxf would quiet its operands first)
  float r;
  asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ float hw_min(float a, float b) {
  float r;
  asm("v_min_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ float hw_max3(float a, float b, float c) {
  float r;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}
struct Top2 { float best, second; };
__device__ __forceinline__ Top2 merge(const Top2& a, const Top2& b) {
  return Top2{hw_max(a.best, b.best), hw_max3(hw_min(a.best, b.best), a.second, b.second)};
}
// Of two values per lane the first reduced over lanes l, l + 32 (l + 16) in the lower half (the even rows of 16 lanes), the
// second in the upper half (the odd rows).
template <bool HALVES>
__device__ __forceinline__ Top2 fold(const Top2& a, const Top2& b) {
  auto swap = [](float x, float y) {
    const uint32_t u = __float_as_uint(x), v = __float_as_uint(y);
    return HALVES ? __builtin_amdgcn_permlane32_swap(u, v, false, false) : __builtin_amdgcn_permlane16_swap(u, v, false, false);
  };
  const auto p = swap(a.best, b.best), q = swap(a.second, b.second);
  return merge(Top2{__uint_as_float(p[0]), __uint_as_float(q[0])}, Top2{__uint_as_float(p[1]), __uint_as_float(q[1])});
}
__device__ __forceinline__ float upper_half(float x) { return __uint_as_float(__float_as_uint(x) & 0xFFFF0000u); }
// f of the constants 1, 2, ...
template <class F, int... O>
__device__ __forceinline__ void each_from_one(F f, std::integer_sequence<int, O...>) {
  (f(std::integral_constant<int, O + 1>{}), ...);
}

template <int M>
__global__ __launch_bounds__(kPqWaves * 64) void pq_assign_kernel(const uint16_t* __restrict__ X,
                                                                  const float* __restrict__ C,
                                                                  uint8_t* __restrict__ codes,
                                                                  float* __restrict__ err, int n, int H, int E, int per) {
  constexpr int Q = M / 4;                       // codebooks of a lane group: Q g .. Q g + Q - 1
  __shared__ uint16_t parts[M][3][kMaxE][kDp];   // upper, next and last 8 bits of the codewords
  __shared__ uint16_t none[kDp];                 // zeros
  __shared__ float cb[M][kMaxE][kDp];
  __shared__ float norm[M][kMaxE];               // -|c|^2 / 2
  __shared__ float tie[M];                       // kPqTie max |c|^2 + kPqFloor
  const int s = blockIdx.y, head = s % H, tid = threadIdx.x, lane = tid & 63, i = lane & 15, g = lane >> 4;
  const int first = blockIdx.x * per, end = min(n, first + per);
  const size_t base = (size_t)s * n;
  int v0 = first + (tid >> 6) * 16;
  auto row = [&](int v) { return reinterpret_cast<const u32x4*>(X + (base + min(v + i, end - 1)) * (M * kDp)); };
  u32x4 x[Q];                                    // (requested before the codebooks are prepared)
#pragma unroll
  for (int p = 0; p < Q; ++p) x[p] = row(v0)[Q * g + p];
  for (int t = tid; t < M * kMaxE * kDp; t += kPqWaves * 64) {
    const int m = t / (kMaxE * kDp), e = t / kDp % kMaxE, j = t % kDp;
    const float c = e < E ? C[((size_t)head * M + m) * E * kDp + e * kDp + j] : 0.f;
    const float r = c - upper_half(c);
    cb[m][e][j] = c;
    parts[m][0][e][j] = (uint16_t)(__float_as_uint(c) >> 16);
    parts[m][1][e][j] = (uint16_t)(__float_as_uint(r) >> 16);
    parts[m][2][e][j] = (uint16_t)(__float_as_uint(r - upper_half(r)) >> 16);
  }
  if (tid < kDp) none[tid] = 0;
  if (tid < M) tie[tid] = 0.f;
  __syncthreads();
  if (tid < M * kMaxE) {
    const int m = tid / kMaxE, e = tid % kMaxE;
    float sq = 0.f;
#pragma unroll
    for (int j = 0; j < kDp; ++j) sq = fmaf(cb[m][e][j], cb[m][e][j], sq);
    // The same codeword once more can go: the lower index has it on every tie.  (A row of 16 lanes is a codebook: hashes
    // first.)
    bool again = false;
    uint32_t hash = 0u;
#pragma unroll
    for (int j = 0; j < kDp; ++j) hash = (hash ^ __float_as_uint(cb[m][e][j])) * 0x9E3779B1u;
    auto compare = [&](auto shift) {
      constexpr int o = decltype(shift)::value;
      const uint32_t other = (uint32_t)__builtin_amdgcn_update_dpp((int)~hash, (int)hash, 0x110 + o, 0xF, 0xF, false);   // lane - o
      if (other == hash) {
        bool same = true;
#pragma unroll
        for (int j = 0; j < kDp; ++j) same &= cb[m][e - o][j] == cb[m][e][j];
        again |= same;
      }
    };
    each_from_one(compare, std::make_integer_sequence<int, kMaxE - 1>{});
    norm[m][e] = e < E && !again ? -0.5f * sq : -3e38f;   // (no codeword: never near the best)
    // (non-negative: their order is that of the bits; infinite, NaN, or too large to tell: everything is near)
    atomicMax(reinterpret_cast<uint32_t*>(&tie[m]), __float_as_uint(sq < 1e38f ? kPqTie * sq + kPqFloor : INFINITY));
  }
  __syncthreads();

  float my_tie[Q];
#pragma unroll
  for (int p = 0; p < Q; ++p) my_tie[p] = tie[Q * g + p];
  for (; v0 < end; v0 += kPqVectors) {
    const u32x4* next = row(min(v0 + kPqVectors, end - 1));
    const bool real = v0 + i < end;
    const size_t at = (base + (real ? v0 + i : v0)) * M + Q * g;
    uint32_t word = 0u, again = 0u;              // this group's Q codes; a bit for each that is not decided
#pragma unroll
    for (int p = 0; p < Q; ++p) {
      const bf16x8 xb = __builtin_bit_cast(bf16x8, x[p]);
      Top2 t[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {              // codebook of group k
        const int m = Q * k + p;
        f32x4 score = *reinterpret_cast<const f32x4*>(&norm[m][4 * g]);
#pragma unroll
        for (int w = 0; w < 3; ++w) {
          const bf16x8 c = *reinterpret_cast<const bf16x8*>(g == k ? &parts[m][w][i][0] : none);
          score = __builtin_amdgcn_mfma_f32_16x16x32_bf16(c, xb, score, 0, 0, 0);
        }
        float y[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) y[r] = __uint_as_float((__float_as_uint(score[r]) & ~15u) | (uint32_t)(4 * g + r));
        t[k] = merge(Top2{hw_max(y[0], y[1]), hw_min(y[0], y[1])}, Top2{hw_max(y[2], y[3]), hw_min(y[2], y[3])});
      }
      const Top2 f = fold<false>(fold<true>(t[0], t[2]), fold<true>(t[1], t[3]));   // group k: codebook Q k + p
      float xx = my_tie[p] * (1.f / kPqTie);
#pragma unroll
      for (int w = 0; w < 4; ++w) xx = dot2(x[p][w], x[p][w], xx);
      x[p] = next[Q * g + p];
      again |= f.best - f.second > kPqTie * xx ? 0u : 1u << p;
      word |= (__float_as_uint(f.best) & 15u) << (8 * p);
    }
    if (__any(again != 0u)) {
#pragma unroll 1
      for (int m = 0; m < M; ++m) {
        const int p = m % Q, owner = m / Q;
        if (!__any(g == owner && (again >> p & 1u))) continue;
        const u32x4 xm = row(v0)[m];
        float d = INFINITY;
        int arg = 4 * g;
#pragma unroll 1
        for (int e = 4 * g; e < 4 * g + 4; ++e) {
          float dist = 0.f;
#pragma unroll
          for (int j = 0; j < kDp; ++j) {
            const float df = (j % 2 ? hi_bf16(xm[j / 2]) : lo_bf16(xm[j / 2])) - cb[m][e][j];
            dist = fmaf(df, df, dist);
          }
          if (e < E && dist < d) { d = dist; arg = e; }   // strict: ties stay with the lower index
        }
#pragma unroll
        for (int o = 16; o < 64; o <<= 1) {
          const float od = __shfl_xor(d, o);
          const int oa = __shfl_xor(arg, o);
          if (od < d || (od == d && oa < arg)) { d = od; arg = oa; }
        }
        if (g == owner && (again >> p & 1u)) word = (word & ~(255u << (8 * p))) | (uint32_t)arg << (8 * p);
      }
    }
    if (err && real) {                           // Algorithm 2, lines 4-5: the quantisation error
#pragma unroll 1
      for (int p = 0; p < Q; ++p) {
        const u32x4 xm = row(v0)[Q * g + p];
        const float* c = cb[Q * g + p][word >> (8 * p) & 15u];
        float dist = 0.f;
#pragma unroll
        for (int j = 0; j < kDp; ++j) {
          const float df = (j % 2 ? hi_bf16(xm[j / 2]) : lo_bf16(xm[j / 2])) - c[j];
          dist = fmaf(df, df, dist);
        }
        err[at + p] = sqrtf(dist < INFINITY ? dist : INFINITY);   // (NaN is no distance: none was found)
      }
    }
    typedef uint32_t u32u __attribute__((aligned(1)));
    typedef uint16_t u16u __attribute__((aligned(1)));
    if (real) {
      if (Q == 4) *reinterpret_cast<u32u*>(codes + at) = word;
      else *reinterpret_cast<u16u*>(codes + at) = (uint16_t)word;
    }
  }
}

// ---------------------------------------------------------------- Algorithm 3 with Eq. 6
// Algorithm 3, bit-sliced: a few LANES per query.  Keys arrive in index order, so bucket s holds the keys of score s in
// index order and only its first L - 1 are ever read; the output is those prefixes concatenated from score M
// down, cut at L, padded with -1.  Per sequence an inverted table is built in
// LDS, table[m][e] = the set of keys (a bit mask over key indices) whose code in codebook m is e.
// A query with codes e_1..e_M reads its M masks and adds them bit-plane-wise (a carry-save adder
// tree on 32 keys at a time), which gives the Eq. 6 score of 32 keys in a few dozen bitwise
// operations; "keys of score s" is then an AND of planes.  Pass A counts every score, pass B emits,
// for each score from M down, the set bits in index order at base[s] + rank, stopping at the
// bucket's readable length L-1 and at the row length L.  Rows are staged in LDS as 16-bit key
// indices and written out whole.  Bound by instructions of the vector units (16 codebooks, n 512: issuing in 79 % of
// the cycles), half of them in pass B's loops over set bits, which go as often as the fullest of the 64 lanes (n 1100, L 137:
// 403 turns of two keys where 69 would do were every lane equally full).
__device__ __forceinline__ void full_add(uint32_t a, uint32_t b, uint32_t c, uint32_t& sum, uint32_t& carry) {
  const uint32_t t = a ^ b;
  sum = t ^ c;
  carry = (a & b) | (c & t);
}
__device__ __forceinline__ void half_add(uint32_t a, uint32_t b, uint32_t& sum, uint32_t& carry) {
  sum = a ^ b;
  carry = a & b;
}
// Bit planes p[0..3] of the number of set bits among eight words, bit position by bit position.
__device__ __forceinline__ void count8(const uint32_t* x, uint32_t (&p)[4]) {
  uint32_t s0, c0, s1, c1, s2, c2, c3, t0, d0, d1;
  full_add(x[0], x[1], x[2], s0, c0);
  full_add(x[3], x[4], x[5], s1, c1);
  half_add(x[6], x[7], s2, c2);
  full_add(s0, s1, s2, p[0], c3);
  full_add(c0, c1, c2, t0, d0);
  half_add(t0, c3, p[1], d1);
  half_add(d0, d1, p[2], p[3]);
}
template <int M>
struct ScorePlanes {
  uint32_t hi[4], lo[4], top;    // products of the two high / two low planes; top: score 16 (M = 16)
  __device__ __forceinline__ void build(const uint32_t* x) {
    uint32_t p[4];
    count8(x, p);
    top = 0u;
    if (M == 16) {
      uint32_t q[4], k0, k1, k2, r0, r1, r2, r3;
      count8(x + 8, q);
      half_add(p[0], q[0], r0, k0);
      full_add(p[1], q[1], k0, r1, k1);
      full_add(p[2], q[2], k1, r2, k2);
      full_add(p[3], q[3], k2, r3, top);
      p[0] = r0; p[1] = r1; p[2] = r2; p[3] = r3;
    }
    const uint32_t n0 = ~p[0], n1 = ~p[1], n2 = ~p[2], n3 = ~p[3];
    lo[0] = n1 & n0; lo[1] = n1 & p[0]; lo[2] = p[1] & n0; lo[3] = p[1] & p[0];
    hi[0] = n3 & n2; hi[1] = n3 & p[2]; hi[2] = p[3] & n2; hi[3] = p[3] & p[2];
    if (M == 16) hi[0] &= ~top;      // score 16 has all four low planes clear
  }
  __device__ __forceinline__ uint32_t level(int sc) const {   // sc is a compile-time constant at every use
    return sc == 16 ? top : (hi[sc >> 2] & lo[sc & 3]);
  }
  __device__ __forceinline__ uint32_t upper() const { return hi[2] | hi[3] | top; }   // scores of 8 and more
};

// Index of the lowest set bit, ~0 without one (one instruction, where __ffs checks for zero).
__device__ __forceinline__ uint32_t lowest_bit(uint32_t x) {
  uint32_t r;
  asm("v_ffbl_b32 %0, %1" : "=v"(r) : "v"(x));
  return r;
}

// A query's keys are split over P = 2 or 4 neighbouring lanes: each takes a contiguous part of the words, and the lanes
// before it tell it where its keys of a score begin.  A wavefront then holds 64 / P queries and is done in a P-th of
// the time, and stages fewer rows: more of them run on a CU (one per SIMD waits twice as long for its own instructions
// as it issues), and a last round costs less.
// Pairs of 32-bit mask words of a part, and words per mask of the inverted table (an odd number of pairs, so that
// the 16 masks of a codebook start on different banks).
__host__ __device__ inline int topl_part_pairs(int n, int P) { return (((n + 63) >> 6) + P - 1) / P; }
__host__ __device__ inline int topl_mask_words(int n, int P) { return ((topl_part_pairs(n, P) * P) | 1) * 2; }
// Words of a staged row: L 16-bit key indices and a slot that is written and never read, to an odd number of words (the rows
// of neighbouring lanes start on different banks).
__host__ __device__ inline int topl_row_words(int L) { return ((L + 2) >> 1) | 1; }

template <int M, int P>
__global__ __launch_bounds__(1024) void topl_lane_kernel(const uint8_t* __restrict__ cq,
                                                        const uint8_t* __restrict__ ck,
                                                        int32_t* __restrict__ idx, int n, int L) {
  constexpr int QW = 64 / P;                        // queries of a wavefront
  extern __shared__ uint32_t lsm[];
  const int s = blockIdx.y;
  const int pairs = topl_part_pairs(n, P), nwp = topl_mask_words(n, P);
  uint32_t* table = lsm;                            // [M][16][nwp]
  const int lw = topl_row_words(L);
  uint32_t* stage = lsm + M * 16 * nwp;             // [waves][QW][lw], 0xFFFF = none
  const int tid = threadIdx.x, nthreads = blockDim.x;
  for (int t = tid; t < M * 8 * nwp; t += nthreads) reinterpret_cast<uint2*>(table)[t] = make_uint2(0u, 0u);
  __syncthreads();
  for (int j = tid; j < n; j += nthreads) {          // one key per thread: its M codes in one load
    uint32_t cw[M / 4];
    const uint32_t* src = reinterpret_cast<const uint32_t*>(ck + ((size_t)s * n + j) * M);
#pragma unroll
    for (int w = 0; w < M / 4; ++w) cw[w] = src[w];
#pragma unroll
    for (int m = 0; m < M; ++m) {
      const uint32_t e = (cw[m >> 2] >> (8 * (m & 3))) & 15u;
      atomicOr(table + __umul24(m * 16 + e, nwp) + (j >> 5), 1u << (j & 31));
    }
  }
  const int wave = tid >> 6, lane = tid & 63, part = lane % P;
  uint32_t* mystage = stage + (size_t)wave * QW * lw;
  for (int t = lane; t < QW * lw; t += 64) mystage[t] = 0xFFFFFFFFu;

  const int q0 = (blockIdx.x * (nthreads >> 6) + wave) * QW;   // first query of this wavefront
  const int qi = q0 + lane / P;
  const bool live = qi < n;
  int off[M];                                         // word offset of this lane's part of its query's mask in every codebook
  {
    uint32_t cw[M / 4];
    const uint32_t* qsrc = reinterpret_cast<const uint32_t*>(cq + ((size_t)s * n + (live ? qi : 0)) * M);
#pragma unroll
    for (int w = 0; w < M / 4; ++w) cw[w] = qsrc[w];
#pragma unroll
    for (int m = 0; m < M; ++m)
      off[m] = (int)__umul24(m * 16 + (cw[m >> 2] >> (8 * (m & 3)) & 15u), nwp) + part * (2 * pairs);
  }
  __syncthreads();

  // Both passes walk the masks a pair of words at a time, the next pair requested before this one is worked on.  `each`
  // gets the score planes of a word and its number in the part.  (Behind the last key a mask has zeros: score 0.)
  auto walk = [&](auto each) {
    u32x2 x[M];
#pragma unroll
    for (int m = 0; m < M; ++m) x[m] = *reinterpret_cast<const u32x2*>(table + off[m]);
    for (int p = 0; p < pairs; ++p) {
      u32x2 next[M];
      const uint32_t* from = table + 2 * (p + 1 < pairs ? p + 1 : p);
#pragma unroll
      for (int m = 0; m < M; ++m) next[m] = *reinterpret_cast<const u32x2*>(from + off[m]);
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {
        uint32_t xw[M];
#pragma unroll
        for (int m = 0; m < M; ++m) xw[m] = x[m][hf];
        ScorePlanes<M> sp;
        sp.build(xw);
        each(sp, 2 * p + hf);
      }
#pragma unroll
      for (int m = 0; m < M; ++m) x[m] = next[m];
    }
  };

  int cnt[M + 1];
#pragma unroll
  for (int b = 0; b <= M; ++b) cnt[b] = 0;
  walk([&](const ScorePlanes<M>& sp, int) {
#pragma unroll
    for (int b = 1; b < 8; ++b) cnt[b] += __popc(sp.level(b));
    if (__ballot(sp.upper() != 0u)) {                  // scores of 8 and more are rare
#pragma unroll
      for (int b = 8; b <= M; ++b) cnt[b] += __popc(sp.level(b));
    }
  });
  const int first = part * pairs * 64;                 // this part's first key
  cnt[0] = max(0, min(n - first, pairs * 64));
#pragma unroll
  for (int b = 1; b <= M; ++b) cnt[0] -= cnt[b];
  // the next slot of every bucket in this lane's row, and how many keys it still takes from this lane
  uint16_t* row = reinterpret_cast<uint16_t*>(mystage + lane / P * lw);
  int slot[M + 1], quota[M + 1];
  int acc = 0;
#pragma unroll
  for (int b = M; b >= 0; --b) {
    int before = 0, total = cnt[b];                    // keys of score b in the parts before, in all parts
#pragma unroll
    for (int o = 1; o < P; o <<= 1) {
      const int other = __shfl_xor(total, o);
      before += part & o ? other : 0;
      total += other;
    }
    const int take = max(0, min(min(total, L - 1), L - acc));   // keys this bucket contributes
    slot[b] = min(acc + before, L);
    quota[b] = live ? max(0, min(cnt[b], take - before)) : 0;
    acc += min(total, L - 1);
  }
  bool need[M + 1];                                   // does any query of this wavefront draw on bucket b
#pragma unroll
  for (int b = 0; b <= M; ++b) need[b] = __ballot(quota[b] > 0) != 0ull;
  walk([&](const ScorePlanes<M>& sp, int w) {
    const int key0 = first + w * 32;
    auto emit = [&](int b) {
      if (!need[b]) return;                            // uniform
      uint32_t bits = sp.level(b);
      if (b == 0) bits &= n - key0 >= 32 ? 0xFFFFFFFFu : n > key0 ? (1u << (n - key0)) - 1u : 0u;
      int c = min((int)__popc(bits), quota[b]);
      uint16_t* to = row + slot[b];
      quota[b] -= c;
      slot[b] += c;
      while (c > 0) {                                  // two keys a turn: the lanes go as often as the fullest of them
        const uint32_t k0 = lowest_bit(bits);
        bits &= bits - 1;
        const uint32_t k1 = lowest_bit(bits);
        bits &= bits - 1;
        to[0] = (uint16_t)(key0 + k0);
        *(c > 1 ? to + 1 : row + L) = (uint16_t)(key0 + k1);
        to += 2;
        c -= 2;
      }
    };
    if (__ballot(sp.upper() != 0u)) {
#pragma unroll
      for (int b = M; b >= 8; --b) emit(b);
    }
#pragma unroll
    for (int b = 7; b >= 0; --b) emit(b);
  });
  wave_lds_fence();
  // stage -> idx: the wavefront's rows are one contiguous run of the output, written 64 neighbouring words at a time
  const int rows = min(QW, n - q0);
  if (rows <= 0) return;
  // (keys are below 2^12, none is 0xFFFF: sign extension makes it -1.  Pieces of one key, or of two where a row holds a whole number of them.  A step is 64
  // pieces on: `down` rows and `right` pieces, and a row more where that leaves the row.  Division by L, three products of 32 bits for every key: 50 us where
  // this takes 48, S 512, n 512, 8 codebooks, L 64.)
  auto write_out = [&](auto keys) {
    constexpr int K = decltype(keys)::value;
    typedef std::conditional_t<K == 2, uint32_t, uint16_t> Staged;
    const int per = L / K, items = rows * per, down = 64 / per, right = 64 - down * per;
    const Staged* from = reinterpret_cast<const Staged*>(mystage);
    const int stride = lw * 2 / K, step = down * stride + right, wrap = stride - per;
    int col = lane % per, at = lane / per * stride + col;
    int32_t* dst = idx + ((size_t)s * n + q0) * L;
    for (int it0 = lane; it0 < items; it0 += 64 * 8) {
      uint32_t key[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        key[u] = from[it0 + u * 64 < items ? at : 0];
        col += right;
        at += step;
        const bool over = col >= per;
        at += over ? wrap : 0;
        col -= over ? per : 0;
      }
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (it0 + u * 64 < items) {
          if constexpr (K == 2) {
            typedef int i32x2u __attribute__((ext_vector_type(2), aligned(4)));
            reinterpret_cast<i32x2u*>(dst)[it0 + u * 64] = i32x2u{(int)(key[u] << 16) >> 16, (int)key[u] >> 16};
          } else {
            dst[it0 + u * 64] = (int16_t)key[u];
          }
        }
    }
  };
  if (L & 1) write_out(std::integral_constant<int, 1>{});
  else       write_out(std::integral_constant<int, 2>{});
}

// ---------------------------------------------------------------- Algorithm 1, lines 4-5 and their backward
// Row accesses are cooperative: DH/8 neighbouring lanes read one 128/256-byte row as 16-byte
// pieces, so a wavefront-wide load touches 64/(DH/8) whole cache lines instead of 64 partial ones.
// Workgroup -> (sequence, block of 4 rows).  Consecutive workgroup ids go round-robin over the 8
// XCDs, each with an L2 of its own: sequence s is pinned to XCD s % 8, so that its K, V, Q, dY rows
// and index lists are fetched into one L2 instead of all eight.
__device__ __forceinline__ bool seq_block(int blocks_per_seq, int S, int& s, int& blk) {
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  s = (slot / blocks_per_seq) * 8 + xcd;
  blk = slot % blocks_per_seq;
  return s < S;
}
inline int seq_block_grid(int blocks_per_seq, int S) { return ((S + 7) / 8) * 8 * blocks_per_seq; }

template <int DH>
struct RowMap {
  static constexpr int LPR = DH / 8;     // lanes per row
  static constexpr int G = 64 / LPR;     // rows per wavefront-wide load
};
__device__ __forceinline__ void fma8(float (&acc)[8], float w, const u32x4& row) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    acc[2 * e] = fmaf(w, lo_bf16(row[e]), acc[2 * e]);
    acc[2 * e + 1] = fmaf(w, hi_bf16(row[e]), acc[2 * e + 1]);
  }
}

// One wavefront per query row v.  With (R, G1, G2) = (Q, K, V) this is the forward pass:
//   w_l = softmax_l(scale * R[v] . G1[idx_l]),  Out[v] = sum_l w_l G2[idx_l],  A <- w.
// With (R, G1, G2) = (dY, V, K) it is the query side of the backward pass:
//   dA_l = R[v] . G1[idx_l],  w_l = A_l (dA_l - sum_m A_m dA_m) scale,  Out[v] = sum_l w_l G2[idx_l],
// and w is kept (dS) for the key side.  Entry l lives on lane l % 64 for the softmax; for the row work lane = (g, c): group g handles entry step * G + g, c is the 16-byte piece of the row.
template <int DH, int LPL, bool BWD>
__global__ __launch_bounds__(256) void attn_row_kernel(const uint16_t* __restrict__ R,
                                                       const uint16_t* __restrict__ G1,
                                                       const uint16_t* __restrict__ G2,
                                                       const int32_t* __restrict__ idx,
                                                       float* __restrict__ A, float* __restrict__ dS,
                                                       uint16_t* __restrict__ Out, int S, int n, int L,
                                                       float scale) {
  constexpr int LPR = RowMap<DH>::LPR, G = RowMap<DH>::G;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  int s, blk;
  if (!seq_block((n + 3) >> 2, S, s, blk)) return;
  const int i = blk * 4 + wave;
  if (i >= n) return;
  const size_t v = (size_t)s * n + i;
  const int g = lane / LPR, c = lane % LPR;
  const uint16_t* g1 = G1 + (size_t)s * n * DH + c * 8;
  const uint16_t* g2 = G2 + (size_t)s * n * DH + c * 8;
  const u32x4 r = *reinterpret_cast<const u32x4*>(R + v * DH + c * 8);

  int32_t jj[LPL];
  float w[LPL];
#pragma unroll
  for (int cc = 0; cc < LPL; ++cc) {
    const int l = cc * 64 + lane;
    jj[cc] = (l < L) ? idx[v * L + l] : -1;
    if ((uint32_t)jj[cc] >= (uint32_t)n) jj[cc] = -1;   // -1 = no key; anything out of range is treated alike
    w[cc] = 0.f;
    u32x4 kr[LPR];
#pragma unroll
    for (int it = 0; it < LPR; ++it) {
      if (cc * 64 + it * G < L) {      // uniform
        const int je = __shfl(jj[cc], it * G + g);
        kr[it] = *reinterpret_cast<const u32x4*>(g1 + (size_t)max(je, 0) * DH);
      }
    }
#pragma unroll
    for (int it = 0; it < LPR; ++it) {
      if (cc * 64 + it * G < L) {
        float dot = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) dot = dot2(r[e], kr[it][e], dot);
#pragma unroll
        for (int o = 1; o < LPR; o <<= 1) dot += __shfl_xor(dot, o);
        // entry l = it * G + g' sits in group g' = l % G: fetch it from that group's first lane
        const float got = __shfl(dot, (lane % G) * LPR);
        if (lane / G == it) w[cc] = got;
      }
    }
  }
  if (!BWD) {
    float mx = -INFINITY;
#pragma unroll
    for (int cc = 0; cc < LPL; ++cc) {
      w[cc] = (jj[cc] >= 0) ? w[cc] * scale : -INFINITY;
      mx = fmaxf(mx, w[cc]);
    }
    mx = wave_max(mx);
    float sum = 0.f;
#pragma unroll
    for (int cc = 0; cc < LPL; ++cc) {
      w[cc] = (jj[cc] >= 0) ? __expf(w[cc] - mx) : 0.f;
      sum += w[cc];
    }
    sum = wave_sum(sum);
    const float inv = sum > 0.f ? 1.0f / sum : 0.f;
#pragma unroll
    for (int cc = 0; cc < LPL; ++cc) {
      w[cc] *= inv;
      const int l = cc * 64 + lane;
      if (l < L) A[v * L + l] = w[cc];
    }
  } else {
    float a[LPL];
    float part = 0.f;
#pragma unroll
    for (int cc = 0; cc < LPL; ++cc) {
      const int l = cc * 64 + lane;
      a[cc] = (jj[cc] >= 0) ? A[v * L + l] : 0.f;
      part = fmaf(a[cc], w[cc], part);
    }
    const float dotsum = wave_sum(part);
#pragma unroll
    for (int cc = 0; cc < LPL; ++cc) {
      const int l = cc * 64 + lane;
      w[cc] = a[cc] * (w[cc] - dotsum) * scale;
      if (l < L) dS[v * L + l] = w[cc];
    }
  }
  // Weighted sum of the gathered rows.  (Entries without a key add zeros: the row read in their place may hold
  // infinities or NaN, which a weight of zero would not take away.)
#pragma unroll
  for (int cc = 0; cc < LPL; ++cc) {
    if (jj[cc] < 0) w[cc] = 0.f;
  }
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int cc = 0; cc < LPL; ++cc) {
#pragma unroll
    for (int i0 = 0; i0 < LPR; i0 += 4) {
      if (cc * 64 + i0 * G < L) {      // uniform; four steps' loads in flight together
        u32x4 row[4];
        float we[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          we[u] = __shfl(w[cc], (i0 + u) * G + g);
          const int je = __shfl(jj[cc], (i0 + u) * G + g);
          row[u] = *reinterpret_cast<const u32x4*>(g2 + (size_t)max(je, 0) * DH);
          if (je < 0) row[u] = u32x4{0u, 0u, 0u, 0u};
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) fma8(acc, we[u], row[u]);
      }
    }
  }
#pragma unroll
  for (int o = LPR; o < 64; o <<= 1) {
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] += __shfl_xor(acc[e], o);
  }
  if (g == 0) {
    u32x4 o4;
#pragma unroll
    for (int e = 0; e < 4; ++e) o4[e] = pack_bf16x2(acc[2 * e], acc[2 * e + 1]);
    *reinterpret_cast<u32x4*>(Out + v * DH + c * 8) = o4;
  }
}

// The index lists of one sequence, transposed: for every key j the entries (query i, slot l) that
// name it, in ascending i, as tlist[toff[j] .. toff[j+1]) = (i << 8) | l.  One workgroup per
// sequence.  The order comes from a bit matrix (bit i of row j = query i kept key j; OR-ing bits
// is order-independent): the rank of an entry inside its key's list is the number of set bits
// below i.  Fast variant (kLds): matrix, per-word prefix counts and the list under assembly all
// sit in LDS and the list is written out in order; it needs n * L <= 65536 and
// transpose_lds_bytes(n, L) of LDS.  Otherwise the matrix lives in the workspace, ranks are
// counted word by word and every entry goes straight to its place.
constexpr int kTransposeThreads = 1024;
constexpr size_t kLdsLimit = 160 * 1024;
inline size_t transpose_lds_bytes(int n, int L) {
  const size_t nwp = ((n + 31) / 32) | 1;
  return ((size_t)n + 1) * 4 + (size_t)n * nwp * 4 + ((size_t)n * nwp + 1) * 2 + (size_t)n * L * 2;
}
inline bool transpose_fits_lds(int n, int L) {
  return (size_t)n * L <= 65536 && transpose_lds_bytes(n, L) + 1024 <= kLdsLimit;   // + static scratch
}

// Exclusive scan in place over start[0..n] (n <= 4096).  Thread t owns the PER = ceil((n+1)/1024)
// consecutive values from t * PER; wavefront prefix by shuffles, wavefront totals through LDS: two
// barriers in all.  `wtot` is 16 words of LDS scratch.
__device__ __forceinline__ void block_exclusive_scan(int32_t* start, int n, int tid, int32_t* wtot) {
  const int per = (n + kTransposeThreads) / kTransposeThreads;   // ceil((n + 1) / 1024) <= 5
  const int j0 = tid * per;
  int v[5], local = 0;
#pragma unroll
  for (int e = 0; e < 5; ++e) {
    v[e] = (e < per && j0 + e <= n) ? start[j0 + e] : 0;
    local += v[e];
  }
  const int lane = tid & 63, wave = tid >> 6;
  int incl = local;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int up = __shfl_up(incl, o);
    if (lane >= o) incl += up;
  }
  if (lane == 63) wtot[wave] = incl;
  __syncthreads();
  int before = incl - local;
  for (int wv = 0; wv < wave; ++wv) before += wtot[wv];
#pragma unroll
  for (int e = 0; e < 5; ++e) {
    if (e < per && j0 + e <= n) start[j0 + e] = before;
    before += v[e];
  }
  __syncthreads();
}

template <bool kLds>
__global__ __launch_bounds__(kTransposeThreads) void transpose_lists_kernel(const int32_t* __restrict__ idx,
                                                                            int32_t* __restrict__ toff,
                                                                            uint32_t* __restrict__ tlist,
                                                                            uint32_t* __restrict__ gbits, int n,
                                                                            int L) {
  extern __shared__ uint32_t tsm[];
  __shared__ int32_t wtot[16];
  const int s = blockIdx.x;
  const int nw = (n + 31) >> 5;
  const int tid = threadIdx.x;
  int32_t* start = reinterpret_cast<int32_t*>(tsm);            // [n + 1]
  const int32_t* ix = idx + (size_t)s * n * L;
  uint32_t* tl = tlist + (size_t)s * n * L;
  if (kLds) {
    const int nwp = nw | 1;                                                // odd row stride: rows start on different banks
    uint32_t* bits = tsm + (n + 1);                                        // [n][nwp]
    uint16_t* pre = reinterpret_cast<uint16_t*>(bits + n * nwp);           // [n][nwp] set bits in earlier words
    uint16_t* staged = pre + n * nwp + (n & 1);                            // [n * L] entry numbers (kept 4-byte aligned)
    for (int t = tid; t < n * nwp; t += kTransposeThreads) bits[t] = 0u;
    __syncthreads();
    // (eight index loads in flight per thread: one at a time, each would wait out its own latency)
    for (int e0 = tid; e0 < n * L; e0 += 8 * kTransposeThreads) {
      int jv[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int e = e0 + u * kTransposeThreads;
        jv[u] = (e < n * L) ? ix[e] : -1;
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        if ((uint32_t)jv[u] < (uint32_t)n) {
          const int i = (e0 + u * kTransposeThreads) / L;
          atomicOr(bits + jv[u] * nwp + (i >> 5), 1u << (i & 31));
        }
      }
    }
    __syncthreads();
    for (int j = tid; j <= n; j += kTransposeThreads) {
      int cnt = 0;
      if (j < n)
        for (int wd = 0; wd < nw; ++wd) {
          pre[j * nwp + wd] = (uint16_t)cnt;
          cnt += __popc(bits[j * nwp + wd]);
        }
      start[j] = cnt;
    }
    __syncthreads();
    block_exclusive_scan(start, n, tid, wtot);
    for (int j = tid; j <= n; j += kTransposeThreads) toff[(size_t)s * (n + 1) + j] = start[j];
    for (int e0 = tid; e0 < n * L; e0 += 8 * kTransposeThreads) {
      int jv[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int e = e0 + u * kTransposeThreads;
        jv[u] = (e < n * L) ? ix[e] : -1;
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int j = jv[u];
        if ((uint32_t)j < (uint32_t)n) {
          const int e = e0 + u * kTransposeThreads;
          const int i = e / L;
          const int wd = j * nwp + (i >> 5);
          const int rank = pre[wd] + __popc(bits[wd] & ((1u << (i & 31)) - 1u));
          staged[start[j] + rank] = (uint16_t)e;
        }
      }
    }
    __syncthreads();
    const int total = start[n];
    for (int t = tid; t < total; t += kTransposeThreads) {
      const int e = staged[t];
      const int i = e / L;
      tl[t] = ((uint32_t)i << 8) | (uint32_t)(e - i * L);
    }
  } else {
    uint32_t* bits = gbits + (size_t)s * n * nw;
    for (int t = tid; t < n * nw; t += kTransposeThreads) bits[t] = 0u;
    __syncthreads();
    for (int e = tid; e < n * L; e += kTransposeThreads) {
      const int j = ix[e];
      if ((uint32_t)j < (uint32_t)n) {
        const int i = e / L;
        atomicOr(bits + (size_t)j * nw + (i >> 5), 1u << (i & 31));
      }
    }
    __syncthreads();
    for (int j = tid; j <= n; j += kTransposeThreads) {
      int cnt = 0;
      if (j < n)
        for (int wd = 0; wd < nw; ++wd) cnt += __popc(bits[(size_t)j * nw + wd]);
      start[j] = cnt;
    }
    __syncthreads();
    block_exclusive_scan(start, n, tid, wtot);
    for (int j = tid; j <= n; j += kTransposeThreads) toff[(size_t)s * (n + 1) + j] = start[j];
    for (int e = tid; e < n * L; e += kTransposeThreads) {
      const int j = ix[e];
      if ((uint32_t)j < (uint32_t)n) {
        const int i = e / L, l = e - i * L;
        const uint32_t* row = bits + (size_t)j * nw;
        int rank = __popc(row[i >> 5] & ((1u << (i & 31)) - 1u));
        for (int wd = 0; wd < (i >> 5); ++wd) rank += __popc(row[wd]);
        tl[start[j] + rank] = ((uint32_t)i << 8) | (uint32_t)l;
      }
    }
  }
}

// One wavefront per key j: dV[j] = sum A[i][l] dY[i], dK[j] = sum dS[i][l] Q[i] over the
// entries of the key's transposed list.  Group g of lanes takes the entries g, g + G, ... in
// order and the groups are added at the end, so the summation order is a fixed function of the
// list (no atomics).
template <int DH>
__global__ __launch_bounds__(256) void attn_kv_kernel(const uint16_t* __restrict__ Q,
                                                      const uint16_t* __restrict__ dY,
                                                      const float* __restrict__ A,
                                                      const float* __restrict__ dS,
                                                      const int32_t* __restrict__ toff,
                                                      const uint32_t* __restrict__ tlist,
                                                      uint16_t* __restrict__ dK, uint16_t* __restrict__ dV,
                                                      int S, int n, int L) {
  constexpr int LPR = RowMap<DH>::LPR, G = RowMap<DH>::G;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  int s, blk;
  if (!seq_block((n + 3) >> 2, S, s, blk)) return;
  const int j = blk * 4 + wave;
  if (j >= n) return;
  const int g = lane / LPR, c = lane % LPR;
  const int beg = toff[(size_t)s * (n + 1) + j], end = toff[(size_t)s * (n + 1) + j + 1];
  const uint32_t* tl = tlist + (size_t)s * n * L;
  const float* As = A + (size_t)s * n * L;
  const float* dSs = dS + (size_t)s * n * L;
  const uint16_t* qs = Q + (size_t)s * n * DH + c * 8;
  const uint16_t* ys = dY + (size_t)s * n * DH + c * 8;
  float av[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  float ak[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int base = beg; base < end; base += 64) {
    const int cnt = min(64, end - base);
    int qi = 0;
    float a = 0.f, ds = 0.f;
    if (lane < cnt) {
      const uint32_t p = tl[base + lane];
      qi = (int)(p >> 8);
      const size_t e = (size_t)qi * L + (p & 255u);
      a = As[e];
      ds = dSs[e];
    }
#pragma unroll
    for (int i0 = 0; i0 < LPR; i0 += 4) {
      if (i0 * G < cnt) {                // uniform; past cnt: zero weights and rows of zeros
        u32x4 yr[4], qr[4];
        float wa[4], wd[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int src = (i0 + u) * G + g;
          const int qe = __shfl(qi, src);
          wa[u] = __shfl(a, src);
          wd[u] = __shfl(ds, src);
          yr[u] = *reinterpret_cast<const u32x4*>(ys + (size_t)qe * DH);
          qr[u] = *reinterpret_cast<const u32x4*>(qs + (size_t)qe * DH);
          if (src >= cnt) yr[u] = qr[u] = u32x4{0u, 0u, 0u, 0u};
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          fma8(av, wa[u], yr[u]);
          fma8(ak, wd[u], qr[u]);
        }
      }
    }
  }
#pragma unroll
  for (int o = LPR; o < 64; o <<= 1) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      av[e] += __shfl_xor(av[e], o);
      ak[e] += __shfl_xor(ak[e], o);
    }
  }
  if (g == 0) {
    const size_t krow = (size_t)s * n + j;
    u32x4 ov, ok;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      ov[e] = pack_bf16x2(av[2 * e], av[2 * e + 1]);
      ok[e] = pack_bf16x2(ak[2 * e], ak[2 * e + 1]);
    }
    *reinterpret_cast<u32x4*>(dV + krow * DH + c * 8) = ov;
    *reinterpret_cast<u32x4*>(dK + krow * DH + c * 8) = ok;
  }
}

// ---------------------------------------------------------------- sequence-resident variants
// When one tensor of a sequence fits LDS (n * dh <= 65536 elements) a workgroup of 16 wavefronts
// takes a whole sequence: it copies the rows that will be gathered (K, V, Q or dY of that
// sequence) into LDS once, with a stride of dh*2 + 16 bytes so that rows start on different
// banks, and every gather after that is an LDS read.  The work splits into a "dots" kernel
// (logits / dA, then the softmax or its Jacobian) and an "accumulate" kernel (weighted row sums),
// each with its own tensor resident.
constexpr int kSeqThreads = 1024;
constexpr int kSeqWaves = kSeqThreads / 64;
template <int DH>
struct SeqTile {
  static constexpr int STRIDE = DH * 2 + 16;   // bytes between rows in LDS
};
inline bool seq_resident(int n, int dh) { return (size_t)n * dh <= 65536; }
inline size_t seq_lds_bytes(int n, int dh) { return (size_t)n * (dh * 2 + 16); }

template <int DH>
__device__ __forceinline__ void stage_rows(const uint16_t* __restrict__ src, uint8_t* smem, int n) {
  constexpr int NC = DH / 8;
  const u32x4* g = reinterpret_cast<const u32x4*>(src);
  for (int q0 = threadIdx.x; q0 < n * NC; q0 += 4 * kSeqThreads) {   // four loads in flight per thread
    u32x4 x[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int q = q0 + u * kSeqThreads;
      if (q < n * NC) x[u] = g[q];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int q = q0 + u * kSeqThreads;
      if (q < n * NC) {
        const int row = q / NC, c = q - row * NC;
        *reinterpret_cast<u32x4*>(smem + row * SeqTile<DH>::STRIDE + c * 16) = x[u];
      }
    }
  }
}

// The accumulate kernel multiplies every gathered element once, so the rows are staged as fp16:
// v_fma_mix_f32 then takes them straight from their 16-bit halves, where bf16 would need a shift or
// mask per element first.  The rows are divided by a power of two >= the largest magnitude of the
// sequence beforehand (exact), which puts every value within 2^-14 of that maximum exactly on an
// fp16 number (fp16 has 3 more mantissa bits than bf16) and rounds smaller ones to multiples of
// 2^-24 of the scale: an absolute error below 6e-8 of the largest element.  Returns the scale.
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
template <int DH>
__device__ __forceinline__ float stage_rows_f16(const uint16_t* __restrict__ src, uint8_t* smem, int n,
                                                uint32_t* red /* [kSeqWaves + 1] words of LDS */) {
  constexpr int NC = DH / 8;
  const u32x4* gsrc = reinterpret_cast<const u32x4*>(src);
  uint32_t mag = 0u;                       // largest |x| as a bf16 bit pattern (monotonic in |x|)
  for (int q0 = threadIdx.x; q0 < n * NC; q0 += 4 * kSeqThreads) {   // four loads in flight per thread
    u32x4 xv[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int q = q0 + u * kSeqThreads;
      xv[u] = (q < n * NC) ? gsrc[q] : u32x4{0u, 0u, 0u, 0u};
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int q = q0 + u * kSeqThreads;
      if (q < n * NC) {
        const int row = q / NC, c = q - row * NC;
        *reinterpret_cast<u32x4*>(smem + row * SeqTile<DH>::STRIDE + c * 16) = xv[u];
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        mag = max(mag, xv[u][e] & 0x7FFFu);
        mag = max(mag, (xv[u][e] >> 16) & 0x7FFFu);
      }
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) mag = max(mag, (uint32_t)__shfl_xor((int)mag, o));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mag;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t m = 0u;
    for (int wv = 0; wv < kSeqWaves; ++wv) m = max(m, red[wv]);
    red[kSeqWaves] = m;
  }
  __syncthreads();
  const int expo = (int)(red[kSeqWaves] >> 7);          // biased exponent of the largest magnitude
  const float down = expo ? ldexpf(1.0f, 126 - expo) : 1.0f;   // 1 / 2^(expo - 126): |x| * down < 1
  const float up = expo ? ldexpf(1.0f, expo - 126) : 1.0f;
  for (int q = threadIdx.x; q < n * NC; q += kSeqThreads) {
    const int row = q / NC, c = q - row * NC;
    u32x4* slot = reinterpret_cast<u32x4*>(smem + row * SeqTile<DH>::STRIDE + c * 16);
    const u32x4 x = *slot;
    f16x8 h;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      h[2 * e] = (_Float16)(lo_bf16(x[e]) * down);
      h[2 * e + 1] = (_Float16)(hi_bf16(x[e]) * down);
    }
    *slot = __builtin_bit_cast(u32x4, h);
  }
  __syncthreads();
  return up;
}
__device__ __forceinline__ void fma8h(float (&acc)[8], float w, const u32x4& row) {
  const f16x8 h = __builtin_bit_cast(f16x8, row);
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = fmaf((float)h[e], w, acc[e]);
}

// Sum over the DH/8 lanes that share a row, with DPP only (quads, then half rows, then rows).
template <int CTRL>
__device__ __forceinline__ float dpp_move(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, false));
}
template <int LPR>
__device__ __forceinline__ float group_sum(float x) {
  x += dpp_move<0xB1>(x);      // quad_perm [1,0,3,2]
  x += dpp_move<0x4E>(x);      // quad_perm [2,3,0,1]
  x += dpp_move<0x141>(x);     // row_half_mirror: lane k of 8 reads lane 7-k
  if (LPR == 16) x += dpp_move<0x140>(x);   // row_mirror: lane k of 16 reads lane 15-k
  return x;
}
// Whole-wavefront reductions without LDS traffic: DPP inside a row of 16 lanes, then the
// gfx950 row / half swaps (v_permlane16_swap exchanges the odd rows of its first operand with the
// even rows of its second; with the same value in both, first + second is the xor-16 butterfly;
// v_permlane32_swap does the same with the two halves).
struct OpAdd { __device__ static float f(float a, float b) { return a + b; } };
struct OpMax { __device__ static float f(float a, float b) { return fmaxf(a, b); } };
template <class Op>
__device__ __forceinline__ float swap16(float x) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return Op::f(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
template <class Op>
__device__ __forceinline__ float swap32(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return Op::f(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
template <class Op>
__device__ __forceinline__ float wave_all(float x) {
  x = Op::f(x, dpp_move<0xB1>(x));
  x = Op::f(x, dpp_move<0x4E>(x));
  x = Op::f(x, dpp_move<0x141>(x));
  x = Op::f(x, dpp_move<0x140>(x));
  x = swap16<Op>(x);
  return swap32<Op>(x);
}
// Two values reduced for the price of one: after the row swap, first + second holds the xor-16
// sums of `a` in the even rows and those of `b` in the odd rows (likewise for the halves).
__device__ __forceinline__ float pair16(float a, float b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float pair32(float a, float b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// "Dots": G1 rows of the sequence resident.  Forward: A = softmax(scale * R . G1[idx]).  Backward:
// dS = A (dA - sum A dA) scale with dA = R . G1[idx] (R = dY, G1 = V).  Lane (g, c) OWNS entry
// c * G + g of every block of 64 entries (it loads that entry's index and A value and stores its
// result); in step `it` the DH/8 lanes of group g work together on the entry owned by the group's
// lane `it`, and that lane keeps the dot product.  The softmax then needs one exp per lane.
template <int DH, int LPL, bool BWD>
__global__ __launch_bounds__(kSeqThreads) void seq_dots_kernel(const uint16_t* __restrict__ R,
                                                               const uint16_t* __restrict__ G1,
                                                               const int32_t* __restrict__ idx,
                                                               const float* __restrict__ Ain,
                                                               float* __restrict__ Wout, int n, int L,
                                                               float scale) {
  constexpr int LPR = RowMap<DH>::LPR, G = RowMap<DH>::G, STRIDE = SeqTile<DH>::STRIDE;
  extern __shared__ uint8_t seq_smem[];
  const int s = blockIdx.x;
  stage_rows<DH>(G1 + (size_t)s * n * DH, seq_smem, n);
  __syncthreads();
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int g = lane / LPR, c = lane % LPR;
  const int own = c * G + g;             // the entry (inside a block of 64) this lane owns
  const uint32_t mine = c * 16;          // byte offset of this lane's piece inside an LDS row
  // One query ahead: the next query's row piece, index list and A values are requested before the
  // current query's arithmetic, so their latency is hidden behind it.
  u32x4 r_next = {0u, 0u, 0u, 0u};
  int jl_next[LPL];
  float al_next[LPL];
  auto request = [&](int i) {
    const size_t v = (size_t)s * n + i;
    r_next = *reinterpret_cast<const u32x4*>(R + v * DH + c * 8);
#pragma unroll
    for (int cc = 0; cc < LPL; ++cc) {
      const int l = cc * 64 + own;
      jl_next[cc] = (l < L) ? idx[v * L + l] : -1;
      al_next[cc] = 0.f;
      if (BWD) al_next[cc] = (l < L) ? Ain[v * L + l] : 0.f;
    }
  };
  if (wave < n) request(wave);
  for (int i = wave; i < n; i += kSeqWaves) {
    const size_t v = (size_t)s * n + i;
    const u32x4 r = r_next;
    int jl[LPL];
    float al[LPL];
#pragma unroll
    for (int cc = 0; cc < LPL; ++cc) { jl[cc] = jl_next[cc]; al[cc] = al_next[cc]; }
    if (i + kSeqWaves < n) request(i + kSeqWaves);
    float w[LPL];
    bool ok[LPL];
#pragma unroll
    for (int cc = 0; cc < LPL; ++cc) {
      ok[cc] = (uint32_t)jl[cc] < (uint32_t)n;     // -1 = no key; anything out of range alike
      const int jrow = ok[cc] ? jl[cc] : 0;
      w[cc] = 0.f;
      // Four steps under one uniform test: no branch between their shuffles and LDS reads.
#pragma unroll
      for (int i0 = 0; i0 < LPR; i0 += 4) {
        if (cc * 64 + i0 * G < L) {
          u32x4 kr[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int je = __shfl(jrow, g * LPR + i0 + u);
            kr[u] = *reinterpret_cast<const u32x4*>(&seq_smem[mine + __umul24((uint32_t)je, (uint32_t)STRIDE)]);
          }
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            float dot = 0.f;
#pragma unroll
            for (int e = 0; e < 4; ++e) dot = dot2(r[e], kr[u][e], dot);
            dot = group_sum<LPR>(dot);
            w[cc] = (c == i0 + u) ? dot : w[cc];
          }
        }
      }
    }
    if (!BWD) {
      float mx = -INFINITY;
#pragma unroll
      for (int cc = 0; cc < LPL; ++cc) {
        w[cc] = ok[cc] ? w[cc] * scale : -INFINITY;
        mx = fmaxf(mx, w[cc]);
      }
      mx = wave_all<OpMax>(mx);
      float sum = 0.f;
#pragma unroll
      for (int cc = 0; cc < LPL; ++cc) {
        w[cc] = ok[cc] ? __expf(w[cc] - mx) : 0.f;
        sum += w[cc];
      }
      sum = wave_all<OpAdd>(sum);
      const float inv = sum > 0.f ? 1.0f / sum : 0.f;
#pragma unroll
      for (int cc = 0; cc < LPL; ++cc) w[cc] *= inv;
    } else {
      float part = 0.f;
#pragma unroll
      for (int cc = 0; cc < LPL; ++cc) {
        al[cc] = ok[cc] ? al[cc] : 0.f;
        part = fmaf(al[cc], w[cc], part);
      }
      const float dotsum = wave_all<OpAdd>(part);
#pragma unroll
      for (int cc = 0; cc < LPL; ++cc) w[cc] = al[cc] * (w[cc] - dotsum) * scale;
    }
#pragma unroll
    for (int cc = 0; cc < LPL; ++cc) {
      const int l = cc * 64 + own;
      if (l < L) Wout[v * L + l] = w[cc];
    }
  }
}

// "Accumulate": the rows to be summed (G2) resident.  Out[row] = sum over the row's entries of
// weight * G2[column].  kKeys = false: output rows are queries, entries idx[v][0..L) with weights
// W[v][l].  kKeys = true: output rows are keys, entries the key's transposed list, (i << 8) | l,
// with weights W[i][l].
template <int DH, bool kKeys>
__global__ __launch_bounds__(kSeqThreads) void seq_accum_kernel(const uint16_t* __restrict__ G2,
                                                                const int32_t* __restrict__ idx,
                                                                const int32_t* __restrict__ toff,
                                                                const uint32_t* __restrict__ tlist,
                                                                const float* __restrict__ W,
                                                                uint16_t* __restrict__ Out, int n, int L,
                                                                int S, int parts) {
  constexpr int LPR = RowMap<DH>::LPR, G = RowMap<DH>::G, STRIDE = SeqTile<DH>::STRIDE;
  extern __shared__ uint8_t seq_smem[];
  // `parts` workgroups share a sequence's output rows (row = part, part + parts, ... in steps of the
  // wavefronts) and run on one XCD (workgroup id mod 8) side by side.
  const int xcd = blockIdx.x & 7, jj = blockIdx.x >> 3;
  const int part = jj % parts, s = (jj / parts) * 8 + xcd;
  if (s >= S) return;
  const float up = stage_rows_f16<DH>(G2 + (size_t)s * n * DH, seq_smem, n,
                                      reinterpret_cast<uint32_t*>(seq_smem + (size_t)n * STRIDE));
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int g = lane / LPR, c = lane % LPR;
  const uint32_t mine = c * 16;          // byte offset of this lane's piece inside an LDS row
  const float* Ws = W + (size_t)s * n * L;
  auto bounds = [&](int row, int& beg, int& end) {
    if (kKeys) {
      beg = toff[(size_t)s * (n + 1) + row];
      end = toff[(size_t)s * (n + 1) + row + 1];
    } else {
      beg = row * L;
      end = beg + L;
    }
  };
  // Entry `base + lane` of the current list: its column and weight (0, 0 past the end).
  auto fetch = [&](int base, int end, int& col, float& wt) {
    col = 0;
    wt = 0.f;
    if (base + lane < end) {
      if (kKeys) {
        const uint32_t p = tlist[(size_t)s * n * L + base + lane];
        col = (int)(p >> 8);
        wt = Ws[(size_t)col * L + (p & 255u)];
      } else {
        col = idx[(size_t)s * n * L + base + lane];
        wt = Ws[base + lane];
        if ((uint32_t)col >= (uint32_t)n) { col = 0; wt = 0.f; }
      }
    }
  };
  // Rows wave, wave + 16, ...; each row's list in chunks of 64 entries.  The chunk after the
  // current one (of this row or the next) is requested before the current one is consumed.
  int row = part * kSeqWaves + wave, beg = 0, end = 0;
  if (row < n) bounds(row, beg, end);
  int base = beg, pcol;
  float pwt;
  fetch(base, end, pcol, pwt);
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  while (row < n) {
    const int col = pcol;
    const float wt = pwt;
    const int cnt = min(64, end - base);
    const bool last = base + 64 >= end;
    int nrow = row, nbase = base + 64, nbeg = beg, nend = end;
    if (last) {
      nrow = row + kSeqWaves * parts;
      nbeg = nend = 0;
      if (nrow < n) bounds(nrow, nbeg, nend);
      nbase = nbeg;
    }
    fetch(nbase, nend, pcol, pwt);
    // A few steps at a time under one uniform test: inside a group nothing branches, so the
    // shuffles and the LDS reads are all in flight before the first multiply.  Lanes past cnt carry
    // weight 0 and column 0.  Index lists are full chunks (groups of 4); the key side's lists end
    // anywhere, so it tests every 2 steps and wastes less on the tail.
    constexpr int GS = kKeys ? 2 : 4;
#pragma unroll
    for (int i0 = 0; i0 < LPR; i0 += GS) {
      if (i0 * G < cnt) {
        u32x4 rowv[GS];
        float we[GS];
#pragma unroll
        for (int u = 0; u < GS; ++u) {
          const int ce = __shfl(col, (i0 + u) * G + g);
          we[u] = __shfl(wt, (i0 + u) * G + g);
          rowv[u] = *reinterpret_cast<const u32x4*>(&seq_smem[mine + __umul24((uint32_t)ce, (uint32_t)STRIDE)]);
        }
#pragma unroll
        for (int u = 0; u < GS; ++u) fma8h(acc, we[u], rowv[u]);
      }
    }
    if (last) {
      // Sum the 8 accumulators over the groups, reduce-scatter fashion: row r (16 lanes) ends up
      // with the totals of channels 2r and 2r + 1 of its lanes' pieces.
      float even = pair32(pair16(acc[0], acc[2]), pair16(acc[4], acc[6]));
      float odd = pair32(pair16(acc[1], acc[3]), pair16(acc[5], acc[7]));
      if (LPR == 8) {                      // two groups share a row: add the other one (lane ^ 8)
        even += dpp_move<0x128>(even);
        odd += dpp_move<0x128>(odd);
      }
      const int r = lane >> 4, pc = lane & 15;
      if (pc < LPR)
        *reinterpret_cast<uint32_t*>(Out + ((size_t)s * n + row) * DH + pc * 8 + 2 * r) =
            pack_bf16x2(even * up, odd * up);
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] = 0.f;
    }
    row = nrow; base = nbase; beg = nbeg; end = nend;
  }
}

// ---------------------------------------------------------------- host side
// Dense tiles on the matrix cores (mha_dense.hip) cost n multiply-adds per query and channel where
// the gathering kernels here cost L.  Measured, forward + backward without the codes and lists, us:
//   S 512, n 512, dh 64    L 8: 345 gathering, 316 dense   L 32: 405, 318   L 64: 642, 343
//   S 512, n 512, dh 128   L 8: 512, 560                   L 32: 720, 569
//   S 128, n 2048, dh 64   L 32: 2348, 701                 L 64: 4385, 923
// (the lists regrouped by key are what the long sequences pay for; at n 2048 only the key side is
// dense on the right).  128-wide heads need the line between L 8 and L 32 at 512 keys; for 64-wide
// heads and for long sequences dense tiles win below the line too.  Dense tiles load list entries
// four at a time, so they want L >= 4.
bool use_dense(const spt_mha_shape_t& s) { return s.L >= 4 && s.n <= 32 * s.L; }

// The query side of dense shapes (forward, dQ).  Up to 512 keys are one pass of the tile kernel.  Longer sequences go
// through it in chunks, and where few keys are kept gathering the rows from L2 is faster; the line is where the two
// met, L about (dh 64) 80, 100, 115, 192, 256 and (dh 128) 80, 87, 103, 130, 170 at n 520, 768, 1024, 1536, 2048.
// us, forward, dense and gathering: n 2048, dh 64, L 64: 309, 152; n 1024, dh 128, L 64: 221, 138; L 128: 220, 273.
constexpr int kDenseRowsKeys = 512;
bool use_dense_rows(const spt_mha_shape_t& s) {
  if (!use_dense(s)) return false;
  return s.n <= kDenseRowsKeys || (s.dh == 64 ? s.L > 64 + s.n * s.n / 22000 : s.L > 50 + s.n / 17);
}
// Gathering query side: out of LDS up to the same length, from L2 beyond.
bool rows_in_lds(const spt_mha_shape_t& s) { return s.n <= kDenseRowsKeys; }

struct MhaWorkspace {
  float* dS;          // [S][n][L]
  int32_t* toff;      // [S][n + 1]
  uint32_t* tlist;    // [S][n * L]
  uint32_t* gbits;    // [S][n][ceil(n/32)] when the transposition does not fit LDS, else null
  size_t bytes;
};

int check_mha(const spt_mha_shape_t* p) {
  if (!p) return SPT_ERR_ARG;
  if (p->S < 1 || p->H < 1 || p->n < 1 || p->dh < 1 || p->M < 1 || p->E < 1 || p->L < 1) return SPT_ERR_ARG;
  if (p->S % p->H != 0 || p->L > p->n || !isfinite(p->scale)) return SPT_ERR_ARG;
  if (p->dh != 64 && p->dh != 128) return SPT_ERR_UNSUPPORTED;
  if (p->M * kDp != p->dh || p->E > kMaxE || p->L > 256 || p->n > 4096 || p->S > 65535) return SPT_ERR_UNSUPPORTED;
  return SPT_OK;
}

MhaWorkspace plan_mha(const spt_mha_shape_t& s, void* ws) {
  MhaWorkspace w;
  char* p = static_cast<char*>(ws);
  size_t off = 0;
  const size_t rows = (size_t)s.S * s.n;
  w.dS = reinterpret_cast<float*>(p + off);        off += align256(rows * s.L * sizeof(float));
  w.gbits = nullptr;
  w.toff = reinterpret_cast<int32_t*>(p + off);    off += align256((size_t)s.S * (s.n + 1) * sizeof(int32_t));
  w.tlist = reinterpret_cast<uint32_t*>(p + off);  off += align256(rows * s.L * sizeof(uint32_t));
  // (the dense tiles need no transposition and leave its lists unused)
  if (!use_dense(s) && !transpose_fits_lds(s.n, s.L)) {
    w.gbits = reinterpret_cast<uint32_t*>(p + off);
    off += align256(rows * ((s.n + 31) / 32) * sizeof(uint32_t));
  }
  w.bytes = off;
  return w;
}

bool aligned16(const void* p) { return p && (reinterpret_cast<uintptr_t>(p) & 15) == 0; }
bool aligned4(const void* p) { return p && (reinterpret_cast<uintptr_t>(p) & 3) == 0; }

template <int DH, bool BWD>
void launch_row(const spt_mha_shape_t& s, const uint16_t* R, const uint16_t* G1, const uint16_t* G2,
                const int32_t* idx, float* A, float* dS, uint16_t* Out, hipStream_t st) {
  const dim3 grid(seq_block_grid((s.n + 3) / 4, s.S));
  const int lpl = (s.L + 63) / 64;
#define SPT_ROW(LPL_) \
  hipLaunchKernelGGL((attn_row_kernel<DH, LPL_, BWD>), grid, dim3(256), 0, st, R, G1, G2, idx, A, dS, Out, s.S, s.n, \
                     s.L, s.scale)
  switch (lpl) {
    case 1: SPT_ROW(1); break;
    case 2: SPT_ROW(2); break;
    case 3: SPT_ROW(3); break;
    default: SPT_ROW(4); break;
  }
#undef SPT_ROW
}

// Lanes per query and wavefronts per workgroup of topl_lane_kernel (at least (4, 1) fits LDS for every shape the library takes).
// The wavefronts of a workgroup share a table.  Time of the launch, in pairs of mask words walked by a
// wavefront that has a SIMD for itself: rounds of workgroups x (the pairs of a part, two more for what a wavefront does
// once, times the wavefronts that share a SIMD; and 8 for every key a lane puts into the table).  us, one box, the kernel
// with a query per lane before -> now: S 512, n 512, 8 codebooks, L 64: 56 -> 51; 16 codebooks 98 -> 80; S 96, n 1100,
// L 137: 189 -> 94; S 32, n 2048, L 128: 145 -> 66; S 8, n 130: 17.6 -> 7.3.  Over nine shapes and every count that fits the
// rule's choice is at most 8 % behind the best.
struct TopLPlan { int parts, waves; size_t lds; };
TopLPlan plan_topl(const spt_mha_shape_t& s) {
  TopLPlan best = {0, 0, 0};
  double least = 0.0;
  for (int P = 2; P <= 4; P *= 2) {
    const int rows = 64 / P;
    const size_t table = (size_t)s.M * 16 * topl_mask_words(s.n, P) * 4, stage = (size_t)rows * topl_row_words(s.L) * 4;
    for (int w = 16; w >= 1; --w) {
      if (table + w * stage > kLdsLimit || (w > 1 && (w - 1) * rows >= s.n)) continue;   // (no idle wavefronts)
      const int by_lds = (int)(kLdsLimit / (table + w * stage)), by_regs = (s.M == 16 ? 16 : 24) / w;
      const int64_t per_cu = by_lds < by_regs ? by_lds : by_regs;                        // workgroups
      const int64_t groups = (int64_t)s.S * ((s.n + w * rows - 1) / (w * rows));
      auto round = [&](int64_t g) {
        return (topl_part_pairs(s.n, P) + 2.0) * (double)((g * w + 3) / 4) + 8.0 * s.n / (64.0 * w);
      };
      const int64_t full = groups / (256 * per_cu), rest = groups % (256 * per_cu);
      const double cost = (double)full * round(per_cu) + (rest ? round((rest + 255) / 256) : 0.0);
      if (best.waves == 0 || cost < least) { least = cost; best = {P, w, table + w * stage}; }
    }
  }
  return best;
}

template <int M, int P>
hipError_t launch_topl(const spt_mha_shape_t& s, const TopLPlan& plan, const uint8_t* cq, const uint8_t* ck, int32_t* idx,
                       hipStream_t st) {
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(topl_lane_kernel<M, P>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsLimit);
  if (e != hipSuccess) return e;
  const int rows = plan.waves * (64 / P);
  topl_lane_kernel<M, P><<<dim3((s.n + rows - 1) / rows, s.S), plan.waves * 64, plan.lds, st>>>(cq, ck, idx, s.n, s.L);
  return hipGetLastError();
}

template <int DH, bool BWD>
void launch_seq_dots(const spt_mha_shape_t& s, const uint16_t* R, const uint16_t* G1, const int32_t* idx,
                     const float* Ain, float* Wout, hipStream_t st) {
  const size_t lds = seq_lds_bytes(s.n, DH);
  static_assert(kDenseRowsKeys <= 32 * 64, "lists longer than 64 entries take the dense tiles");
  (void)hipFuncSetAttribute(reinterpret_cast<const void*>(seq_dots_kernel<DH, 1, BWD>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  hipLaunchKernelGGL((seq_dots_kernel<DH, 1, BWD>), dim3(s.S), dim3(kSeqThreads), lds, st, R, G1, idx, Ain, Wout, s.n,
                     s.L, s.scale);
}

template <int DH, bool kKeys>
void launch_seq_accum(const spt_mha_shape_t& s, const uint16_t* G2, const int32_t* idx, const int32_t* toff,
                      const uint32_t* tlist, const float* W, uint16_t* Out, hipStream_t st) {
  const size_t lds = seq_lds_bytes(s.n, DH) + (kSeqWaves + 1) * sizeof(uint32_t);
  (void)hipFuncSetAttribute(reinterpret_cast<const void*>(seq_accum_kernel<DH, kKeys>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  // Key side, 64-wide heads: two workgroups per sequence.  The weights W[i][l] are gathered 4 bytes at
  // a time out of 2 x 128 KiB per sequence; with 32 sequences resident per XCD that is twice its L2,
  // with 16 it fits (measured 0.285 -> 0.262 ms on the OPT-2048 shape; four parts, or two with
  // 128-wide heads, whose rows take twice as long to stage, cost more than they save).
  const int parts = (kKeys && DH == 64 && s.n >= 2 * kSeqWaves) ? 2 : 1;
  hipLaunchKernelGGL((seq_accum_kernel<DH, kKeys>), dim3(8 * parts * ((s.S + 7) / 8)), dim3(kSeqThreads), lds, st,
                     G2, idx, toff, tlist, W, Out, s.n, s.L, s.S, parts);
}

}  // namespace
}  // namespace spt

using namespace spt;

extern "C" {

size_t spt_mha_workspace_bytes(const spt_mha_shape_t* shape) {
  if (check_mha(shape) != SPT_OK) return 0;
  return plan_mha(*shape, nullptr).bytes;
}

int spt_mha_pq_assign(const spt_mha_shape_t* shape, const void* X, const float* C, uint8_t* codes,
                      float* err, void* stream) {
  const int rc = check_mha(shape);
  if (rc != SPT_OK) return rc;
  if (!aligned16(X) || !aligned4(C) || !codes || (err && !aligned4(err))) return SPT_ERR_ARG;
  hipStream_t st = static_cast<hipStream_t>(stream);
  // 512 vectors per workgroup, for what it prepares once; fewer where that would be less than two workgroups per CU.
  int groups = (shape->n + 511) / 512;
  while ((int64_t)groups * shape->S < 512 && groups * kPqVectors < shape->n) ++groups;
  const int per = ((shape->n + groups - 1) / groups + kPqVectors - 1) / kPqVectors * kPqVectors;
  const dim3 grid((shape->n + per - 1) / per, shape->S);
  {
    ScopedKernelTimer tm(kSlotMhaPq, st);
    if (shape->M == 8)
      hipLaunchKernelGGL(pq_assign_kernel<8>, grid, dim3(kPqWaves * 64), 0, st, static_cast<const uint16_t*>(X), C, codes,
                         err, shape->n, shape->H, shape->E, per);
    else
      hipLaunchKernelGGL(pq_assign_kernel<16>, grid, dim3(kPqWaves * 64), 0, st, static_cast<const uint16_t*>(X), C, codes,
                         err, shape->n, shape->H, shape->E, per);
  }
  return hipGetLastError() == hipSuccess ? SPT_OK : SPT_ERR_HIP;
}

int spt_mha_topl(const spt_mha_shape_t* shape, const uint8_t* cq, const uint8_t* ck, int32_t* idx,
                 void* stream) {
  const int rc = check_mha(shape);
  if (rc != SPT_OK) return rc;
  if (!cq || !ck || ((reinterpret_cast<uintptr_t>(cq) | reinterpret_cast<uintptr_t>(ck)) & 7) || !aligned4(idx))
    return SPT_ERR_ARG;
  hipStream_t st = static_cast<hipStream_t>(stream);
  ScopedKernelTimer tm(kSlotMhaTopl, st);
  const TopLPlan plan = plan_topl(*shape);
#define SPT_TOPL(M, P) launch_topl<M, P>(*shape, plan, cq, ck, idx, st)
  const hipError_t e = shape->M == 8 ? (plan.parts == 2 ? SPT_TOPL(8, 2) : SPT_TOPL(8, 4))
                                     : (plan.parts == 2 ? SPT_TOPL(16, 2) : SPT_TOPL(16, 4));
#undef SPT_TOPL
  return e == hipSuccess ? SPT_OK : SPT_ERR_HIP;
}

int spt_mha_attn_fwd(const spt_mha_shape_t* shape, const void* Q, const void* K, const void* V,
                     const int32_t* idx, float* A, void* Y, void* stream) {
  const int rc = check_mha(shape);
  if (rc != SPT_OK) return rc;
  if (!aligned16(Q) || !aligned16(K) || !aligned16(V) || !aligned4(idx) || !aligned4(A) || !aligned16(Y))
    return SPT_ERR_ARG;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const uint16_t* q = static_cast<const uint16_t*>(Q);
  const uint16_t* k = static_cast<const uint16_t*>(K);
  const uint16_t* v = static_cast<const uint16_t*>(V);
  {
    ScopedKernelTimer tm(kSlotMhaFwd, st);
    uint16_t* y = static_cast<uint16_t*>(Y);
    if (use_dense_rows(*shape)) return mha_dense_fwd(*shape, Q, K, V, idx, A, Y, st) == hipSuccess ? SPT_OK : SPT_ERR_HIP;
    if (rows_in_lds(*shape)) {
      if (shape->dh == 64) {
        launch_seq_dots<64, false>(*shape, q, k, idx, nullptr, A, st);
        launch_seq_accum<64, false>(*shape, v, idx, nullptr, nullptr, A, y, st);
      } else {
        launch_seq_dots<128, false>(*shape, q, k, idx, nullptr, A, st);
        launch_seq_accum<128, false>(*shape, v, idx, nullptr, nullptr, A, y, st);
      }
    } else if (shape->dh == 64) {
      launch_row<64, false>(*shape, q, k, v, idx, A, nullptr, y, st);
    } else {
      launch_row<128, false>(*shape, q, k, v, idx, A, nullptr, y, st);
    }
  }
  return hipGetLastError() == hipSuccess ? SPT_OK : SPT_ERR_HIP;
}

int spt_mha_attn_bwd(const spt_mha_shape_t* shape, const void* Q, const void* K, const void* V,
                     const void* dY, const int32_t* idx, const float* A, void* dQ, void* dK, void* dV,
                     void* ws, size_t ws_bytes, void* stream) {
  const int rc = check_mha(shape);
  if (rc != SPT_OK) return rc;
  if (!aligned16(Q) || !aligned16(K) || !aligned16(V) || !aligned16(dY) || !aligned4(idx) || !aligned4(A) ||
      !aligned16(dQ) || !aligned16(dK) || !aligned16(dV) || !ws || (reinterpret_cast<uintptr_t>(ws) & 255))
    return SPT_ERR_ARG;
  const MhaWorkspace w = plan_mha(*shape, ws);
  if (ws_bytes < w.bytes) return SPT_ERR_WORKSPACE;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const uint16_t* q = static_cast<const uint16_t*>(Q);
  const uint16_t* k = static_cast<const uint16_t*>(K);
  const uint16_t* v = static_cast<const uint16_t*>(V);
  const uint16_t* dy = static_cast<const uint16_t*>(dY);
  float* Amut = const_cast<float*>(A);   // read-only in the backward instantiation
  const bool resident = seq_resident(shape->n, shape->dh);
  if (use_dense_rows(*shape)) {
    ScopedKernelTimer tm(kSlotMhaBwdQ, st);
    if (mha_dense_bwd_q(*shape, K, V, dY, idx, A, w.dS, dQ, st) != hipSuccess) return SPT_ERR_HIP;
  } else {
    ScopedKernelTimer tm(kSlotMhaBwdQ, st);
    uint16_t* dq = static_cast<uint16_t*>(dQ);
    if (rows_in_lds(*shape)) {
      if (shape->dh == 64) {
        launch_seq_dots<64, true>(*shape, dy, v, idx, A, w.dS, st);
        launch_seq_accum<64, false>(*shape, k, idx, nullptr, nullptr, w.dS, dq, st);
      } else {
        launch_seq_dots<128, true>(*shape, dy, v, idx, A, w.dS, st);
        launch_seq_accum<128, false>(*shape, k, idx, nullptr, nullptr, w.dS, dq, st);
      }
    } else if (shape->dh == 64) {
      launch_row<64, true>(*shape, dy, v, k, idx, Amut, w.dS, dq, st);
    } else {
      launch_row<128, true>(*shape, dy, v, k, idx, Amut, w.dS, dq, st);
    }
  }
  if (use_dense(*shape)) {
    ScopedKernelTimer tm(kSlotMhaBwdKV, st);
    return mha_dense_bwd_kv(*shape, Q, dY, idx, A, w.dS, dK, dV, st) == hipSuccess ? SPT_OK : SPT_ERR_HIP;
  }
  {
    ScopedKernelTimer tm(kSlotMhaTranspose, st);
    if (!w.gbits) {
      const size_t lds = transpose_lds_bytes(shape->n, shape->L);
      (void)hipFuncSetAttribute(reinterpret_cast<const void*>(transpose_lists_kernel<true>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      hipLaunchKernelGGL(transpose_lists_kernel<true>, dim3(shape->S), dim3(kTransposeThreads), lds, st, idx,
                         w.toff, w.tlist, nullptr, shape->n, shape->L);
    } else {
      const size_t lds = ((size_t)shape->n + 1) * sizeof(int32_t);
      hipLaunchKernelGGL(transpose_lists_kernel<false>, dim3(shape->S), dim3(kTransposeThreads), lds, st, idx,
                         w.toff, w.tlist, w.gbits, shape->n, shape->L);
    }
  }
  {
    ScopedKernelTimer tm(kSlotMhaBwdKV, st);
    const dim3 grid(seq_block_grid((shape->n + 3) / 4, shape->S));
    uint16_t* dk = static_cast<uint16_t*>(dK);
    uint16_t* dv = static_cast<uint16_t*>(dV);
    if (resident) {
      if (shape->dh == 64) {
        launch_seq_accum<64, true>(*shape, dy, nullptr, w.toff, w.tlist, A, dv, st);
        launch_seq_accum<64, true>(*shape, q, nullptr, w.toff, w.tlist, w.dS, dk, st);
      } else {
        launch_seq_accum<128, true>(*shape, dy, nullptr, w.toff, w.tlist, A, dv, st);
        launch_seq_accum<128, true>(*shape, q, nullptr, w.toff, w.tlist, w.dS, dk, st);
      }
    } else if (shape->dh == 64)
      hipLaunchKernelGGL(attn_kv_kernel<64>, grid, dim3(256), 0, st, q, dy, A, w.dS, w.toff, w.tlist,
                         static_cast<uint16_t*>(dK), static_cast<uint16_t*>(dV), shape->S, shape->n, shape->L);
    else
      hipLaunchKernelGGL(attn_kv_kernel<128>, grid, dim3(256), 0, st, q, dy, A, w.dS, w.toff, w.tlist,
                         static_cast<uint16_t*>(dK), static_cast<uint16_t*>(dV), shape->S, shape->n, shape->L);
  }
  return hipGetLastError() == hipSuccess ? SPT_OK : SPT_ERR_HIP;
}

}  // extern "C"
