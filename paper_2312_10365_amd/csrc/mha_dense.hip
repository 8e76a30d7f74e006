// Sparse attention of section 4.1 (SDDMM, softmax over the kept keys, SpMM and their derivative) on
// the matrix cores.
//
// A query keeps L of n keys, L / n about 1/8.  Gathered row by row (mha.hip) the products run on
// the vector units at 128-256 bytes of LDS per multiply-add pair; as dense tiles they are n / L
// times the multiply-adds on units sixteen times as fast, and every operand byte is shared by a
// 32 x 32 tile.  What stays sparse is what the method stores: the index lists, A and dS.  Between
// the two a tile of one query block lives in LDS with one 32-bit word per (query, key):
//
//   rows kernel (query side)    S = R G1^T for a block of queries (bf16 MFMA, fp32) -> tile; every
//     list entry gathers its word; softmax (forward) or its Jacobian (backward) over the list;
//     the weights go back to the same words, all other words are zero; Out = tile x G2.
//     forward (R, G1, G2) = (Q, K, V): A, Y.   backward (dY, V, K): dS, dQ.
//   keys kernel (backward)      the lists of a block of queries are scattered into two tiles
//     (A, dS) of 256 keys; dV += A^T dY, dK += dS^T Q stay in accumulators over all queries.  No
//     transposed lists, no atomics: the sum order is the query order.
//
// Precision.  Weights are fp32 in the lists.  As MFMA operands they are two fp16 numbers, hi = w
// rounded and lo = (w - hi) rounded, packed in the word: off by at most 2^-24 of w, as an fp32
// rounding is, while w is within 2^-17 of the largest weight of its row (rows kernel) or sequence
// (keys kernel), and by at most 2^-40 of that largest weight below.  The other operand (V, K, dY, Q)
// is bf16 by nature; moved to fp16 with the sequence's largest exponent at the top of fp16's range
// every value within 2^-29 of the largest is exact.  Both products, hi and lo, accumulate in fp32.
#include <math.h>
#include <type_traits>

#include "ffn_common.hpp"
#include "mha_host.hpp"

namespace spt {
namespace {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4u __attribute__((ext_vector_type(4), aligned(4)));   // 4-byte aligned: rows of L entries
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32x2u __attribute__((ext_vector_type(2), aligned(4)));
typedef float f32x2u __attribute__((ext_vector_type(2), aligned(4)));

// Accesses at a wave-uniform base plus a 32-bit byte offset (one address register per lane).
template <class T>
__device__ __forceinline__ T load_at(const void* base, uint32_t bytes) {
  return *reinterpret_cast<const T*>(static_cast<const char*>(base) + bytes);
}
template <class T>
__device__ __forceinline__ void store_at(void* base, uint32_t bytes, const T& v) {
  *reinterpret_cast<T*>(static_cast<char*>(base) + bytes) = v;
}

__device__ __forceinline__ f16x8 as_f16x8(const u32x4& v) { return __builtin_bit_cast(f16x8, v); }

// Workgroup -> (sequence, part): the parts of a sequence run side by side on one XCD (sequence mod 8).
__device__ __forceinline__ bool seq_part(int parts, int S, int& s, int& part) {
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  s = (slot / parts) * 8 + xcd;
  part = slot % parts;
  return s < S;
}

// ---- bf16 -> fp16.  A bf16 number with biased exponent E maps to the fp16 number with biased
// exponent E - off: a subtraction and a shift on the 16-bit pattern.  `off` puts the largest
// exponent of the sequence at 30; what falls below 2^-29 of it becomes at most 2^-29 of it.
// (Infinities and NaNs, exponent 255, stay what they are.)
struct F16Scale {
  uint32_t off2;   // off << 7 in both halves
  float up;        // true value = fp16 value * up
};
__device__ __forceinline__ F16Scale f16_scale(uint32_t maxbits) {   // largest |x| as a bf16 pattern
  const int e = (int)(maxbits >> 7);
  const int off = e == 255 ? 224 : (e > 30 ? e - 30 : 0);
  return F16Scale{(uint32_t)off * 0x00800080u, ldexpf(1.0f, off - 112)};
}
__device__ __forceinline__ uint32_t bf16x2_to_f16x2(uint32_t w, uint32_t off2) {
  typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
  const u16x2 mag = __builtin_bit_cast(u16x2, w & 0x7FFF7FFFu);
  const u16x2 sub = __builtin_elementwise_sub_sat(mag, __builtin_bit_cast(u16x2, off2));
  const u16x2 sh = sub << (unsigned short)3;
  return (w & 0x80008000u) | __builtin_bit_cast(uint32_t, sh);
}
__device__ __forceinline__ u32x4 to_f16(const u32x4& v, uint32_t off2) {
  return u32x4{bf16x2_to_f16x2(v[0], off2), bf16x2_to_f16x2(v[1], off2), bf16x2_to_f16x2(v[2], off2),
               bf16x2_to_f16x2(v[3], off2)};
}
__device__ __forceinline__ uint32_t max_mag(uint32_t m, const u32x4& v) {
#pragma unroll
  for (int e = 0; e < 4; ++e) m = max(m, max(v[e] & 0x7FFFu, (v[e] >> 16) & 0x7FFFu));
  return m;
}

// A weight as hi | lo << 16 (already scaled into fp16's range).
__device__ __forceinline__ uint32_t split_f16(float w) {
  const _Float16 hi = (_Float16)w;
  const _Float16 lo = (_Float16)(w - (float)hi);
  return (uint32_t)__builtin_bit_cast(uint16_t, hi) | ((uint32_t)__builtin_bit_cast(uint16_t, lo) << 16);
}
// Eight words hi | lo << 16 -> the two MFMA fragments.
__device__ __forceinline__ void unzip(const u32x4& a, const u32x4& b, f16x8& hi, f16x8& lo) {
  constexpr uint32_t kLow = 0x05040100u, kHigh = 0x07060302u;   // low / high halves of (second, first)
  u32x4 h, l;
  h[0] = __builtin_amdgcn_perm(a[1], a[0], kLow);  l[0] = __builtin_amdgcn_perm(a[1], a[0], kHigh);
  h[1] = __builtin_amdgcn_perm(a[3], a[2], kLow);  l[1] = __builtin_amdgcn_perm(a[3], a[2], kHigh);
  h[2] = __builtin_amdgcn_perm(b[1], b[0], kLow);  l[2] = __builtin_amdgcn_perm(b[1], b[0], kHigh);
  h[3] = __builtin_amdgcn_perm(b[3], b[2], kLow);  l[3] = __builtin_amdgcn_perm(b[3], b[2], kHigh);
  hi = as_f16x8(h);
  lo = as_f16x8(l);
}
// 2^x with x chosen so that max * 2^x lies in [2^14, 2^15) (1 for zero, infinity and NaN).
__device__ __forceinline__ int scale_exponent(float maxabs) {
  const int e = (int)((__float_as_uint(maxabs) >> 23) & 255u);
  return (e == 0 || e == 255) ? 0 : 141 - e;
}

// Reductions over the 16 lanes that share a query.
template <int CTRL>
__device__ __forceinline__ float dpp16(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ float row_sum(float x) {
  x += dpp16<0xB1>(x);
  x += dpp16<0x4E>(x);
  x += dpp16<0x141>(x);
  return x + dpp16<0x140>(x);
}
__device__ __forceinline__ float row_max(float x) {
  x = fmaxf(x, dpp16<0xB1>(x));
  x = fmaxf(x, dpp16<0x4E>(x));
  x = fmaxf(x, dpp16<0x141>(x));
  return fmaxf(x, dpp16<0x140>(x));
}

// Transposing fragment reads out of rows of DH 16-bit values (row = K index): byte offset of the lane's
// r = 0 read of column tile `ct`, K-step 0; K-step s is 16 rows further, the r = 1 read 4 rows.  The
// 16-byte chunks of a row are permuted so the 16 lanes of a pass hit different banks.
template <int DH>
__device__ __forceinline__ uint32_t chunk_swizzle(int row) {
  return DH == 64 ? (uint32_t)(((row >> 1) & 1) << 2) : (uint32_t)((row & 3) << 2);
}
template <int DH>
__device__ __forceinline__ uint32_t tr_offset(int lane, int ct) {
  const int g = lane >> 4, sl = lane & 15, a4 = sl & 3;
  const int krow = 8 * (g >> 1) + (sl >> 2);
  const int col = ct * 32 + 4 * (4 * (a4 & 1) + 2 * (g & 1) + (a4 >> 1));   // rho32: a lane ends up with 16 adjacent columns
  return (uint32_t)(krow * (DH * 2) + (((uint32_t)(col >> 3) ^ chunk_swizzle<DH>(krow)) * 16) + (col & 4) * 2);
}
// (the r = 1 read is 4 rows on: the swizzle terms repeat with period 4, so it is a constant further)
template <int DH>
__device__ __forceinline__ u32x4 tr_frag(const char* p) {
  return __builtin_bit_cast(u32x4, tr_read_frag(p, p + 4 * DH * 2));
}

// ------------------------------------------------------------------------------------------
// Rows kernel.  NW wavefronts, BQ = 32 QT = 4 NW queries per block, KC = 32 KT NW keys per chunk.
//   S phase: wavefront w multiplies its KT tiles of 32 keys (fragments in registers) with all QT
//            query tiles; MFMA rows = keys (rho32), so a lane writes 16 adjacent words of ITS query.
//   lists:   16 lanes per query, four adjacent entries per lane and vector; rows 4w .. 4w+3 of the
//            tile belong to wavefront w from the gather to the scatter, so no barrier inside.
//   PV:      wavefront = (key group of KPG keys) x (column group of CT 32-column tiles), G2
//            fragments in registers; the key groups' partial products are added through LDS in
//            group order.
// STAT: the sequence is one chunk, G1 and G2 fragments stay in registers for all of the
// workgroup's query blocks.  Otherwise they are fetched again for every block.
// A block is bound by LDS traffic: for DH = 64 about 435 KiB per 32 queries x 512 keys (tile written,
// cleared and read 66 KiB each, partial products 128, R 36, gathers and scatters) against 1500
// cycles of MFMA.
// Registers: 128 per lane (two workgroups of 8 wavefronts on a CU, or one of 16) where that holds the
// fragments and the lists without spilling, 256 otherwise.
template <int DH, int NW, int KT, int LPL>
constexpr int rows_waves_per_simd() { return NW == 16 || (KT * DH <= 128 && LPL <= 2) ? 4 : 2; }

template <int DH, int NW, int QT, int KT, int KG, int LPL, bool BWD, bool STAT>
__global__ __launch_bounds__(NW * 64, (rows_waves_per_simd<DH, NW, KT, LPL>())) void mha_rows_kernel(
    const uint16_t* __restrict__ R, const uint16_t* __restrict__ G1, const uint16_t* __restrict__ G2,
    const int32_t* __restrict__ idx, const float* __restrict__ Ain, float* __restrict__ Wout,
    uint16_t* __restrict__ Out, float2* __restrict__ maxes, int S, int n, int L, float scale, int parts, int kc) {
  constexpr int BQ = 32 * QT, KS = DH / 16, CG = NW / KG, CT = DH / 32 / CG;
  constexpr int KPG = NW * KT * 32 / KG, VS = KPG / 16, NT = NW * 64;
  constexpr int RSTRIDE = DH * 2 + 16;
  constexpr bool KSTAT = STAT;
  static_assert(BQ == 4 * NW && CT >= 1, "shape of the workgroup");
  extern __shared__ uint4 md_smem[];
  char* smem = reinterpret_cast<char*>(md_smem);
  // (lane roles are formed again for every block from a value the compiler cannot follow: as loop
  // invariants the dozens of addresses built on them would be hoisted into registers and spilled)
  uint32_t tid = threadIdx.x, lane = tid & 63, i = lane & 31, h = lane >> 5;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  uint32_t ql = 4 * wave + (lane >> 4), e4 = 4 * (lane & 15);   // list role: query of the block, first entry of a vector of four
  auto fresh_roles = [&]() {
    asm volatile("" : "+v"(tid));
    lane = tid & 63; i = lane & 31; h = lane >> 5;
    ql = 4 * wave + (lane >> 4); e4 = 4 * (lane & 15);
  };
  int s, part;
  if (!seq_part(parts, S, s, part)) return;
  const int ts = kc + 4;                                   // words per tile row
  uint32_t* tile = reinterpret_cast<uint32_t*>(smem);
  const int tile_bytes = max(BQ * ts * 4, max(KG * BQ * DH * 4, kc * DH * 2));
  char* rlds = smem + tile_bytes;                          // [BQ] rows of R
  float* rowup = reinterpret_cast<float*>(rlds + BQ * RSTRIDE);   // [BQ] output scale of a query
  uint32_t* red = reinterpret_cast<uint32_t*>(rowup + BQ);        // [NW + 1]
  const size_t base = (size_t)s * n;
  // (pointers of the sequence are wave-uniform, offsets inside it fit 32 bits)
  const uint16_t* g1 = G1 + base * DH;
  const uint16_t* g2 = G2 + base * DH;
  R += base * DH;
  Out += base * DH;
  idx += base * L;
  Ain += base * L;
  Wout += base * L;
  const int nblk = (n + BQ - 1) / BQ, nch = (n + kc - 1) / kc;

  const uint32_t kg = wave / CG, cg = wave % CG;
  uint32_t vtr[CT];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) vtr[ct] = tr_offset<DH>(lane, cg * CT + ct);

  bf16x8 kf[KT][KS];
  auto load_k = [&](uint32_t c0) {
#pragma unroll
    for (int t = 0; t < KT; ++t) {
      // (padding keys: any row, their words are never read)
      const uint32_t key = min(c0 + (wave * KT + t) * 32 + rho32(i), (uint32_t)n - 1);
#pragma unroll
      for (int k = 0; k < KS; ++k) kf[t][k] = as_bf16x8(load_at<uint4>(g1, key * (DH * 2) + h * DH + k * 16));
    }
  };
  // G2 rows c0 .. c0 + kc of the sequence into the tile's space; `mag`: largest magnitude on the way.
  auto stage_v = [&](uint32_t c0, uint32_t& mag) {
    constexpr uint32_t NC = DH / 8;
    for (uint32_t q0 = tid; q0 < kc * NC; q0 += 8 * NT) {
      u32x4 x[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const uint32_t q = q0 + u * NT, row = min(c0 + q / NC, (uint32_t)n - 1);
        if (q < kc * NC) x[u] = load_at<u32x4>(g2, row * (DH * 2) + (q % NC) * 16);
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const uint32_t q = q0 + u * NT, row = q / NC;
        if (q < kc * NC) {
          mag = max_mag(mag, x[u]);
          *reinterpret_cast<u32x4*>(smem + row * (DH * 2) + ((uint32_t)(q % NC) ^ chunk_swizzle<DH>(row)) * 16) = x[u];
        }
      }
    }
  };
  u32x4 vf[VS][CT];
  auto read_v = [&](uint32_t off2) {
#pragma unroll
    for (int k = 0; k < VS; ++k) {
      const uint32_t row0 = kg * KPG + 16 * k;
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        vf[k][ct] = u32x4{0u, 0u, 0u, 0u};
        if (row0 < (uint32_t)kc) vf[k][ct] = to_f16(tr_frag<DH>(smem + row0 * (DH * 2) + vtr[ct]), off2);
      }
    }
  };
  auto block_max = [&](uint32_t mag) -> uint32_t {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mag = max(mag, (uint32_t)__shfl_xor((int)mag, o));
    if (lane == 0) red[wave] = mag;
    __syncthreads();
    uint32_t m = 0u;
#pragma unroll
    for (int w = 0; w < NW; ++w) m = max(m, red[w]);
    return m;
  };

  // R rows of a block: thread -> 16-byte pieces, requested early, written to LDS when the rows are free.
  constexpr int RP = BQ * (DH / 8) / NT > 0 ? BQ * (DH / 8) / NT : 1;
  u32x4 rnext[RP];
  auto request_r = [&](int b) {
#pragma unroll
    for (int u = 0; u < RP; ++u) {
      const uint32_t q = tid + u * NT, row = min((uint32_t)(b * BQ) + q / (DH / 8), (uint32_t)n - 1);
      if (RP * NT == BQ * (DH / 8) || q < BQ * (DH / 8)) rnext[u] = load_at<u32x4>(R, row * (DH * 2) + (q % (DH / 8)) * 16);
    }
  };
  auto store_r = [&]() {
#pragma unroll
    for (int u = 0; u < RP; ++u) {
      const uint32_t q = tid + u * NT;
      if (RP * NT == BQ * (DH / 8) || q < BQ * (DH / 8)) *reinterpret_cast<u32x4*>(rlds + (q / (DH / 8)) * RSTRIDE + (q % (DH / 8)) * 16) = rnext[u];
    }
  };
  // The four queries of this wavefront: lane = (query 4 wave + lane / 16, entries at(v) + 0..3 of its
  // row).  at(v) is 64 v + e4 moved back where that would leave the row: those lanes repeat entries of
  // their neighbours (same index, same value, same place) and leave them out of the sums.  Queries past
  // the end repeat the last one.
  auto at = [&](int v) -> uint32_t { return min(64u * v + e4, (uint32_t)L - 4); };
  auto row_bytes = [&](int b) -> uint32_t { return min(b * BQ + ql, (uint32_t)n - 1) * (uint32_t)L * 4; };
  int jj[LPL][4];
  float aa[LPL][4];
  auto request_lists = [&](int b) {
    const uint32_t row = row_bytes(b);
#pragma unroll
    for (int v = 0; v < LPL; ++v) {
      const u32x4 x = load_at<u32x4u>(idx, row + at(v) * 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) jj[v][e] = (int)x[e];
      if (BWD) {
        const f32x4 y = load_at<f32x4u>(Ain, row + at(v) * 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) aa[v][e] = y[e];
      }
    }
  };

  // ---- once per workgroup
  F16Scale gs;
  {
    uint32_t mag = 0u;
    if (STAT) {
      stage_v(0, mag);
      gs = f16_scale(block_max(mag));       // (its barrier also makes the staged rows visible)
      read_v(gs.off2);
      __syncthreads();
    } else {
      const uint32_t np = n * (DH / 8);
      for (uint32_t q0 = tid; q0 < np; q0 += 8 * NT) {      // eight loads in flight
        u32x4 x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = load_at<u32x4>(g2, min(q0 + u * NT, np - 1) * 16);
#pragma unroll
        for (int u = 0; u < 8; ++u) mag = max_mag(mag, x[u]);
      }
      gs = f16_scale(block_max(mag));
    }
  }
  int b = part;
  if (b < nblk) { request_r(b); request_lists(b); load_k(0); store_r(); }
  __syncthreads();

  for (; b < nblk; b += parts) {
    fresh_roles();
    float w[LPL][4];
    for (int c = 0; c < (STAT ? 1 : nch); ++c) {
      const int c0 = c * kc;
#pragma unroll
      for (int t = 0; t < KT; ++t) {
        if ((wave * KT + t) * 32 >= (uint32_t)kc) continue;          // uniform
#pragma unroll
        for (int qt = 0; qt < QT; ++qt) {
          f32x16 acc;
#pragma unroll
          for (int v = 0; v < 16; ++v) acc[v] = 0.f;
#pragma unroll
          for (int k = 0; k < KS; ++k) {
            const bf16x8 rf = as_bf16x8(*reinterpret_cast<const uint4*>(rlds + (qt * 32 + i) * RSTRIDE + h * DH + k * 16));
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[t][k], rf, acc, 0, 0, 0);
          }
          f32x4* dst = reinterpret_cast<f32x4*>(tile + (qt * 32 + i) * ts + (wave * KT + t) * 32 + 16 * h);
#pragma unroll
          for (int e = 0; e < 4; ++e) dst[e] = f32x4{acc[4 * e], acc[4 * e + 1], acc[4 * e + 2], acc[4 * e + 3]};
          __builtin_amdgcn_sched_barrier(0);               // (one tile's fragments at a time: registers)
        }
      }
      if (!STAT && c + 1 < nch) load_k(c0 + kc);
      __syncthreads();
      const uint32_t* trow = tile + ql * ts;
#pragma unroll
      for (int v = 0; v < LPL; ++v)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t jl = (uint32_t)(jj[v][e] - c0);
          const bool in = jl < (uint32_t)min(kc, n - c0);
          const float got = __uint_as_float(trow[in ? jl : 0u]);
          if (STAT) w[v][e] = got;
          else w[v][e] = in ? got : (c == 0 ? 0.f : w[v][e]);
        }
      if (!STAT) __syncthreads();
    }
    // ---- softmax / Jacobian over the list, in registers
    bool ok[LPL][4], own[LPL][4];
#pragma unroll
    for (int v = 0; v < LPL; ++v)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        ok[v][e] = (uint32_t)jj[v][e] < (uint32_t)n;        // -1 = no key; out of range alike
        own[v][e] = at(v) + e >= 64u * v + e4;
      }
    int up_e = 0;
    if (!BWD) {
      float mx = -INFINITY;
#pragma unroll
      for (int v = 0; v < LPL; ++v)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          w[v][e] = ok[v][e] ? w[v][e] * scale : -INFINITY;
          mx = fmaxf(mx, w[v][e]);
        }
      mx = row_max(mx);
      float sum = 0.f;
#pragma unroll
      for (int v = 0; v < LPL; ++v)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          w[v][e] = ok[v][e] ? __expf(w[v][e] - mx) : 0.f;
          sum += own[v][e] ? w[v][e] : 0.f;
        }
      sum = row_sum(sum);
      const float inv = sum > 0.f ? 1.0f / sum : 0.f;
#pragma unroll
      for (int v = 0; v < LPL; ++v)
#pragma unroll
        for (int e = 0; e < 4; ++e) w[v][e] *= inv;
      up_e = 14;                                            // weights are at most 1
    } else {
      float sum = 0.f, ma = 0.f, mx = 0.f;
#pragma unroll
      for (int v = 0; v < LPL; ++v)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          aa[v][e] = ok[v][e] ? aa[v][e] : 0.f;
          sum = fmaf(own[v][e] ? aa[v][e] : 0.f, ok[v][e] ? w[v][e] : 0.f, sum);
          ma = fmaxf(ma, fabsf(aa[v][e]));
        }
      sum = row_sum(sum);
#pragma unroll
      for (int v = 0; v < LPL; ++v)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          w[v][e] = ok[v][e] ? aa[v][e] * (w[v][e] - sum) * scale : 0.f;
          mx = fmaxf(mx, fabsf(w[v][e]));
        }
      mx = row_max(mx);
      up_e = scale_exponent(mx);
      // the largest A and dS of these four queries, for the keys kernel
      ma = row_max(ma);
      ma = fmaxf(ma, __shfl_xor(ma, 16)); ma = fmaxf(ma, __shfl_xor(ma, 32));
      mx = fmaxf(mx, __shfl_xor(mx, 16)); mx = fmaxf(mx, __shfl_xor(mx, 32));
      if (lane == 0 && b * BQ + 4 * wave < (uint32_t)n) maxes[(size_t)s * ((n + 3) / 4) + (b * BQ + 4 * wave) / 4] = make_float2(ma, mx);
    }
    {
      const uint32_t row = row_bytes(b);
#pragma unroll
      for (int v = 0; v < LPL; ++v)
        store_at<f32x4u>(Wout, row + at(v) * 4, f32x4{w[v][0], w[v][1], w[v][2], w[v][3]});
    }
    const float fs = ldexpf(1.0f, up_e);
    if ((lane & 15) == 0) rowup[ql] = ldexpf(gs.up, -up_e);
    uint32_t word[LPL][4];
#pragma unroll
    for (int v = 0; v < LPL; ++v)
#pragma unroll
      for (int e = 0; e < 4; ++e) word[v][e] = split_f16(w[v][e] * fs);

    // ---- Out = tile x G2
    f32x16 acc[QT][CT];
#pragma unroll
    for (int qt = 0; qt < QT; ++qt)
#pragma unroll
      for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[qt][ct][v] = 0.f;
    for (int c = 0; c < (STAT ? 1 : nch); ++c) {
      const int c0 = c * kc;
      if (!STAT) {
        uint32_t unused = 0u;
        __syncthreads();
        stage_v(c0, unused);
        __syncthreads();
        read_v(gs.off2);
        __syncthreads();
      }
      // this wavefront's four rows: cleared, then the list entries
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        uint4* dst = reinterpret_cast<uint4*>(tile + (4 * wave + r) * ts);
        for (uint32_t e = lane; e < (uint32_t)kc / 4; e += 64) dst[e] = make_uint4(0u, 0u, 0u, 0u);
      }
      wave_lds_fence();
      uint32_t* trow = tile + ql * ts;
#pragma unroll
      for (int v = 0; v < LPL; ++v)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t jl = (uint32_t)(jj[v][e] - c0);
          if (jl < (uint32_t)min(kc, n - c0)) trow[jl] = word[v][e];
        }
      if (c == (STAT ? 0 : nch - 1) && b + parts < nblk) { request_r(b + parts); request_lists(b + parts); }
      __syncthreads();
#pragma unroll
      for (int k = 0; k < VS; ++k) {
        const uint32_t k0 = kg * KPG + 16 * k;
        if (k0 < (uint32_t)kc) {                                      // uniform
#pragma unroll
          for (int qt = 0; qt < QT; ++qt) {
            const u32x4* src = reinterpret_cast<const u32x4*>(tile + (qt * 32 + i) * ts + k0 + 8 * h);
            f16x8 hi, lo;
            unzip(src[0], src[1], hi, lo);
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
              acc[qt][ct] = __builtin_amdgcn_mfma_f32_32x32x16_f16(as_f16x8(vf[k][ct]), hi, acc[qt][ct], 0, 0, 0);
              acc[qt][ct] = __builtin_amdgcn_mfma_f32_32x32x16_f16(as_f16x8(vf[k][ct]), lo, acc[qt][ct], 0, 0, 0);
            }
            if (k % 2 == 1) __builtin_amdgcn_sched_barrier(0);
          }
        }
      }
    }
    __syncthreads();
    // ---- partial products [group][query][DH], 16-byte chunks permuted by query
    const uint32_t groups = STAT ? min(KG, (kc + KPG - 1) / KPG) : KG;
    float* partial = reinterpret_cast<float*>(smem);
    constexpr int PC = DH / 4;                              // 16-byte chunks per row
    if (kg < groups) {
#pragma unroll
      for (int qt = 0; qt < QT; ++qt)
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const uint32_t ch = ((cg * CT + ct) * 8 + 4 * h + e) ^ (i & 15);
            const f32x16& a = acc[qt][ct];
            *reinterpret_cast<f32x4*>(partial + ((size_t)kg * BQ + qt * 32 + i) * DH + ch * 4) =
                f32x4{a[4 * e], a[4 * e + 1], a[4 * e + 2], a[4 * e + 3]};
          }
    }
    if (b + parts < nblk) {
      if (!KSTAT) load_k(0);                                // (not held across the products above: registers)
      store_r();
    }
    __syncthreads();
    for (uint32_t it = tid; it < BQ * PC; it += NT) {
      const uint32_t r = it / PC, ch = it % PC;
      const float* p = partial + (size_t)r * DH + (ch ^ (r & 15)) * 4;
      f32x4 sum = *reinterpret_cast<const f32x4*>(p);
      for (uint32_t gidx = 1; gidx < groups; ++gidx) sum += *reinterpret_cast<const f32x4*>(p + (size_t)gidx * BQ * DH);
      const float up = rowup[r];
      if (b * BQ + r < (uint32_t)n)
        store_at<uint2>(Out, (b * BQ + r) * (DH * 2) + ch * 8,
                        make_uint2(pack_bf16x2(sum[0] * up, sum[1] * up), pack_bf16x2(sum[2] * up, sum[3] * up)));
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------------------------------------
// Keys kernel: dV = A^T dY, dK = dS^T Q for 256 keys of a sequence, 32 queries per step.  A wavefront
// owns 64 keys and 64 columns of one of the two gradients in accumulators: 8 wavefronts for 64-wide
// heads (two workgroups per CU), 16 for 128-wide ones.  The A and dS words of a step are scattered
// into two LDS tiles [key][query] and taken out again afterwards (only the words that were set), by
// the wavefront that owns the query: two barriers per step.  Entries whose key is another
// workgroup's go to dummy words behind the tile.
// 16-byte chunk c of tile row r sits at c ^ ((r >> 1) & 7): the 16 rows of a pass hit all banks.
constexpr int KV_KEYS = 256, KV_Q = 32;
constexpr int KV_TILE = KV_KEYS * KV_Q;                    // words
constexpr int KV_TS = KV_TILE + 64;                        // ... and the 64 dummy words behind them
template <int DH, int LPL>
__global__ __launch_bounds__(DH * 8, DH == 128 || LPL <= 2 ? 4 : 2) void mha_keys_kernel(
    const uint16_t* __restrict__ Q, const uint16_t* __restrict__ dY, const int32_t* __restrict__ idx,
    const float* __restrict__ A, const float* __restrict__ dS, const float2* __restrict__ maxes,
    uint16_t* __restrict__ dK, uint16_t* __restrict__ dV, int S, int n, int L, int parts) {
  constexpr int NT = DH * 8, NW = NT / 64, NC = DH / 8;
  constexpr int QW = KV_Q / NW, EL = QW;                   // queries per wavefront; 64 / QW lanes x EL entries cover 64
  constexpr int ROWS = KV_Q * DH * 2;                      // bytes of a step's dY (then Q) rows
  extern __shared__ uint4 kv_smem[];
  char* smem = reinterpret_cast<char*>(kv_smem);           // A tile, dS tile, dY rows, Q rows
  char* rows = smem + 2 * KV_TS * 4;
  uint32_t* red = reinterpret_cast<uint32_t*>(rows);       // (before the loop)
  uint32_t* words = reinterpret_cast<uint32_t*>(smem);
  const uint32_t tid = threadIdx.x, lane = tid & 63, i = lane & 31, h = lane >> 5;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t t = wave & 1, kg = (wave >> 1) & 3, dhalf = wave >> 3;
  int s, part;
  if (!seq_part(parts, S, s, part)) return;
  const size_t base = (size_t)s * n;
  const int key0 = part * KV_KEYS;
  const uint16_t* src[2] = {dY + base * DH, Q + base * DH};
  idx += base * L;
  A += base * L;
  dS += base * L;

  // scales of the sequence: largest |dY|, |Q| (bf16 patterns), |A|, |dS|
  F16Scale rs[2];
  int we[2];
  {
    uint32_t m[4] = {0u, 0u, 0u, 0u};
    for (uint32_t q0 = tid; q0 < (uint32_t)(n * NC); q0 += 4 * NT) {   // eight loads in flight
      u32x4 x[2][4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const uint32_t at = min(q0 + u * NT, (uint32_t)(n * NC) - 1) * 16;   // (past the end: the last piece again)
        x[0][u] = load_at<u32x4>(src[0], at);
        x[1][u] = load_at<u32x4>(src[1], at);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) { m[0] = max_mag(m[0], x[0][u]); m[1] = max_mag(m[1], x[1][u]); }
    }
    const int n4 = (n + 3) / 4;
    for (uint32_t q = tid; q < (uint32_t)n4; q += NT) {
      const float2 v = maxes[(size_t)s * n4 + q];
      m[2] = max(m[2], __float_as_uint(v.x));              // non-negative: ordered like their bits
      m[3] = max(m[3], __float_as_uint(v.y));
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) m[e] = max(m[e], (uint32_t)__shfl_xor((int)m[e], o));
      if (lane == 0) red[wave * 4 + e] = m[e];
    }
    for (uint32_t e = tid; e < 2 * KV_TS / 4; e += NT) reinterpret_cast<uint4*>(smem)[e] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int w = 0; w < NW; ++w) m[e] = max(m[e], red[w * 4 + e]);
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      rs[x] = f16_scale(m[x]);
      we[x] = scale_exponent(__uint_as_float(m[2 + x]));
    }
    __syncthreads();
  }
  const float fsA = ldexpf(1.0f, we[0]), fsS = ldexpf(1.0f, we[1]);
  const uint32_t last = min(KV_KEYS, n - key0);

  // rows of a step: thread = one 16-byte piece of dY or of Q (2 x 32 x NC = NT pieces)
  static_assert(2 * KV_Q * NC == NT, "one piece per thread");
  const uint32_t px = tid / (KV_Q * NC), pr = (tid / NC) % KV_Q, pc = tid % NC;
  const uint16_t* rsrc = px ? src[1] : src[0];
  const uint32_t row_dst = px * ROWS + pr * (DH * 2) + (pc ^ chunk_swizzle<DH>(pr)) * 16;
  const uint32_t row_off2 = px ? rs[1].off2 : rs[0].off2;
  const uint32_t row_end = (uint32_t)(n - 1) * (DH * 2) + pc * 16;
  uint32_t row_at = pr * (DH * 2) + pc * 16;
  u32x4 rnext;
  auto request_rows = [&]() {
    rnext = load_at<u32x4>(rsrc, min(row_at, row_end));
    row_at += KV_Q * DH * 2;
  };
  // lists: lane = (query QW wave + lane / (64 / QW), entries at(v) .. at(v) + EL - 1 of its row); lanes past
  // the row's end repeat its last entries (same word, same value)
  const uint32_t ql = QW * wave + lane / (64 / QW), el = EL * (lane % (64 / QW));
  const uint32_t list_end = (uint32_t)(n - 1) * (uint32_t)L * 4;
  uint32_t list_at = ql * (uint32_t)L * 4;
  int jn[LPL][EL];
  float an[LPL][EL], dn[LPL][EL];
  auto request_lists = [&]() {
    const uint32_t row = min(list_at, list_end);
    list_at += KV_Q * (uint32_t)L * 4;
#pragma unroll
    for (int v = 0; v < LPL; ++v) {
      const uint32_t at = row + min(64u * v + el, (uint32_t)L - EL) * 4;
      if constexpr (EL == 4) {
        const u32x4 x = load_at<u32x4u>(idx, at);
        const f32x4 y = load_at<f32x4u>(A, at), z = load_at<f32x4u>(dS, at);
#pragma unroll
        for (int e = 0; e < EL; ++e) { jn[v][e] = (int)x[e]; an[v][e] = y[e]; dn[v][e] = z[e]; }
      } else {
        const u32x2u x = load_at<u32x2u>(idx, at);
        const f32x2u y = load_at<f32x2u>(A, at), z = load_at<f32x2u>(dS, at);
#pragma unroll
        for (int e = 0; e < EL; ++e) { jn[v][e] = (int)x[e]; an[v][e] = y[e]; dn[v][e] = z[e]; }
      }
    }
  };
  uint32_t old[LPL][EL];                                   // the words this lane has set
#pragma unroll
  for (int v = 0; v < LPL; ++v)
#pragma unroll
    for (int e = 0; e < EL; ++e) old[v][e] = KV_TILE + lane;
  auto scatter = [&](int b) {
#pragma unroll
    for (int v = 0; v < LPL; ++v)
#pragma unroll
      for (int e = 0; e < EL; ++e) { words[old[v][e]] = 0u; words[old[v][e] + KV_TS] = 0u; }
    const uint32_t lim = b * KV_Q + ql < (uint32_t)n ? last : 0;   // queries past the end have no entries
#pragma unroll
    for (int v = 0; v < LPL; ++v)
#pragma unroll
      for (int e = 0; e < EL; ++e) {
        const uint32_t j = (uint32_t)(jn[v][e] - key0);
        const uint32_t at = j * KV_Q + (((ql >> 2) ^ ((j >> 1) & 7)) << 2) + (ql & 3);
        uint32_t to = KV_TILE + lane;
        to = j < lim ? at : to;
        words[to] = split_f16(an[v][e] * fsA);
        words[to + KV_TS] = split_f16(dn[v][e] * fsS);
        old[v][e] = to;
      }
  };

  uint32_t vtr[2];
#pragma unroll
  for (int ct = 0; ct < 2; ++ct) vtr[ct] = t * ROWS + tr_offset<DH>(lane, 2 * dhalf + ct);
  uint32_t wrow[2];                                        // this lane's key rows in its tensor's tile
#pragma unroll
  for (int kt = 0; kt < 2; ++kt) wrow[kt] = t * KV_TS + (kg * 64 + kt * 32 + i) * KV_Q;
  const uint32_t wsw = (i >> 1) & 7;                       // (32 and 64 rows on: the same swizzle)
  f32x16 acc[2][2];                                        // [32-key tile][32-column tile]
#pragma unroll
  for (int kt = 0; kt < 2; ++kt)
#pragma unroll
    for (int ct = 0; ct < 2; ++ct)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[kt][ct][v] = 0.f;

  const int nblk = (n + KV_Q - 1) / KV_Q;
  request_rows();
  request_lists();
  for (int b = 0; b < nblk; ++b) {
    scatter(b);
    *reinterpret_cast<u32x4*>(rows + row_dst) = to_f16(rnext, row_off2);
    request_rows();
    request_lists();
    __syncthreads();
    if (kg * 64 < last) {                                   // uniform
#pragma unroll
      for (int k = 0; k < KV_Q / 16; ++k) {
        f16x8 hi[2], lo[2];
#pragma unroll
        for (int kt = 0; kt < 2; ++kt) {
          const u32x4* trow = reinterpret_cast<const u32x4*>(words + wrow[kt]);
          unzip(trow[(4 * k + 2 * h) ^ wsw], trow[(4 * k + 2 * h + 1) ^ wsw], hi[kt], lo[kt]);
        }
#pragma unroll
        for (int ct = 0; ct < 2; ++ct) {
          const f16x8 rf = as_f16x8(tr_frag<DH>(rows + 16 * k * (DH * 2) + vtr[ct]));
#pragma unroll
          for (int kt = 0; kt < 2; ++kt) {
            acc[kt][ct] = __builtin_amdgcn_mfma_f32_32x32x16_f16(rf, hi[kt], acc[kt][ct], 0, 0, 0);
            acc[kt][ct] = __builtin_amdgcn_mfma_f32_32x32x16_f16(rf, lo[kt], acc[kt][ct], 0, 0, 0);
          }
        }
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int kt = 0; kt < 2; ++kt) {
    const uint32_t krow = kg * 64 + kt * 32 + i;
    if (krow >= last) continue;
    const float up = ldexpf(t ? rs[1].up : rs[0].up, -(t ? we[1] : we[0]));
    uint16_t* out = (t ? dK : dV) + (base + key0 + krow) * DH + dhalf * 64 + 16 * h;
#pragma unroll
    for (int ct = 0; ct < 2; ++ct) {
      const f32x16& a = acc[kt][ct];
      uint32_t p[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) p[e] = pack_bf16x2(a[2 * e] * up, a[2 * e + 1] * up);
      reinterpret_cast<uint4*>(out + ct * 32)[0] = make_uint4(p[0], p[1], p[2], p[3]);
      reinterpret_cast<uint4*>(out + ct * 32)[1] = make_uint4(p[4], p[5], p[6], p[7]);
    }
  }
}

// ------------------------------------------------------------------------------------------
// host side
template <int DH, int NW, int QT, int KT, int KG, int LPL, bool BWD, bool STAT>
hipError_t launch_rows(const spt_mha_shape_t& s, const uint16_t* R, const uint16_t* G1, const uint16_t* G2,
                       const int32_t* idx, const float* Ain, float* Wout, uint16_t* Out, float2* maxes,
                       hipStream_t st) {
  constexpr int BQ = 32 * QT, KC = NW * KT * 32;
  // one chunk: the keys rounded up to a K-step of 16 per half wavefront tile; several: equal chunks
  const int nch = (s.n + KC - 1) / KC;
  const int kc = ((s.n + nch - 1) / nch + 31) / 32 * 32;
  const size_t tile = (size_t)BQ * (kc + 4) * 4, part = (size_t)KG * BQ * DH * 4, vrows = (size_t)kc * DH * 2;
  size_t lds = tile > part ? tile : part;
  if (vrows > lds) lds = vrows;
  lds += (size_t)BQ * (DH * 2 + 16) + BQ * 4 + (NW + 1) * 4;
  const int nblk = (s.n + BQ - 1) / BQ;
  int parts = nblk;
  if (STAT) {
    // workgroups per sequence: as many rounds as the chip needs times blocks per workgroup, plus
    // about one block's time for fetching the fragments
    const int slots = 256 * (rows_waves_per_simd<DH, NW, KT, LPL>() * 4 / NW);
    int64_t best = -1;
    for (int p = 1; p <= nblk; ++p) {
      const int64_t rounds = ((int64_t)s.S * p + slots - 1) / slots, cost = rounds * ((nblk + p - 1) / p + 1);
      if (best < 0 || cost < best) { best = cost; parts = p; }
    }
  }
  static bool attr_set = false;
  if (!attr_set) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(mha_rows_kernel<DH, NW, QT, KT, KG, LPL, BWD, STAT>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  mha_rows_kernel<DH, NW, QT, KT, KG, LPL, BWD, STAT><<<8 * parts * ((s.S + 7) / 8), NW * 64, lds, st>>>(
      R, G1, G2, idx, Ain, Wout, Out, maxes, s.S, s.n, s.L, s.scale, parts, kc);
  return hipGetLastError();
}

template <int LPL, bool BWD>
hipError_t rows_by_shape(const spt_mha_shape_t& s, const uint16_t* R, const uint16_t* G1, const uint16_t* G2,
                         const int32_t* idx, const float* Ain, float* Wout, uint16_t* Out, float2* maxes,
                         hipStream_t st) {
#define SPT_ROWS(DH, NW, QT, KT, KG, STAT) \
  return launch_rows<DH, NW, QT, KT, KG, LPL, BWD, STAT>(s, R, G1, G2, idx, Ain, Wout, Out, maxes, st)
  if (s.dh == 64) {
    if (s.n <= 256) SPT_ROWS(64, 8, 1, 1, 4, true);
    if (s.n <= 512) SPT_ROWS(64, 8, 1, 2, 4, true);
    SPT_ROWS(64, 8, 1, 2, 4, false);
  }
  if (s.n <= 256) SPT_ROWS(128, 8, 1, 1, 2, true);
  if (s.n <= 512) SPT_ROWS(128, 8, 1, 2, 4, true);
  SPT_ROWS(128, 8, 1, 2, 4, false);
#undef SPT_ROWS
}

template <bool BWD>
hipError_t rows_by_length(const spt_mha_shape_t& s, const void* R, const void* G1, const void* G2, const int32_t* idx,
                          const float* Ain, float* Wout, void* Out, float2* maxes, hipStream_t st) {
  const uint16_t *r = static_cast<const uint16_t*>(R), *g1 = static_cast<const uint16_t*>(G1), *g2 = static_cast<const uint16_t*>(G2);
  uint16_t* out = static_cast<uint16_t*>(Out);
  switch ((s.L + 63) / 64) {
    case 1: return rows_by_shape<1, BWD>(s, r, g1, g2, idx, Ain, Wout, out, maxes, st);
    case 2: return rows_by_shape<2, BWD>(s, r, g1, g2, idx, Ain, Wout, out, maxes, st);
    case 3: return rows_by_shape<3, BWD>(s, r, g1, g2, idx, Ain, Wout, out, maxes, st);
    default: return rows_by_shape<4, BWD>(s, r, g1, g2, idx, Ain, Wout, out, maxes, st);
  }
}

template <int DH, int LPL>
hipError_t launch_keys_t(const spt_mha_shape_t& s, const uint16_t* Q, const uint16_t* dY, const int32_t* idx,
                         const float* A, const float* dS, const float2* maxes, uint16_t* dK, uint16_t* dV,
                         hipStream_t st) {
  const size_t lds = 2 * KV_TS * 4 + 2 * KV_Q * DH * 2;
  static bool attr_set = false;
  if (!attr_set) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(mha_keys_kernel<DH, LPL>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  const int parts = (s.n + KV_KEYS - 1) / KV_KEYS;
  mha_keys_kernel<DH, LPL><<<8 * parts * ((s.S + 7) / 8), DH * 8, lds, st>>>(Q, dY, idx, A, dS, maxes, dK, dV, s.S, s.n,
                                                                         s.L, parts);
  return hipGetLastError();
}

}  // namespace

hipError_t mha_dense_fwd(const spt_mha_shape_t& s, const void* Q, const void* K, const void* V, const int32_t* idx,
                         float* A, void* Y, hipStream_t st) {
  return rows_by_length<false>(s, Q, K, V, idx, nullptr, A, Y, nullptr, st);
}

hipError_t mha_dense_bwd_q(const spt_mha_shape_t& s, const void* K, const void* V, const void* dY, const int32_t* idx,
                           const float* A, float* dS, float2* maxes, void* dQ, hipStream_t st) {
  return rows_by_length<true>(s, dY, V, K, idx, A, dS, dQ, maxes, st);
}

hipError_t mha_dense_bwd_kv(const spt_mha_shape_t& s, const void* Q, const void* dY, const int32_t* idx,
                            const float* A, const float* dS, const float2* maxes, void* dK, void* dV, hipStream_t st) {
  const uint16_t *q = static_cast<const uint16_t*>(Q), *dy = static_cast<const uint16_t*>(dY);
  uint16_t *dk = static_cast<uint16_t*>(dK), *dv = static_cast<uint16_t*>(dV);
#define SPT_KEYS(LPL)                                                              \
  (s.dh == 64 ? launch_keys_t<64, LPL>(s, q, dy, idx, A, dS, maxes, dk, dv, st)    \
              : launch_keys_t<128, LPL>(s, q, dy, idx, A, dS, maxes, dk, dv, st))
  switch ((s.L + 63) / 64) {
    case 1: return SPT_KEYS(1);
    case 2: return SPT_KEYS(2);
    case 3: return SPT_KEYS(3);
    default: return SPT_KEYS(4);
  }
#undef SPT_KEYS
}

}  // namespace spt
