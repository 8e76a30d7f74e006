// Sparse attention of section 4.1 (SDDMM, softmax over the kept keys, SpMM and their derivative) on
// the matrix cores.
//
// A query keeps L of n keys, L / n about 1/8.  Gathered row by row (mha.hip) the products run on
// the vector units at 128-256 bytes of LDS per multiply-add pair; as dense tiles they are n / L
// times the multiply-adds on units sixteen times as fast, and every operand byte is shared by a
// 32 x 32 tile.  What stays sparse is what the method stores: the index lists, A and dS.  Between
// the two a tile of one query block lives in LDS:
//
//   rows kernel (query side)    S = R G1^T for a block of queries (bf16 MFMA, fp32) -> tile; every
//     list entry gathers its word; softmax (forward) or its Jacobian (backward) over the list;
//     the weights go back to the same words, all other words are zero; Out = tile x G2.
//     forward (R, G1, G2) = (Q, K, V): A, Y.   backward (dY, V, K): dS, dQ.
//   keys kernel (backward)      the lists of a block of queries are scattered into two tiles
//     (A, dS) of 256 keys; dV += A^T dY, dK += dS^T Q stay in accumulators over all queries.  No
//     transposed lists, no atomics: the sum order is the query order.
//
// Precision.  Weights (A, dS) are fp32, in the lists and in the tiles.  As MFMA operands each is three
// bf16 numbers, its leading 8 bits, the next 8 and the last 8 (split_bf16x3): their sum is the weight
// itself, whatever its size (below 2^-110, where the last part leaves bf16's denormals, which the matrix
// cores keep, it is off by less than 2^-133).  The other operand (V, K, dY, Q) is bf16 as stored, so every product
// is exact and the sums are fp32, as with one fused multiply-add per kept key.  (Two fp16 halves under a
// common scale are a product in three less -- 104 / 105 / 110 us for the three launches of 64-wide heads below,
// where these take 127 / 122 / 129 -- but lose what is small beside the largest weight or value.)
//
// Infinities and NaN.  A dense tile multiplies every key of the sequence with a weight, zero where the query
// does not keep it, and 0 x inf is NaN.  So both kernels look for such values while they stage their operands.  A
// wavefront's four queries that meet any are summed over their kept entries alone (rows kernel); a step multiplies
// zeros in their place, and the terms that hold one are added to the rounded results at the end (keys kernel).  A query
// or key that nothing of the kind is kept with never sees it.
#include <math.h>
#include <type_traits>

#include "ffn_common.hpp"
#include "mha_host.hpp"

namespace spt {
namespace {

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

// Workgroup -> (sequence, part): the parts of a sequence run side by side on one XCD (sequence mod 8).
__device__ __forceinline__ bool seq_part(int parts, int S, int& s, int& part) {
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  s = (slot / parts) * 8 + xcd;
  part = slot % parts;
  return s < S;
}

// Largest magnitude of bf16 values (two per word), as bit patterns; kInf or more: an infinity or a NaN.
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
constexpr uint32_t kInf = 0x7F80u;
__device__ __forceinline__ u16x2 max_mag(u16x2 m, const u32x4& v) {
#pragma unroll
  for (int e = 0; e < 4; ++e) m = __builtin_elementwise_max(m, __builtin_bit_cast(u16x2, v[e] & 0x7FFF7FFFu));
  return m;
}
__device__ __forceinline__ bool not_finite(u16x2 m) { return max((uint32_t)m[0], (uint32_t)m[1]) >= kInf; }
__device__ __forceinline__ bool not_finite(float x) { return (__float_as_uint(x) & 0x7FFFFFFFu) >= 0x7F800000u; }
// Largest of m, |x| and |y|, NaN left out.
__device__ __forceinline__ float max_mag(float m, float x, float y) {
  asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(m) : "v"(x), "v"(y));
  return m;
}

// One weight on its way to the tile: the first two parts in a word, the third for itself.
__device__ __forceinline__ float split_weight(float w, uint16_t& third) {
  const float r = less_upper_half(w);
  third = (uint16_t)(__float_as_uint(less_upper_half(r)) >> 16);
  return __uint_as_float(__builtin_amdgcn_perm(__float_as_uint(w), __float_as_uint(r), 0x07060302u));
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
// Rows kernel.  NW = 8 wavefronts, BQ = 32 queries per block, KC = 32 KT NW keys per chunk.
//   S phase: wavefront w multiplies its KT tiles of 32 keys (fragments in registers) with the query tile;
//            MFMA rows = keys (rho32), so a lane writes 16 adjacent words of ITS query.
//   lists:   16 lanes per query, four adjacent entries per lane and vector; rows 4w .. 4w+3 of the
//            tile belong to wavefront w from the gather to the scatter, so no barrier inside.
//   PV:      wavefront = (key group: every KG-th K-step of 16 keys) x (column group of CT 32-column tiles),
//            G2 fragments in registers; the key groups' partial products are added through LDS in
//            group order.
// STAT: the sequence is one chunk, G1 and G2 fragments stay in registers for all of the
// workgroup's query blocks.  Otherwise a workgroup does one block and walks the keys twice: in chunks of kc for the
// scores, the next chunk's G1 fragments requested a gather ahead, and in chunks of PC for the second product, whose
// rows of G2 are copied into LDS behind the tile of weights while the chunk before is multiplied.  Two of these workgroups share a
// CU, so LDS (80 KiB each) sets PC, and 128 registers per lane kc.
// PLANES: an entry is split on its way into the tile, a word with the first two parts and a plane of halves with
// the third (6 bytes per key and query).  Else the tile holds the weights and what the products read is split, n / L
// times as many: cheaper only where the larger tile would cost the second workgroup of the CU (64-wide heads, 512 keys).
// 128-wide heads, 512 keys: 219 / 214 us splitting behind the tile, 211 / 205 in front of it.
// No unit is saturated: at 64-wide heads, 512 keys, the vector units issue in 60 % of the cycles, LDS is active in as many,
// the matrix cores in 24 %; what remains are the waits between the phases of a block.
// us, forward / backward, S 512, n 512, L 64: 127 / 122 (64-wide heads), 211 / 205 (128).  Several chunks, with one workgroup per CU
// and G2 fetched between barriers -> this: S 96, n 1100, L 137, 128-wide 398 / 396 -> 242 / 244; S 160, n 600, L 90
// 223 / 218 -> 131 / 131; S 32, n 2048, L 256 374 / 388 -> 341 / 268; 64-wide, S 256, n 600, L 90 159 / 161 -> 148 / 148; S 64,
// n 1024, L 200 92 / 132 -> 92 / 91; S 32, n 2048, L 256 174 / 234 -> 149 / 147.  (128-wide with 512 keys per chunk of scores and
// the fragments of one tile fetched behind the other's products: 262 / 265 where 242 / 244 is; a barrier more, to start the
// copies before the scatter: 266 / 266; 64-wide with 256 keys per chunk of scores 184 / 182 where 149 / 147 is.)
// 64-wide heads of several chunks: eight key groups, each wavefront both column tiles, so a weight is split once and not by two
// column groups (the vector units' largest part); forward, four groups -> eight: S 32, n 2048, L 256 139 -> 129; S 64, n 1024, L 200
// 81 -> 77; S 256, n 600, L 90 131 -> 127; backward 138 -> 130, 82 -> 79, 135 -> 132; few entries gain nothing: n 768, L 48 49 / 47 both, n 700, L 8 50
// both, 47 -> 48 backward.  With one chunk the second accumulator spills and nothing is gained (121 / 122); 128-wide
// heads with four groups and chunks of 128 keys spill: 241 -> 314 at S 96, n 1100, L 137.
constexpr int NW = 8, BQ = 32, NT = NW * 64;
template <int DH, int KT>
constexpr bool rows_planes() { return DH == 128 || KT == 1; }
// Registers: 128 per lane (two workgroups on a CU) where that holds the fragments and the lists, 256 otherwise.  Where it
// does not quite: 64-wide heads, 257 to 512 keys, 65 to 128 entries, backward keep one K fragment in scratch, read back once per
// block; 128-wide heads beyond 512 keys with more than 192 entries keep 12 (backward 13) registers of the lists there, stored
// once per block and read back once per chunk of the second product.  No other variant spills.
template <int DH, int KT, int LPL, bool STAT>
constexpr int rows_waves_per_simd() { return !STAT || (KT * DH <= 128 && LPL <= 2) ? 4 : 2; }
// Keys of a chunk of the second product where a sequence takes several: what two workgroups of a CU have LDS for.
template <int DH>
constexpr int rows_pv_keys() { return DH == 128 ? 160 : 256; }

template <int DH, int KT, int KG, int LPL, bool BWD, bool STAT>
__global__ __launch_bounds__(NT, (rows_waves_per_simd<DH, KT, LPL, STAT>())) void mha_rows_kernel(
    const uint16_t* __restrict__ R, const uint16_t* __restrict__ G1, const uint16_t* __restrict__ G2,
    const int32_t* __restrict__ idx, const float* __restrict__ Ain, float* __restrict__ Wout,
    uint16_t* __restrict__ Out, int S, int n, int L, float scale, int parts, int kc) {
  constexpr int KS = DH / 16, CG = NW / KG, CT = DH / 32 / CG;
  constexpr int PC = rows_pv_keys<DH>();                   // keys of a chunk of the second product (!STAT)
  constexpr int VS = (STAT ? NW * KT * 32 : PC) / 16 / KG; // K-steps of 16 keys of a wavefront: kg, kg + KG, ...
  constexpr int RSTRIDE = DH * 2 + 16;
  constexpr bool PLANES = rows_planes<DH, KT>();
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
  const int ts = STAT && PLANES ? kc + kc / 2 + 4 : kc + 4;   // words per tile row
  const int pk = STAT ? kc : PC, ps = PLANES ? pk + pk / 2 + 4 : pk + 4;   // keys and words per row of the tile of weights
  float* tile = reinterpret_cast<float*>(smem);
  const uint32_t vlds = BQ * ps * 4;                       // !STAT: a chunk of G2 behind the tile of weights
  const int tile_bytes = STAT ? max(BQ * ts * 4, max(KG * BQ * DH * 4, kc * DH * 2))
                              : max(max(BQ * ts * 4, KG * BQ * DH * 4), (int)vlds + PC * DH * 2);
  char* rlds = smem + tile_bytes;                          // [BQ] rows of R
  uint32_t* bad = reinterpret_cast<uint32_t*>(rlds + BQ * RSTRIDE);   // [NW] a wavefront has staged an infinity or a NaN
  uint32_t* done = bad + NW;                               // [NW] the wavefront's four queries are written already
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
  // (!STAT: four lanes in a row, which want four rows, request 64 adjacent bytes of each of them in turn and exchange the 16-byte pieces
  // afterwards: pieces of one line that four such lanes ask for cost a quarter of pieces of four lines.  us, forward / backward, before and now: S 96,
  // n 1100, L 137, 128-wide 251 / 255, 234 / 238; S 64, n 1024, L 200, 64-wide 85 / 84, 81 / 79.  128-wide heads exchange in front of the products, 64-wide
  // ones at once: the other way round 239 / 242 and 84 / 84.)
  auto order_k = [&](int from, int to) {
#pragma unroll
    for (int t = from; t < to; ++t)
#pragma unroll
      for (int k = 0; k < KS; k += 4) quad_transpose(&kf[t][k], lane);
  };
  auto load_k = [&](uint32_t c0) {
#pragma unroll
    for (int t = 0; t < KT; ++t)
#pragma unroll
      for (int k = 0; k < KS; ++k) {
        // (padding keys: any row, their words are never read)
        const uint32_t row = STAT ? i : (i & ~3u) + k % 4, piece = STAT ? (uint32_t)k : k / 4 * 4 + (lane & 3);
        const uint32_t key = min(c0 + (wave * KT + t) * 32 + rho32(row), (uint32_t)n - 1);
        kf[t][k] = as_bf16x8(load_at<u32x4>(g1, key * (DH * 2) + h * DH + piece * 16));
      }
    if (!STAT && DH == 64) order_k(0, KT);
  };
  // G2 rows c0 .. c0 + kc of the sequence into the tile's space; `mag`: largest magnitude so far.
  u16x2 mag = {0, 0};
  auto stage_v = [&](uint32_t c0) {
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
  auto any_bad = [&]() -> bool {                            // (after a barrier behind the stores)
    uint32_t m = 0u;
#pragma unroll
    for (int w = 0; w < NW; ++w) m |= bad[w];
    return __builtin_amdgcn_readfirstlane(m) != 0u;
  };
  bf16x8 vf[VS][CT];
  auto read_v = [&]() {
#pragma unroll
    for (int k = 0; k < VS; ++k) {
      const uint32_t row0 = 16 * (kg + KG * k);
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        vf[k][ct] = as_bf16x8(u32x4{0u, 0u, 0u, 0u});
        if (!STAT) vf[k][ct] = as_bf16x8(tr_frag<DH>(smem + vlds + row0 * (DH * 2) + vtr[ct]));
        else if (row0 < (uint32_t)kc) vf[k][ct] = as_bf16x8(tr_frag<DH>(smem + row0 * (DH * 2) + vtr[ct]));
      }
    }
  };

  // !STAT: rows c0 .. c0 + PC of G2 on their way into LDS (rows past the end: the last one); they are looked at for
  // infinities and NaN as fragments.
  auto fetch_v = [&](int c0) {
    constexpr int RI = 1024 / (DH * 2);                     // rows of a copy instruction
#pragma unroll
    for (int j = 0; j < PC / RI / NW; ++j) {
      const uint32_t row0 = (wave * (PC / RI / NW) + j) * RI, r = row0 + lane / (DH / 8);
      const uint32_t row = min((uint32_t)c0 + r, (uint32_t)n - 1);
      dma16(reinterpret_cast<const char*>(g2) + row * (DH * 2) + ((lane % (DH / 8)) ^ chunk_swizzle<DH>(r)) * 16,
            __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)smem + vlds + row0 * (DH * 2)));
    }
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
  float aa[LPL][4], w[LPL][4];
  auto request_lists = [&](int b) {
    const uint32_t row = row_bytes(b);
#pragma unroll
    for (int v = 0; v < LPL; ++v) {
      const u32x4 x = load_at<u32x4u>(idx, row + at(v) * 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) jj[v][e] = (int)x[e];
    }
  };
  auto request_a = [&](int b) {
    const uint32_t row = row_bytes(b);
#pragma unroll
    for (int v = 0; v < LPL; ++v) {
      const f32x4 y = load_at<f32x4u>(Ain, row + at(v) * 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) aa[v][e] = y[e];
    }
  };

  // The rows of Out of this wavefront's queries as sums over their kept entries (see the top).
  auto sum_kept = [&](int b) {
    constexpr int C = DH / 16;                              // columns per lane
    float o[C] = {};
    const uint32_t list = row_bytes(b);
#pragma unroll
    for (int v = 0; v < LPL; ++v) {
      const f32x4 wv = load_at<f32x4u>(Wout, list + at(v) * 4);   // (this lane's own stores)
#pragma unroll 1
      for (uint32_t l = 0; l < 16; ++l) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int src = (int)((lane & 48) + l);
          const uint32_t j = (uint32_t)__shfl(jj[v][e], src), first = 64u * v + 4 * l;
          const bool kept = j < (uint32_t)n && min(first, (uint32_t)L - 4) + e >= first;
          const float got = __shfl(wv[e], src), we = kept ? got : 0.f;
          const uint32_t from = (kept ? j : 0u) * (DH * 2) + (lane & 15) * (C * 2);
#pragma unroll
          for (int x = 0; x < C; x += 2) {
            const uint32_t y = kept ? load_at<uint32_t>(g2, from + x * 2) : 0u;
            o[x] = fmaf(we, lo_bf16(y), o[x]);
            o[x + 1] = fmaf(we, hi_bf16(y), o[x + 1]);
          }
        }
      }
    }
    const uint32_t q = b * BQ + ql;
    if (q < (uint32_t)n)
#pragma unroll
      for (int x = 0; x < C; x += 2) store_at<uint32_t>(Out, q * (DH * 2) + ((lane & 15) * C + x) * 2, pack_bf16x2(o[x], o[x + 1]));
  };

  // ---- once per workgroup
  bool g2_bad = false;
  if (STAT) {
    stage_v(0);
    const bool mine = __any(not_finite(mag));
    if (lane == 0) bad[wave] = mine;
    __syncthreads();
    g2_bad = any_bad();
    read_v();
    __syncthreads();
  }
  int b = part;
  if (b < nblk) { request_r(b); request_lists(b); load_k(0); store_r(); }
  __syncthreads();

  for (; b < nblk; b += parts) {
    fresh_roles();
    if (BWD && STAT) request_a(b);
    for (int c = 0; c < (STAT ? 1 : nch); ++c) {
      const int c0 = c * kc;
#pragma unroll
      for (int t = 0; t < KT; ++t) {
        if ((wave * KT + t) * 32 >= (uint32_t)kc) continue;          // uniform
        f32x16 acc;
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] = 0.f;
        if (!STAT && DH == 128) order_k(t, t + 1);
#pragma unroll
        for (int k = 0; k < KS; ++k) {
          const bf16x8 rf = as_bf16x8(*reinterpret_cast<const u32x4*>(rlds + i * RSTRIDE + h * DH + k * 16));
          acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[t][k], rf, acc, 0, 0, 0);
          if (!STAT && DH == 128 && LPL > 2 && k == KS / 2 - 1) __builtin_amdgcn_sched_barrier(0);   // (half of R's fragments at a time: registers)
        }
        f32x4* dst = reinterpret_cast<f32x4*>(tile + i * ts + (wave * KT + t) * 32 + 16 * h);
#pragma unroll
        for (int e = 0; e < 4; ++e) dst[e] = f32x4{acc[4 * e], acc[4 * e + 1], acc[4 * e + 2], acc[4 * e + 3]};
        __builtin_amdgcn_sched_barrier(0);                 // (one tile's fragments at a time: registers)
      }
      if (!STAT && c + 1 < nch) load_k(c0 + kc);
      __syncthreads();
      const float* trow = tile + ql * ts;
#pragma unroll
      for (int v = 0; v < LPL; ++v) {
        bool in[4];
        float got[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t jl = (uint32_t)(jj[v][e] - c0);
          in[e] = jl < (uint32_t)min(kc, n - c0);
          got[e] = trow[in[e] ? jl : 0u];
        }
        // (opaque: left to itself the compiler reads each word of a later chunk behind a branch, one LDS latency per entry)
        if (!STAT) asm volatile("" : "+v"(got[0]), "+v"(got[1]), "+v"(got[2]), "+v"(got[3]));
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if (STAT) w[v][e] = got[e];
          else w[v][e] = in[e] ? got[e] : (c == 0 ? 0.f : w[v][e]);
        }
      }
      if (!STAT) __syncthreads();
    }
    if (BWD && !STAT) request_a(b);
    if (!STAT) fetch_v(0);
    // ---- softmax / Jacobian over the list, in registers
    bool ok[LPL][4], own[LPL][4];
#pragma unroll
    for (int v = 0; v < LPL; ++v)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        ok[v][e] = (uint32_t)jj[v][e] < (uint32_t)n;        // -1 = no key; out of range alike
        own[v][e] = at(v) + e >= 64u * v + e4;
      }
    bool w_bad = false;                                     // an infinite weight
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
    } else {
      float sum = 0.f;
      float wmag = 0.f;
#pragma unroll
      for (int v = 0; v < LPL; ++v)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          aa[v][e] = ok[v][e] ? aa[v][e] : 0.f;
          sum = fmaf(own[v][e] ? aa[v][e] : 0.f, ok[v][e] ? w[v][e] : 0.f, sum);
        }
      sum = row_sum(sum);
#pragma unroll
      for (int v = 0; v < LPL; ++v)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          w[v][e] = ok[v][e] ? aa[v][e] * (w[v][e] - sum) * scale : 0.f;
          if (e % 2 == 1) wmag = max_mag(wmag, w[v][e - 1], w[v][e]);
        }
      w_bad = not_finite(wmag);
    }
    {
      const uint32_t row = row_bytes(b);
#pragma unroll
      for (int v = 0; v < LPL; ++v)
        store_at<f32x4u>(Wout, row + at(v) * 4, f32x4{w[v][0], w[v][1], w[v][2], w[v][3]});
    }
    uint32_t third[LPL][2];                                 // PLANES: w holds the first two parts of a weight from here on
    if (PLANES) {
#pragma unroll
      for (int v = 0; v < LPL; ++v)
#pragma unroll
        for (int e = 0; e < 4; e += 2) {
          uint16_t t0, t1;
          w[v][e] = split_weight(w[v][e], t0);
          w[v][e + 1] = split_weight(w[v][e + 1], t1);
          third[v][e / 2] = t0 | (uint32_t)t1 << 16;
        }
    }

    // ---- Out = tile x G2
    f32x16 acc[CT];
    auto clear_acc = [&]() {
#pragma unroll
      for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[ct][v] = 0.f;
    };
    if (!STAT) clear_acc();
    for (int c = 0; c < (STAT ? 1 : (n + PC - 1) / PC); ++c) {
      const int c0 = c * PC;
      const bool last_chunk = STAT || c0 + PC >= n;
      if (!STAT) {
        wait_vmcnt<0>();
        __syncthreads();                                    // the chunk of G2 is there, the tile of weights has been read
        read_v();
#pragma unroll
        for (int k = 0; k < VS; ++k)
#pragma unroll
          for (int ct = 0; ct < CT; ++ct) mag = max_mag(mag, __builtin_bit_cast(u32x4, vf[k][ct]));
        if (last_chunk) {
          const bool mine = __any(not_finite(mag));
          if (lane == 0) bad[wave] = mine;
        }
      }
      // this wavefront's four rows: cleared, then the list entries
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        uint4* dst = reinterpret_cast<uint4*>(tile + (4 * wave + r) * ps);
        for (uint32_t e = lane; e < (uint32_t)(ps - 4) / 4; e += 64) dst[e] = make_uint4(0u, 0u, 0u, 0u);
      }
      wave_lds_fence();
      float* trow = tile + ql * ps;
#pragma unroll
      for (int v = 0; v < LPL; ++v)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t jl = (uint32_t)(jj[v][e] - c0);
          if (jl < (uint32_t)min(pk, n - c0)) {
            trow[jl] = w[v][e];
            if (PLANES) reinterpret_cast<uint16_t*>(trow + pk)[jl] = (uint16_t)(third[v][e / 2] >> (e % 2 * 16));
          }
        }
      auto finish_slow = [&]() {
        const bool slow = g2_bad || (BWD && __any(w_bad));   // uniform over the wavefront
        if (slow) sum_kept(b);
        if (lane == 0) done[wave] = slow;
      };
      if (STAT) finish_slow();
      if (STAT && b + parts < nblk) request_r(b + parts);
      __syncthreads();
      fresh_roles();
      if (!STAT && !last_chunk) fetch_v(c0 + PC);
      if (!STAT && last_chunk) {
        g2_bad = any_bad();
        finish_slow();
      }
      if (STAT) clear_acc();
#pragma unroll
      for (int k = 0; k < VS; ++k) {
        const uint32_t k0 = 16 * (kg + KG * k);
        if (STAT && k0 >= (uint32_t)kc) continue;           // uniform
        const float* row = tile + i * ps + k0 + 8 * h;
        const u32x4* src = reinterpret_cast<const u32x4*>(row);
        bf16x8 hi, mid, lo;
        if (PLANES) {
          hi = upper_halves(src[0], src[1]);
          mid = lower_halves(src[0], src[1]);
          lo = as_bf16x8(*reinterpret_cast<const u32x4*>(row + pk - (k0 + 8 * h) / 2));
        } else {
          split_bf16x3(src[0], src[1], hi, mid, lo);
        }
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
          acc[ct] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[k][ct], hi, acc[ct], 0, 0, 0);
          acc[ct] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[k][ct], mid, acc[ct], 0, 0, 0);
          acc[ct] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[k][ct], lo, acc[ct], 0, 0, 0);
        }
      }
    }
    __syncthreads();
    // ---- partial products [group][query][DH], 16-byte chunks permuted by query
    fresh_roles();
    const uint32_t groups = STAT ? min(KG, kc / 16) : KG;
    float* partial = reinterpret_cast<float*>(smem);
    constexpr int PC = DH / 4;                              // 16-byte chunks per row
    if (kg < groups) {
#pragma unroll
      for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t ch = ((cg * CT + ct) * 8 + 4 * h + e) ^ (i & 15);
          const f32x16& a = acc[ct];
          *reinterpret_cast<f32x4*>(partial + ((size_t)kg * BQ + i) * DH + ch * 4) =
              f32x4{a[4 * e], a[4 * e + 1], a[4 * e + 2], a[4 * e + 3]};
        }
    }
    if (STAT && b + parts < nblk) { store_r(); request_lists(b + parts); }
    __syncthreads();
    for (uint32_t it = tid; it < BQ * PC; it += NT) {
      const uint32_t r = it / PC, ch = it % PC;
      const float* p = partial + (size_t)r * DH + (ch ^ (r & 15)) * 4;
      f32x4 sum = *reinterpret_cast<const f32x4*>(p);
      for (uint32_t gidx = 1; gidx < groups; ++gidx) sum += *reinterpret_cast<const f32x4*>(p + (size_t)gidx * BQ * DH);
      if (b * BQ + r < (uint32_t)n && !done[r / 4])
        store_at<uint2>(Out, (b * BQ + r) * (DH * 2) + ch * 8,
                        make_uint2(pack_bf16x2(sum[0], sum[1]), pack_bf16x2(sum[2], sum[3])));
    }
    if (!STAT) break;                                       // (one block per workgroup)
    __syncthreads();
  }
}

// ------------------------------------------------------------------------------------------
// Keys kernel: dV = A^T dY, dK = dS^T Q for 256 keys of a sequence, 32 queries per step.  A wavefront
// owns 64 keys and all columns of one of the two gradients in accumulators (64-wide heads: two workgroups per CU,
// up to 128 entries; one otherwise).  The A and dS words of a step are scattered
// into two LDS tiles [key][query] and taken out again afterwards (only the words that were set), by
// the wavefront that owns the query.  Entries whose key is another workgroup's go to dummy words behind the tile.
// One pair of tiles: scatter, barrier, products, barrier; the matrix cores stand still while the lists are scattered, unless
// another workgroup of the CU has products to do.  Where there is one workgroup per CU and the lists have more than 64 entries, so that
// the scatter is a good part of a step, there are two pairs (keys_two_tiles): the lists of the next step go out among the products of
// this one.  us, one pair and two: 128-wide heads, S 96, n 1100, L 137 267 -> 241; S 128, n 384, L 100 48 -> 44; 64-wide, S 192, n 700, L 170
// 219 -> 198; not where a list is one vector: 128-wide, S 512, n 512, L 64 228 -> 238 (twice the tiles to clear before 16 steps).
// 16-byte chunk c of tile row r sits at c ^ ((r >> 1) & 7): the 16 rows of a pass hit all banks.
// What the products read is split into its three parts here: split in front of the tile (one gradient per workgroup, or the
// tiles would not fit) the scatter, which is what a step waits for, has half as much again to do: 129 -> 166 us at 64-wide
// heads, S 512, n 512, L 64, 259 -> 575 at 128-wide, n 1100, L 137.  128-wide heads on 16 wavefronts of 64 columns
// split every word twice: 255 us against 227 (n 512), 270 against 259 (n 1100).  The words of the next quarter are read in front
// of the products of this one where registers allow, and a part of the weights goes through all column tiles before the next part
// does: no product waits for the one in front of it (128-wide heads, L 64: 706 -> 697 us a training pass; L 240 572 -> 556).
constexpr int KV_KEYS = 256, KV_Q = 32;
constexpr int KV_TILE = KV_KEYS * KV_Q;                    // words
constexpr int KV_TS = KV_TILE + 64;                        // ... and the 64 dummy words behind them
constexpr int KV_FLAGS = 16;                               // bytes
template <int DH, int LPL>
constexpr bool keys_two_tiles() { return LPL > 2 || (DH == 128 && LPL == 2); }
template <int DH, int LPL>
__global__ __launch_bounds__(NT, DH == 64 && LPL <= 2 ? 4 : 2) void mha_keys_kernel(
    const uint16_t* __restrict__ Q, const uint16_t* __restrict__ dY, const int32_t* __restrict__ idx,
    const float* __restrict__ A, const float* __restrict__ dS, uint16_t* __restrict__ dK,
    uint16_t* __restrict__ dV, int S, int n, int L, int parts) {
  constexpr int NC = DH / 8, CT = DH / 32;                 // 16-byte pieces and 32-column tiles of a row
  constexpr int QW = KV_Q / NW, EL = QW;                   // queries per wavefront; 64 / QW lanes x EL entries cover 64
  constexpr int ROWS = KV_Q * DH * 2;                      // bytes of a step's dY (then Q) rows
  constexpr int TILES = keys_two_tiles<DH, LPL>() ? 2 : 1;
  constexpr bool AHEAD = DH == 128 || TILES == 2;          // (registers)
  extern __shared__ uint4 kv_smem[];
  char* smem = reinterpret_cast<char*>(kv_smem);           // A tile, dS tile (of even steps, of odd ones), dY rows, Q rows
  char* rows = smem + TILES * 2 * KV_TS * 4;
  uint32_t* steps = reinterpret_cast<uint32_t*>(rows + 2 * ROWS);   // [4] a bit for every step (n <= 4096: at most 128) that meets an infinity or a NaN
  float* words = reinterpret_cast<float*>(smem);
  // (lane roles are formed again for every step from a value the compiler cannot follow, see the rows kernel)
  uint32_t tid = threadIdx.x, lane = tid & 63, i = lane & 31, h = lane >> 5;
  auto fresh_roles = [&]() {
    asm volatile("" : "+v"(tid));
    lane = tid & 63; i = lane & 31; h = lane >> 5;
  };
  const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t t = wave & 1, kg = wave >> 1;
  int s, part;
  if (!seq_part(parts, S, s, part)) return;
  const size_t base = (size_t)s * n;
  const int key0 = part * KV_KEYS;
  const uint16_t* src[2] = {dY + base * DH, Q + base * DH};
  idx += base * L;
  A += base * L;
  dS += base * L;

  for (uint32_t e = tid; e < TILES * 2 * KV_TS / 4; e += NT) reinterpret_cast<uint4*>(smem)[e] = make_uint4(0u, 0u, 0u, 0u);
  if (tid < 4) steps[tid] = 0u;
  __syncthreads();
  const uint32_t last = min(KV_KEYS, n - key0);

  // rows of a step: a thread copies RP 16-byte pieces, of the first half of the queries and of the second (DH 128) of
  // dY or of Q
  constexpr int RP = 2 * KV_Q * NC / NT, RQ = KV_Q / RP;
  const uint16_t* rsrc = tid / (NT / 2) ? src[1] : src[0];      // uniform over a wavefront
  auto row_dst = [&]() -> uint32_t {                        // (piece u: u RQ rows on, the same swizzle)
    const uint32_t pr = (tid / NC) % RQ, pc = tid % NC;
    return tid / (NT / 2) * ROWS + pr * (DH * 2) + (pc ^ chunk_swizzle<DH>(pr)) * 16;
  };
  u32x4 rnext[RP];
  auto request_rows = [&](int b) {                          // (rows past the end: the last one again)
#pragma unroll
    for (int u = 0; u < RP; ++u)
      rnext[u] = load_at<u32x4>(rsrc, min(b * KV_Q + u * RQ + (tid / NC) % RQ, (uint32_t)n - 1) * (DH * 2) + tid % NC * 16);
  };
  // lists: lane = (query QW wave + lane / (64 / QW), entries at(v) .. at(v) + EL - 1 of its row); lanes past
  // the row's end repeat its last entries (same word, same value)
  auto query = [&]() -> uint32_t { return QW * wave + lane / (64 / QW); };
  int jn[LPL][EL];
  float an[LPL][EL], dn[LPL][EL];
  auto request_lists = [&](int b, auto from, auto to) {     // vectors from .. to - 1
    const uint32_t row = min(b * KV_Q + query(), (uint32_t)n - 1) * (uint32_t)L * 4, el = EL * (lane % (64 / QW));
#pragma unroll
    for (int v = from; v < to; ++v) {
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
  uint32_t old[TILES][LPL][EL / 2];                        // the words this lane has set, two to a register
#pragma unroll
  for (int x = 0; x < TILES; ++x)
#pragma unroll
    for (int v = 0; v < LPL; ++v)
#pragma unroll
      for (int e = 0; e < EL / 2; ++e) old[x][v][e] = (KV_TILE + lane) * 0x10001u;
  auto clear = [&](float* words, uint32_t (&old)[LPL][EL / 2]) {
#pragma unroll
    for (int v = 0; v < LPL; ++v)
#pragma unroll
      for (int e = 0; e < EL; ++e) {
        const uint32_t at = e % 2 ? old[v][e / 2] >> 16 : old[v][e / 2] & 0xFFFFu;
        words[at] = 0.f;
        words[at + KV_TS] = 0.f;
      }
  };
  auto scatter = [&](int b, float* words, uint32_t (&old)[LPL][EL / 2], auto from, auto to) {   // entries from .. to - 1
    const uint32_t ql = query(), lim = b * KV_Q + ql < (uint32_t)n ? last : 0;   // queries past the end have no entries
#pragma unroll
    for (int x = from; x < to; ++x) {
      const int v = x / EL, e = x % EL;
      const uint32_t j = (uint32_t)(jn[v][e] - key0);
      const uint32_t at = j * KV_Q + (((ql >> 2) ^ ((j >> 1) & 7)) << 2) + (ql & 3);
      uint32_t to = KV_TILE + lane;
      to = j < lim ? at : to;
      words[to] = an[v][e];
      words[to + KV_TS] = dn[v][e];
      old[v][e / 2] = e % 2 ? old[v][e / 2] | to << 16 : to;
    }
  };
  // What is infinite or NaN in the rows of a step, or infinite among its weights, in the registers it has arrived in: zeros
  // are multiplied in its place, and the step is marked.  (A NaN weight reaches its own key only.)
  auto drop_not_finite = [&](int b) {
    float m = 0.f;
#pragma unroll
    for (int v = 0; v < LPL; ++v)
#pragma unroll
      for (int e = 0; e < EL; ++e) m = max_mag(m, an[v][e], dn[v][e]);
    u16x2 r = {0, 0};
#pragma unroll
    for (int u = 0; u < RP; ++u) r = max_mag(r, rnext[u]);
    if (!__any(not_finite(m) || not_finite(r))) return;
    if (lane == 0) atomicOr(steps + b / 32, 1u << (b % 32));
#pragma unroll
    for (int v = 0; v < LPL; ++v)
#pragma unroll
      for (int e = 0; e < EL; ++e) {
        an[v][e] = not_finite(an[v][e]) ? 0.f : an[v][e];
        dn[v][e] = not_finite(dn[v][e]) ? 0.f : dn[v][e];
      }
#pragma unroll
    for (int u = 0; u < RP; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if ((rnext[u][e] & kInf) == kInf) rnext[u][e] &= 0xFFFF0000u;
        if ((rnext[u][e] >> 16 & kInf) == kInf) rnext[u][e] &= 0xFFFFu;
      }
  };

  f32x16 acc[2][CT];                                       // [32-key tile][32-column tile]
#pragma unroll
  for (int kt = 0; kt < 2; ++kt)
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[kt][ct][v] = 0.f;

  const int nblk = (n + KV_Q - 1) / KV_Q;
  const std::integral_constant<int, 0> zero;
  const std::integral_constant<int, LPL> all;
  const std::integral_constant<int, LPL * EL> entries;
  auto store_rows = [&]() {
#pragma unroll
    for (int u = 0; u < RP; ++u) *reinterpret_cast<u32x4*>(rows + row_dst() + u * RQ * DH * 2) = rnext[u];
  };
  // The products of a step with this wavefront's 64 keys, `behind` what goes out behind each quarter of them.
  auto products = [&](const float* words, auto behind) {
    if (kg * 64 >= last) {                                 // uniform
      behind(0); behind(1); behind(2); behind(3);
      return;
    }
    fresh_roles();
    uint32_t vtr[CT], wrow[2];                             // fragments of the rows; this lane's key rows in its tensor's tile
#pragma unroll
    for (int x = 0; x < CT; ++x) vtr[x] = t * ROWS + tr_offset<DH>(lane, x);
#pragma unroll
    for (int x = 0; x < 2; ++x) wrow[x] = t * KV_TS + (kg * 64 + x * 32 + i) * KV_Q;
    const uint32_t wsw = (i >> 1) & 7;                     // (32 and 64 rows on: the same swizzle)
    u32x4 w[2];
    auto read_words = [&](int x) {                         // quarter x: keys 32 (x % 2) .., queries 16 (x / 2) ..
      const u32x4* trow = reinterpret_cast<const u32x4*>(words + wrow[x % 2]);
      w[0] = trow[(4 * (x / 2) + 2 * h) ^ wsw];
      w[1] = trow[(4 * (x / 2) + 2 * h + 1) ^ wsw];
    };
    if (AHEAD) read_words(0);
#pragma unroll
    for (int k = 0; k < KV_Q / 16; ++k) {
      bf16x8 rf[CT];
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) rf[ct] = as_bf16x8(tr_frag<DH>(rows + 16 * k * (DH * 2) + vtr[ct]));
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) {
        bf16x8 hi, mid, lo;
        if (!AHEAD) read_words(2 * k + kt);
        split_bf16x3(w[0], w[1], hi, mid, lo);
        if (AHEAD && k + kt < 2) read_words(2 * k + kt + 1);
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) acc[kt][ct] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(rf[ct], hi, acc[kt][ct], 0, 0, 0);
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) acc[kt][ct] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(rf[ct], mid, acc[kt][ct], 0, 0, 0);
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) acc[kt][ct] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(rf[ct], lo, acc[kt][ct], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);                 // (one key tile's fragments at a time: registers)
        behind(2 * k + kt);
      }
    }
  };
  request_rows(0);
  request_lists(0, zero, all);
  if constexpr (TILES == 2) {
    // The lists of the next step go into the other pair of tiles among the products of this one; its rows, into the one place
    // for them, between two barriers.  64-wide heads, with half of the products, look at the lists behind the first half of them and ask for those of the step after
    // as soon as all words are out: looked at in front and asked for behind the third quarter, as 128-wide heads do, they are waited for where long
    // lists come from memory.  us, one pair / so / this: S 156, n 1500, L 140 527 / 550 / 502; S 120, n 2048, L 130 703 / 735 / 670; S 192, n 700, L 170
    // 219 / 217 / 198; 128-wide, S 96, n 1100, L 137 256 / 230, looked at later 238.
    const std::integral_constant<int, LPL * EL / 2> half;
    drop_not_finite(0);
    scatter(0, words, old[0], zero, entries);
    store_rows();
    request_rows(1);
    request_lists(1, zero, all);
    __syncthreads();
    auto step = [&](int b, const float* from, float* into, uint32_t (&old)[LPL][EL / 2]) {
      fresh_roles();
      if (DH == 128 && b + 1 < nblk) drop_not_finite(b + 1);
      products(from, [&](int quarter) {
        if (quarter == 0) clear(into, old);
        if (quarter == 1) {
          if (DH == 64 && b + 1 < nblk) drop_not_finite(b + 1);
          scatter(b + 1, into, old, zero, half);
        }
        if (quarter == (DH == 64 ? 1 : 2)) {
          scatter(b + 1, into, old, half, entries);
          request_lists(b + 2, zero, all);
        }
      });
      __syncthreads();
      store_rows();
      request_rows(b + 2);
      __syncthreads();
    };
    for (int b = 0; b < nblk; b += 2) {
      step(b, words, words + 2 * KV_TS, old[1]);
      if (b + 1 < nblk) step(b + 1, words + 2 * KV_TS, words, old[0]);
    }
  } else {
    // vectors requested ahead of the products; the others, where registers for them are lacking, behind
    const std::integral_constant<int, LPL == 2 ? 1 : LPL> early;
    for (int b = 0; b < nblk; ++b) {
      fresh_roles();
      drop_not_finite(b);
      clear(words, old[0]);
      scatter(b, words, old[0], zero, entries);
      store_rows();
      request_rows(b + 1);
      request_lists(b + 1, zero, early);
      __syncthreads();
      products(words, [](int) {});
      request_lists(b + 1, early, all);
      __syncthreads();
    }
  }
#pragma unroll
  for (int kt = 0; kt < 2; ++kt) {
    const uint32_t krow = kg * 64 + kt * 32 + i;
    if (krow >= last) continue;
    uint16_t* out = (t ? dK : dV) + (base + key0 + krow) * DH + 16 * h;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      const f32x16& a = acc[kt][ct];
      uint32_t p[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) p[e] = pack_bf16x2(a[2 * e], a[2 * e + 1]);
      reinterpret_cast<uint4*>(out + ct * 32)[0] = make_uint4(p[0], p[1], p[2], p[3]);
      reinterpret_cast<uint4*>(out + ct * 32)[1] = make_uint4(p[4], p[5], p[6], p[7]);
    }
  }
  // What the products left out: the terms with an infinity or a NaN, entry by entry of the steps that have any.  They
  // make the sum infinite or NaN in any order, so they are added to the rounded results.
  __syncthreads();
  for (int b = 0; b < nblk; ++b) {
    if (!(steps[b / 32] >> (b % 32) & 1u)) continue;        // uniform
#pragma unroll 1
    for (int q = b * KV_Q; q < min((b + 1) * KV_Q, n); ++q) {
#pragma unroll 1
      for (uint32_t l = tid / NC; l < (uint32_t)L; l += NT / NC) {
        const uint32_t at = ((uint32_t)q * L + l) * 4, j = load_at<uint32_t>(idx, at) - key0;
        if (j >= last) continue;
#pragma unroll 1
        for (int y = 0; y < 2; ++y) {
          const float wt = load_at<float>(y ? dS : A, at);
          const u32x4 x = load_at<u32x4>(src[y], (uint32_t)q * (DH * 2) + (tid % NC) * 16);
          const bool all = not_finite(wt);
          if (!all && !not_finite(max_mag(u16x2{0, 0}, x))) continue;
          u32x4* out = reinterpret_cast<u32x4*>((y ? dK : dV) + (base + key0 + j) * DH) + tid % NC;
          u32x4 o = *out;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float lo = all || (x[e] & kInf) == kInf ? lo_bf16(o[e]) + wt * lo_bf16(x[e]) : lo_bf16(o[e]);
            const float hi = all || (x[e] >> 16 & kInf) == kInf ? hi_bf16(o[e]) + wt * hi_bf16(x[e]) : hi_bf16(o[e]);
            o[e] = pack_bf16x2(lo, hi);
          }
          *out = o;
        }
      }
      __syncthreads();                                      // (a key is kept once by a query, but by several)
    }
  }
}

// ------------------------------------------------------------------------------------------
// host side
template <int DH, int KT, int KG, int LPL, bool BWD, bool STAT>
hipError_t launch_rows(const spt_mha_shape_t& s, const uint16_t* R, const uint16_t* G1, const uint16_t* G2,
                       const int32_t* idx, const float* Ain, float* Wout, uint16_t* Out, hipStream_t st) {
  constexpr int KC = NW * KT * 32;
  // one chunk: the keys rounded up to a K-step of 16 per half wavefront tile; several: equal chunks
  const int nch = (s.n + KC - 1) / KC;
  const int kc = ((s.n + nch - 1) / nch + 31) / 32 * 32;
  constexpr int PC = rows_pv_keys<DH>();
  const size_t tile = (size_t)BQ * (kc + (STAT && rows_planes<DH, KT>() ? kc / 2 : 0) + 4) * 4, part = (size_t)KG * BQ * DH * 4;
  const size_t vrows = STAT ? (size_t)kc * DH * 2 : (size_t)BQ * (PC + (rows_planes<DH, KT>() ? PC / 2 : 0) + 4) * 4 + PC * DH * 2;
  size_t lds = tile > part ? tile : part;
  if (vrows > lds) lds = vrows;
  lds += (size_t)BQ * (DH * 2 + 16) + 2 * NW * 4;
  const int nblk = (s.n + BQ - 1) / BQ;
  int parts = nblk;
  if (STAT) {
    // workgroups per sequence: as many rounds as the chip needs times blocks per workgroup, plus
    // about one block's time for fetching the fragments
    const int slots = 256 * (rows_waves_per_simd<DH, KT, LPL, STAT>() * 4 / NW);
    int64_t best = -1;
    for (int p = 1; p <= nblk; ++p) {
      const int64_t rounds = ((int64_t)s.S * p + slots - 1) / slots, cost = rounds * ((nblk + p - 1) / p + 1);
      if (best < 0 || cost < best) { best = cost; parts = p; }
    }
  }
  static bool attr_set = false;
  if (!attr_set) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(mha_rows_kernel<DH, KT, KG, LPL, BWD, STAT>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  mha_rows_kernel<DH, KT, KG, LPL, BWD, STAT><<<8 * parts * ((s.S + 7) / 8), NW * 64, lds, st>>>(
      R, G1, G2, idx, Ain, Wout, Out, s.S, s.n, s.L, s.scale, parts, kc);
  return hipGetLastError();
}

template <int LPL, bool BWD>
hipError_t rows_by_shape(const spt_mha_shape_t& s, const uint16_t* R, const uint16_t* G1, const uint16_t* G2,
                         const int32_t* idx, const float* Ain, float* Wout, uint16_t* Out, hipStream_t st) {
#define SPT_ROWS(DH, KT, KG, STAT) return launch_rows<DH, KT, KG, LPL, BWD, STAT>(s, R, G1, G2, idx, Ain, Wout, Out, st)
  if (s.dh == 64) {
    if (s.n <= 256) SPT_ROWS(64, 1, 4, true);
    if (s.n <= 512) SPT_ROWS(64, 2, 4, true);
    SPT_ROWS(64, 2, 8, false);
  }
  if (s.n <= 256) SPT_ROWS(128, 1, 2, true);
  if (s.n <= 512) SPT_ROWS(128, 2, 4, true);
  SPT_ROWS(128, 1, 2, false);
#undef SPT_ROWS
}

template <bool BWD>
hipError_t rows_by_length(const spt_mha_shape_t& s, const void* R, const void* G1, const void* G2, const int32_t* idx,
                          const float* Ain, float* Wout, void* Out, hipStream_t st) {
  const uint16_t *r = static_cast<const uint16_t*>(R), *g1 = static_cast<const uint16_t*>(G1), *g2 = static_cast<const uint16_t*>(G2);
  uint16_t* out = static_cast<uint16_t*>(Out);
  switch ((s.L + 63) / 64) {
    case 1: return rows_by_shape<1, BWD>(s, r, g1, g2, idx, Ain, Wout, out, st);
    case 2: return rows_by_shape<2, BWD>(s, r, g1, g2, idx, Ain, Wout, out, st);
    case 3: return rows_by_shape<3, BWD>(s, r, g1, g2, idx, Ain, Wout, out, st);
    default: return rows_by_shape<4, BWD>(s, r, g1, g2, idx, Ain, Wout, out, st);
  }
}

template <int DH, int LPL>
hipError_t launch_keys_t(const spt_mha_shape_t& s, const uint16_t* Q, const uint16_t* dY, const int32_t* idx,
                         const float* A, const float* dS, uint16_t* dK, uint16_t* dV, hipStream_t st) {
  const size_t lds = (keys_two_tiles<DH, LPL>() ? 4 : 2) * KV_TS * 4 + 2 * KV_Q * DH * 2 + KV_FLAGS;
  static bool attr_set = false;
  if (!attr_set) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(mha_keys_kernel<DH, LPL>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  const int parts = (s.n + KV_KEYS - 1) / KV_KEYS;
  mha_keys_kernel<DH, LPL><<<8 * parts * ((s.S + 7) / 8), NT, lds, st>>>(Q, dY, idx, A, dS, dK, dV, s.S, s.n, s.L,
                                                                         parts);
  return hipGetLastError();
}

}  // namespace

hipError_t mha_dense_fwd(const spt_mha_shape_t& s, const void* Q, const void* K, const void* V, const int32_t* idx,
                         float* A, void* Y, hipStream_t st) {
  return rows_by_length<false>(s, Q, K, V, idx, nullptr, A, Y, st);
}

hipError_t mha_dense_bwd_q(const spt_mha_shape_t& s, const void* K, const void* V, const void* dY, const int32_t* idx,
                           const float* A, float* dS, void* dQ, hipStream_t st) {
  return rows_by_length<true>(s, dY, V, K, idx, A, dS, dQ, st);
}

hipError_t mha_dense_bwd_kv(const spt_mha_shape_t& s, const void* Q, const void* dY, const int32_t* idx,
                            const float* A, const float* dS, void* dK, void* dV, hipStream_t st) {
  const uint16_t *q = static_cast<const uint16_t*>(Q), *dy = static_cast<const uint16_t*>(dY);
  uint16_t *dk = static_cast<uint16_t*>(dK), *dv = static_cast<uint16_t*>(dV);
#define SPT_KEYS(LPL)                                                              \
  (s.dh == 64 ? launch_keys_t<64, LPL>(s, q, dy, idx, A, dS, dk, dv, st)    \
              : launch_keys_t<128, LPL>(s, q, dy, idx, A, dS, dk, dv, st))
  switch ((s.L + 63) / 64) {
    case 1: return SPT_KEYS(1);
    case 2: return SPT_KEYS(2);
    case 3: return SPT_KEYS(3);
    default: return SPT_KEYS(4);
  }
#undef SPT_KEYS
}

}  // namespace spt
