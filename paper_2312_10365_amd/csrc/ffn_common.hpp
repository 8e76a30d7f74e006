// Device-side building blocks shared by the routed-FFN GEMM kernels (gfx950 only): the LDS DMA
// copy, the hand-placed wait, LDS slot swizzles, the transposing LDS read, the MFMA row
// permutation, and the row-tile record of the schedule tables.
#pragma once
#include "spt_device.hpp"

namespace spt {

constexpr int TILE = 128;  // output tile edge of the narrow-block kernels

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ bf16x8 as_bf16x8(const uint4& v) { return __builtin_bit_cast(bf16x8, v); }

// "Fragment order" of the per-pair hidden values of narrow blocks (act(H), dHpre: written by the
// K = d GEMM, read by the K = Bs and the weight-gradient GEMMs): 32 consecutive sorted positions x
// 16 consecutive hidden units form one contiguous kilobyte, [position / 32][unit / 16]
// [position % 32][unit % 16].  A wavefront whose lanes hold consecutive positions then reads one
// K-step of a 32-row MFMA operand as one contiguous kilobyte instead of 32 pieces 2 Bs bytes
// apart.  A tensor of P positions holds ceil(P / 32) * 32 rows.
__host__ __device__ __forceinline__ size_t hfrag_off(int q, int u, int Bs) {
  return ((size_t)(q >> 5) * (size_t)(Bs >> 4) + (size_t)(u >> 4)) * 512 + (size_t)((q & 31) * 16 + (u & 15));
}
template <bool FRAG>
__device__ __forceinline__ size_t hval_off(int q, int u, int Bs) {
  return FRAG ? hfrag_off(q, u, Bs) : (size_t)q * Bs + u;
}

// One row tile of a bucket in an XCD's run order: bucket id (below 1024), rows (at most: the bucket may end before) and first
// sorted position.
struct KdTile { uint16_t bucket, rows; int32_t q0; };

// Run table.  For token range r (tokens r R .. r R + R - 1) and bucket b the rows of the bucket
// that belong to the range are one contiguous run of sorted positions (inside a bucket the token
// ids ascend): [starts[r][b], starts[r+1][b]), a dense table the schedule kernel fills.  One
// wavefront per range turns its two table rows into the list of the range's NON-EMPTY runs, in
// ascending block order and cut into pieces (the K = Bs kernel's 16-row tiles start at a multiple of
// four positions, so a piece ends run_rows behind one), as (block, first, end, piece) records, and
// their count.  A range has at most N + (R k + 3 N) / run_rows records.
struct RunRec { int32_t b, lo, hi, piece; };

__device__ __forceinline__ void compact_runs(const int32_t* starts, int N, int cap, int run_rows, RunRec* runs, int32_t* nruns, int r,
                                             int lane) {
  const int32_t* s0 = starts + (size_t)r * N;
  const int32_t* s1 = s0 + N;
  RunRec* list = runs + (size_t)r * cap;
  int count = 0;
  for (int b0 = 0; b0 < N; b0 += 64) {
    const int b = b0 + lane;
    const int first = (b < N) ? s0[b] : 0, end = (b < N) ? s1[b] : 0;
    const int base = first & ~3;
    const int pieces = end > first ? (end - base + run_rows - 1) / run_rows : 0;
    int incl = pieces;  // inclusive scan over the wavefront
#pragma unroll
    for (int sft = 1; sft < 64; sft <<= 1) {
      const int up = __shfl_up(incl, sft);
      if (lane >= sft) incl += up;
    }
    int at = count + incl - pieces;
    for (int p = 0; p < pieces; ++p, ++at)
      if (at < cap) list[at] = RunRec{b, max(first, base + p * run_rows), min(base + (p + 1) * run_rows, end), p};
    count += __shfl(incl, 63);
  }
  if (lane == 0) nruns[r] = count < cap ? count : cap;
}

// 16-byte slot of (row, chunk) in a stage region with 4 chunks (64 bytes, 32 K-values) per row.
__device__ __forceinline__ int kd_slot(int row, int chunk) { return row * 4 + (chunk ^ ((row >> 2) & 3)); }

// Asynchronous copy global -> LDS, 16 bytes per lane; lane L's data lands at lds_base + 16 L.
__device__ __forceinline__ void dma16(const void* gptr, uint32_t lds_base) {
  asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds_base), "v"(gptr) : "memory");
}
// The same with 4 bytes per lane.
__device__ __forceinline__ void dma4(const void* gptr, uint32_t lds_base) {
  asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dword %1, off" ::"s"(lds_base), "v"(gptr) : "memory");
}
// s_waitcnt vmcnt(N) alone (N <= 63): the other counters are left at their maxima.
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | (0x7 << 4) | (0xF << 8));
}

// MFMA row i of a 32-row tile can be fed any operand row; feeding it row
// rho32(i) = 16*((i>>2)&1) + 4*(i>>3) + (i&3) makes the 16 accumulator values of a lane 16
// CONSECUTIVE rows of the operand.
__device__ __forceinline__ int rho32(int i) { return 16 * ((i >> 2) & 1) + 4 * (i >> 3) + (i & 3); }

// ds_read_b64_tr_b16 hands each lane 4 consecutive K-values of ONE column out of a K-major
// tile.  Within a group of 16 lanes, lane s points at row (s >> 2), 4-column group (s & 3), and
// result[j][e] = memory[address of lane 4e + (j >> 2)][j & 3].  Two of them make one 8-value
// MFMA operand fragment.
typedef short v4s __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) v4s* lds_v4s_ptr;

__device__ __forceinline__ bf16x8 tr_read_frag(const char* lds_lo, const char* lds_hi) {
  struct { v4s a, b; } t;
  t.a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s_ptr)(uintptr_t)lds_lo);
  t.b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s_ptr)(uintptr_t)lds_hi);
  return __builtin_bit_cast(bf16x8, t);
}

__device__ __forceinline__ bf16x8 as_bf16x8(const u32x4& v) { return __builtin_bit_cast(bf16x8, v); }

// 4 x 4 transpose of 16-byte pieces over four lanes in a row: piece j of lane q becomes piece q of lane j.
template <int CTRL>
__device__ __forceinline__ void quad_exchange(bf16x8& pa, bf16x8& pb, bool second) {   // a of the second lane of a pair for b of the first
  u32x4 a = __builtin_bit_cast(u32x4, pa), b = __builtin_bit_cast(u32x4, pb);
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const uint32_t from_b = (uint32_t)__builtin_amdgcn_mov_dpp((int)b[e], CTRL, 0xF, 0xF, true);
    const uint32_t from_a = (uint32_t)__builtin_amdgcn_mov_dpp((int)a[e], CTRL, 0xF, 0xF, true);
    a[e] = second ? from_b : a[e];
    b[e] = second ? b[e] : from_a;
  }
  pa = as_bf16x8(a);
  pb = as_bf16x8(b);
}
__device__ __forceinline__ void quad_transpose(bf16x8* x, uint32_t lane) {
  quad_exchange<0xB1>(x[0], x[1], lane & 1);
  quad_exchange<0xB1>(x[2], x[3], lane & 1);
  quad_exchange<0x4E>(x[0], x[2], lane & 2);
  quad_exchange<0x4E>(x[1], x[3], lane & 2);
}

// Halves of eight words -> an MFMA fragment.
__device__ __forceinline__ bf16x8 pick_halves(const u32x4& a, const u32x4& b, uint32_t which) {
  return as_bf16x8(u32x4{__builtin_amdgcn_perm(a[1], a[0], which), __builtin_amdgcn_perm(a[3], a[2], which),
                         __builtin_amdgcn_perm(b[1], b[0], which), __builtin_amdgcn_perm(b[3], b[2], which)});
}
__device__ __forceinline__ bf16x8 upper_halves(const u32x4& a, const u32x4& b) { return pick_halves(a, b, 0x07060302u); }
__device__ __forceinline__ bf16x8 lower_halves(const u32x4& a, const u32x4& b) { return pick_halves(a, b, 0x05040100u); }

// fp32 as three bf16 whose sum it is: its upper half, that of what it leaves, and that of what is left then
// (truncations, so exact down to bf16's denormals).  Eight words at once.
__device__ __forceinline__ float less_upper_half(float x) { return x - __uint_as_float(__float_as_uint(x) & 0xFFFF0000u); }
__device__ __forceinline__ void split_bf16x3(u32x4 a, u32x4 b, bf16x8& hi, bf16x8& mid, bf16x8& lo) {
  auto step = [](u32x4& x) {
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = __float_as_uint(less_upper_half(__uint_as_float(x[e])));
  };
  hi = upper_halves(a, b);
  step(a); step(b);
  mid = upper_halves(a, b);
  step(a); step(b);
  lo = upper_halves(a, b);
}

}  // namespace spt
