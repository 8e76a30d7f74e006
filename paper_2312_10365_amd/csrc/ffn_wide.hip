// Routed FFN, blocks wider than 128 hidden units (the paper's own regime, section 4.2: G = 4 or 8
// groups of D/G units, so a block is 1024-2752 units wide).  Every stage is then a large GEMM
// per bucket and the matrix cores, not the partial-row traffic, bound the path, so all six
// GEMMs of Eq. 4 / Alg. 4 and their derivatives share one mainloop built for reuse:
//
//   C[a][n] = sum_k A[a][k] * B[n][k],  256 x 256 outputs per workgroup, 4 wavefronts 2 x 2,
//   128 x 128 per wavefront (4 x 4 tiles of v_mfma_f32_32x32x16_bf16, 256 accumulator
//   registers), K in stages of 32 through a 5-slot LDS ring (32 KiB per stage, three stages
//   in flight, two resident) filled by global_load_lds_dwordx4 with hand-placed vmcnt waits.
//   The weight gradients have four slots, two stages in flight, and the token ids of their gathered
//   rows in the last one's place (global_load_lds_dword, 2 KiB).
//
//   GEMM                       | A side (MFMA rows)           | B side (MFMA columns)        | K
//   up  (Alg. 4 inner proj.)   | hidden units: rows of W1_b   | bucket rows: gathered X rows | d
//   dH  (backward)             | hidden units: rows of W2_b   | bucket rows: gathered dY     | d
//   down / dX partial rows     | output columns of W2_b / W1_b| bucket rows of H / dHpre     | Bs
//   dW2 / dW1                  | columns of gathered dY / X   | hidden units of H / dHpre    | bucket rows
//
// An operand whose K axis is contiguous in memory (rows of W for up/dH, gathered activation
// rows, rows of H) lands in LDS as 256 rows x 64 bytes and is read with ds_read_b128; one
// whose K axis is the slow one (W for down/dX, everything for dW) lands as 32 K-rows x 512
// bytes exactly as stored and is read with the transposing ds_read_b64_tr_b16.  Either way the
// A side is fed to the MFMA rows through the permutation rho32, so a lane ends up with 16
// CONSECUTIVE A-side indices of one B-side index: every epilogue writes 32- or 64-byte runs.
// Rows or columns past the end of a bucket, of the block or of d are pointed at a valid
// address and never stored; K rows past a bucket's end (dW only) read a row of zeros on the
// B side, so they add nothing.
#include "ffn_common.hpp"
#include "spt_host.hpp"
#include "profile.hpp"

namespace spt {

constexpr int WD = 256;                      // tile edge, both sides
constexpr int WK = 32;                       // K values per stage
constexpr int W_RT = 4;                      // row tiles per scheduling group

// A tile of MA x NB MFMA tiles per wavefront: 4 x 4 is the 256 x 256 one, 4 x 2 has half the B-side rows, 2 x 2 is
// a quarter (both for what is left after the last full round of the CUs), 1 x 1 for a bucket's last rows (at most 64).  Fewer products
// per stage hide less of a copy's latency, so the smaller ones keep more stages in flight, in rings of the same 160 KiB or less.
template <int MA, int NB>
struct WideTile {
  static constexpr int A_EDGE = 64 * MA, B_EDGE = 64 * NB;
  static constexpr int A_REGION = A_EDGE * WK * 2, B_REGION = B_EDGE * WK * 2;  // bytes of an operand in a stage
  static constexpr int STAGE = A_REGION + B_REGION;                            // 32, 24, 16, 8 KiB
  static constexpr int STAGES = 160 * 1024 / STAGE;                            // 5, 6, 10, 20
};
constexpr int W_SMEM = WideTile<4, 4>::STAGES * WideTile<4, 4>::STAGE;   // 160 KiB, the whole LDS of a CU

enum { OP_UP = 0, OP_DH = 1, OP_PART = 2, OP_DW = 3 };

// Identity the compiler cannot see through.  An accumulator value that is used more than once
// would otherwise be copied out of the accumulator registers right after the K loop -- all
// 256 of them at once -- instead of where it is used.
__device__ __forceinline__ float pin_vgpr(float x) {
  asm volatile("" : "+v"(x));
  return x;
}

__device__ __forceinline__ uint4 pack_bf16x8(const float (&v)[8]) {
  return make_uint4(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7]));
}

// One A_EDGE x B_EDGE output tile.  b: block; a0 / n0: first A-side / B-side index; [qb, qe): the K
// range (OP_DW: the bucket's rows) -- for the other GEMMs qe bounds the B-side rows.
template <int OP, int ACT, int MA, int NB>
__device__ __forceinline__ void wide_tile(const WideArgs& p, uint4* smem, int b, int a0, int n0,
                                          int qb, int qe) {
  constexpr bool A_TR = (OP == OP_PART || OP == OP_DW);
  constexpr bool B_TR = (OP == OP_DW);
  static_assert((MA == 4 && NB == 4) || OP != OP_DW, "the weight gradients have full tiles only");
  using Tile = WideTile<MA, NB>;
  // (weight gradients: a slot less, for the token ids)
  constexpr int W_STAGE = Tile::STAGE, W_STAGES = OP == OP_DW ? Tile::STAGES - 1 : Tile::STAGES;
  static_assert(OP != OP_DW || W_STAGES * W_STAGE + 4 * 512 <= W_SMEM, "the token ids lie behind the ring");
  constexpr bool SMALL = MA * NB == 1;
  constexpr int GROUP = 4;                         // SMALL: stages between barriers
  static_assert(!SMALL || W_STAGES % GROUP == 0, "whole groups");
  constexpr int A_CH = 8 * MA, B_CH = 8 * NB;      // 16-byte chunks of a K-row of a K-major operand
  constexpr int A_HALF = 32 * MA, B_HALF = 32 * NB;  // A-side / B-side indices of a wavefront
  const int Bs = p.Bs, d = p.d;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int i = lane & 31, h = lane >> 5;
  const uint32_t lds0 = (uint32_t)(uintptr_t)smem;
  const uint16_t* __restrict__ Aop = static_cast<const uint16_t*>(p.A);
  const uint16_t* __restrict__ Bop = static_cast<const uint16_t*>(p.B);
  const int a_lim = (OP == OP_UP || OP == OP_DH) ? Bs : d;
  // Low-rank adapters (section 2.2) extend the K = d GEMMs by two stages: 64 more K-values per
  // gathered row (Xe[token][64]) and per hidden unit (We[unit][64]).
  // (Compiled in only when bit 2 of ACT is set, so the plain path pays nothing for it.)
  constexpr bool EXT = (OP == OP_UP || OP == OP_DH) && (ACT & 4) != 0;
  const int nkd = d / WK;
  const int nk = (OP == OP_DW) ? (qe - qb + WK - 1) / WK : ((OP == OP_PART) ? Bs / WK : nkd + (EXT ? 2 : 0));

  // ---- DMA lane roles.  A wavefront issues MA (NB) instructions for the A (B) operand of a stage;
  // instruction (wave, j) fills 1 KiB: for a K-contiguous operand rows 16 (MA wave + j) + lane / 4, physical
  // chunk lane % 4 (logical chunk = physical ^ swizzle(row)); for a K-major operand (MA = 4) K-rows
  // 2 (4 wave + j) + lane / 32, physical chunk lane % 32 (logical = physical ^ ((krow & 3) << 2)); MA = 2: K-rows
  // 4 (2 wave + j) + lane / 16, chunk lane % 16.
  auto k_swizzle = [](int krow) { return A_CH == 8 ? (krow >> 1 & 1) << 2 : (krow & 3) << 2; };   // (MA = 1: 8 chunks)
  const uint16_t* a_ptr[MA];
  const uint16_t* b_ptr[NB];
  int a_coloff[MA], b_coloff[NB];
  int a_unit[MA], b_tok[NB];  // K = d GEMMs: hidden unit / token id of this lane's row (for the extension)
#pragma unroll
  for (int j = 0; j < MA; ++j) {
    const int row = (wave * MA + j) * 16 + (lane >> 2);
    const int ch = (lane & 3) ^ ((row >> 2) & 3);
    const int krow = (64 / A_CH) * (wave * MA + j) + lane / A_CH;
    const int kcol = ((lane & (A_CH - 1)) ^ k_swizzle(krow)) << 3;
    if (!A_TR) {
      const int u = (a0 + row < Bs) ? a0 + row : a0;
      a_ptr[j] = Aop + ((size_t)b * Bs + u) * d + ch * 8;
      a_coloff[j] = 0;
      a_unit[j] = b * Bs + u;
    } else {
      const int col = (a0 + kcol < d) ? a0 + kcol : a0;
      a_coloff[j] = col;
      a_ptr[j] = (OP == OP_PART) ? Aop + ((size_t)b * Bs + krow) * d + col : Aop;
      a_unit[j] = 0;
    }
  }
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int row = (wave * NB + j) * 16 + (lane >> 2);
    const int ch = (lane & 3) ^ ((row >> 2) & 3);
    const int krow = (64 / B_CH) * (wave * NB + j) + lane / B_CH;
    const int kcol = ((lane & (B_CH - 1)) ^ ((krow & 3) << 2)) << 3;
    if (!B_TR) {
      const int q = (n0 + row < qe) ? n0 + row : n0;
      b_tok[j] = (OP == OP_PART) ? 0 : p.tok[q];
      b_ptr[j] = (OP == OP_PART) ? Bop + (size_t)q * Bs + ch * 8 : Bop + (size_t)b_tok[j] * d + ch * 8;
      b_coloff[j] = 0;
    } else {
      b_coloff[j] = (n0 + kcol < Bs) ? n0 + kcol : n0;
      b_ptr[j] = Bop;
      b_tok[j] = 0;
    }
  }
  const int lane_half = lane >> 5;
  // Token ids of the gathered K-rows (dW only), copied to LDS as well: the eight rows of this wavefront of 8 stages
  // are a group of 256 bytes, two groups per wavefront.  (As scalar loads they shared a counter with the fragment
  // reads, and every stage waited for a load from L2: us, T 8192, d 4096, 4 blocks of 2752, 2 active, a gradient: 395 -> 345.)
  const uint32_t ids0 = W_STAGES * W_STAGE + wave * 512;
  auto fetch_ids = [&](int group) {
    const int q = qb + (group * 8 + (lane >> 3)) * WK + 8 * wave + (lane & 7);
    dma4(p.tok + min(q, qe - 1), __builtin_amdgcn_readfirstlane(lds0 + ids0 + (group & 1) * 256));
  };
  auto load_ids = [&](int kt, int (&ids)[4]) {   // of the lane's row of each copy of stage kt
    const int* at = reinterpret_cast<const int*>(reinterpret_cast<const char*>(smem) + ids0 + (kt & 15) * 32 + lane_half * 4);
#pragma unroll
    for (int j = 0; j < 4; ++j) ids[j] = at[2 * j];
  };
  // One DMA instruction: j-th of this wavefront for operand A (which = 0) or B (which = 1),
  // K-stage kt into ring slot `stage`.
  auto issue_one = [&](int which, int j, int stage, int kt, const int (&ids)[4]) {
    const uint32_t dst = __builtin_amdgcn_readfirstlane(
        lds0 + (uint32_t)(stage * W_STAGE + (which ? Tile::A_REGION : 0) + (wave * (which ? NB : MA) + j) * 1024));
    if (which == 0) {
      if (!A_TR) {
        // (selects, not a branch: the loop body stays one basic block)
        const int ch8 = ((lane & 3) ^ ((lane >> 4) & 3)) * 8;
        const bool ext = EXT && kt >= nkd;
        const uint16_t* src = ext ? p.We + (size_t)a_unit[j] * 64 + (kt - nkd) * WK + ch8 : a_ptr[j] + kt * WK;
        dma16(src, dst);
      } else if (OP == OP_PART) {
        dma16(a_ptr[j] + (size_t)kt * WK * d, dst);
      } else {
        dma16(Aop + (size_t)ids[j] * d + a_coloff[j], dst);
      }
    } else {
      if (!B_TR) {
        const int ch8 = ((lane & 3) ^ ((lane >> 4) & 3)) * 8;
        const bool ext = EXT && kt >= nkd;
        const uint16_t* src = ext ? p.Xe + (size_t)b_tok[j] * 64 + (kt - nkd) * WK + ch8 : b_ptr[j] + kt * WK;
        dma16(src, dst);
      } else {
        const int q = qb + kt * WK + 2 * (wave * 4 + j) + lane_half;
        const uint16_t* src = (q < qe) ? Bop + (size_t)q * Bs + b_coloff[j] : p.zero_row + ((lane & 15) << 3);
        dma16(src, dst);
      }
    }
  };

  // ---- fragment addressing.  Transposing reads, lane (group g = lane / 16, s = lane % 16):
  // K-row 8 (g >> 1) + 4 r + (s >> 2) of the 16-row K-step; column group: natural order
  // 16 (g & 1) + 4 (s & 3) on the B side, the rho32-permuted one on the A side.
  const int g = lane >> 4, sl = lane & 15;
  const int sw = ((sl >> 2) & 3) << 2, sw_a = k_swizzle(sl >> 2);
  const int ag = sl & 3;
  const int acol = 4 * (4 * (ag & 1) + 2 * (g & 1) + (ag >> 1));
  const int bcol = 16 * (g & 1) + 4 * (sl & 3);
  const uint32_t tr_row0 = (uint32_t)((8 * (g >> 1) + (sl >> 2)) * 16);   // (times the chunks of a K-row)
  const int arow = rho32(i);

  // Fragment f of K-step s of the stage at st: f < MA is A-side tile f, else B-side tile f - MA.
  auto load_frag = [&](const char* st, int s, int f) -> bf16x8 {
    if (f < MA) {
      if (!A_TR) return as_bf16x8(reinterpret_cast<const uint4*>(st)[kd_slot(wm * A_HALF + f * 32 + arow, 2 * s + h)]);
      const uint32_t ch = (uint32_t)((((wm * MA + f) * 4 + (acol >> 3)) ^ sw_a) * 16 + (acol & 4) * 2);
      const char* base = st + s * 16 * A_CH * 16 + tr_row0 * A_CH + ch;
      return tr_read_frag(base, base + 4 * A_CH * 16);
    }
    const char* stB = st + Tile::A_REGION;
    if (!B_TR) return as_bf16x8(reinterpret_cast<const uint4*>(stB)[kd_slot(wn * B_HALF + (f - MA) * 32 + i, 2 * s + h)]);
    const uint32_t ch = (uint32_t)((((wn * NB + (f - MA)) * 4 + (bcol >> 3)) ^ sw) * 16 + (bcol & 4) * 2);
    const char* base = stB + s * 16 * B_CH * 16 + tr_row0 * B_CH + ch;
    return tr_read_frag(base, base + 4 * B_CH * 16);
  };

  f32x16 acc[MA][NB];
#pragma unroll
  for (int mi = 0; mi < MA; ++mi)
#pragma unroll
    for (int ni = 0; ni < NB; ++ni)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[mi][ni][v] = 0.f;

  // The previous tile's epilogue stores are drained and every wavefront has left its last stage
  // before the ring is refilled.
  wait_vmcnt<0>();
  __builtin_amdgcn_s_barrier();
  // Ring schedule (W_STAGES = S slots).  "Issue j" copies K-stage min(j, nk-1) into slot j % S: past the
  // last stage it copies the last one again into a slot nobody reads, which keeps the number of
  // copies per iteration -- and with it every vmcnt wait -- the same from the first to the last
  // iteration, and the loop body free of branches.  Issues 0..S-2 go out up front; iteration kt
  // sends issue kt+S-1 (into the slot stage kt-1 left).  At the top of iteration kt the stages kt
  // and kt+1 have landed and are visible to every wavefront, and the fragments of (stage kt,
  // K-step 0) are in registers.
  //
  // A wavefront is alone on its SIMD, so nothing hides what it does between two MFMAs: every
  // other instruction of the iteration is therefore placed right behind an MFMA (each keeps the
  // matrix pipe busy for 32 cycles): after MFMA 0..7 of a K-step one fragment read for the next
  // K-step (issued half an iteration before its data are used), after MFMA 8..11 one DMA
  // instruction, after MFMA 12 the reads of the token ids for the next iteration's DMA.
  // (The smaller tiles: a fragment read behind each of the first MFMAs, the copies behind the last ones.)
  const int klast = nk - 1;
  auto kclamp = [&](int j) { return j < klast ? j : klast; };
  int ids[4] = {0, 0, 0, 0}, ids_next[4] = {0, 0, 0, 0};
  bf16x8 fa[2][MA], fb[2][NB];
  const char* ring = reinterpret_cast<const char*>(smem);
  if (nk > 0) {
    if (OP == OP_DW) {
      fetch_ids(0);
      fetch_ids(1);
      wait_vmcnt<0>();
    }
#pragma unroll
    for (int st = 0; st < (SMALL ? W_STAGES - GROUP : W_STAGES - 1); ++st) {
      if (OP == OP_DW) load_ids(kclamp(st), ids);
#pragma unroll
      for (int j = 0; j < MA; ++j) issue_one(0, j, st, kclamp(st), ids);
#pragma unroll
      for (int j = 0; j < NB; ++j) issue_one(1, j, st, kclamp(st), ids);
    }
    if (OP == OP_DW) load_ids(kclamp(W_STAGES - 1), ids);
    if (!SMALL) {
      wait_vmcnt<(W_STAGES - 3) * (MA + NB)>();  // issues 0 and 1 have landed (2 .. S-2 may be out)
      __builtin_amdgcn_s_barrier();
#pragma unroll
      for (int f = 0; f < MA; ++f) fa[0][f] = load_frag(ring, 0, f);
#pragma unroll
      for (int f = 0; f < NB; ++f) fb[0][f] = load_frag(ring, 0, f + MA);
    }
  }
  if constexpr (SMALL) {
    // Two products a stage: four stages between barriers, four groups of them in flight, and the copies of a group go out in front of
    // the products of the one that has landed.
    for (int kt = 0; kt < nk; kt += GROUP) {
      wait_vmcnt<(W_STAGES / GROUP - 2) * GROUP * (MA + NB)>();
      __builtin_amdgcn_s_barrier();                        // (everyone's copies, and everyone has read the group before)
      const int at = kt % W_STAGES, into = (at == 0 ? W_STAGES : at) - GROUP;
#pragma unroll
      for (int u = 0; u < GROUP; ++u) {
        const int kfill = kclamp(kt + W_STAGES - GROUP + u);
        issue_one(0, 0, into + u, kfill, ids);
        issue_one(1, 0, into + u, kfill, ids);
      }
#pragma unroll
      for (int u = 0; u < GROUP; ++u) {
        if (kt + u >= nk) break;                           // uniform
        const char* st0 = ring + (at + u) * W_STAGE;
#pragma unroll
        for (int sx = 0; sx < 2; ++sx)
          acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(load_frag(st0, sx, 0), load_frag(st0, sx, 1), acc[0][0], 0, 0, 0);
      }
    }
  } else {
    int stage = 0;
    for (int kt = 0; kt < nk; ++kt) {
      const int next = (stage + 1 == W_STAGES) ? 0 : stage + 1;
      const int fill = (stage == 0) ? W_STAGES - 1 : stage - 1;  // slot of stage kt-1 = (kt+S-1) % S
      const char* st0 = ring + stage * W_STAGE;
      // after the last stage the look-ahead reads the current one again: harmless
      const char* st1 = ring + ((kt + 1 < nk) ? next : stage) * W_STAGE;
      const int kfill = kclamp(kt + W_STAGES - 1);
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        // half 0: multiply K-step 0, read (stage kt, K-step 1), copy the A part of issue kt+S-1;
        // half 1: multiply K-step 1, read (stage kt+1, K-step 0), copy the B part.
        constexpr int M = MA * NB;
        const int copies = half ? NB : MA, c0 = M == 16 ? 8 : M - copies;   // c0: first MFMA with a copy behind it
#pragma unroll
        for (int m = 0; m < M; ++m) {
          const int mi = m / NB, ni = m % NB;
          acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[half][mi], fb[half][ni], acc[mi][ni], 0, 0, 0);
          if (m < MA + NB) {
            const bf16x8 fr = load_frag(half ? st1 : st0, half ? 0 : 1, m);
            if (m < MA) fa[half ^ 1][m] = fr; else fb[half ^ 1][m - MA] = fr;
          }
          if (m >= c0 && m < c0 + copies) {
            issue_one(half, m - c0, fill, kfill, ids);
          } else if (m == 12 && half == 1 && OP == OP_DW) {
            if (((kt + W_STAGES) & 7) == 0 && kt + W_STAGES < klast) fetch_ids((kt + W_STAGES) / 8 + 1);   // (over the group read to its end)
            load_ids(kclamp(kt + W_STAGES), ids_next);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) ids[e] = ids_next[e];
      // own copies of stage kt+2 have landed: only issues kt+3 .. kt+S-1 (MA + NB instructions each) may
      // be outstanding; the barrier makes everyone's visible and ends all reads of stage kt
      wait_vmcnt<(W_STAGES - 3) * (MA + NB)>();
      __builtin_amdgcn_s_barrier();
      stage = next;
    }
  }
  wait_vmcnt<0>();  // the trailing copies (repeats of the last stage) are done too

  // ---- epilogue: lane (i, h) holds, for B-side index n0 + B_HALF wn + 32 ni + i, the A-side
  // indices a0 + A_HALF wm + 32 mi + 16 h + (0..15).
  // dH reads the saved pre-activations of its whole tile first (32 loads of 16 bytes per lane, all
  // in flight together; the fragment registers of the main loop are free by now), so the epilogue
  // waits for memory once instead of once per fragment.
  if (OP == OP_DW) {
    // Stored as they lie, the 64-byte runs of a lane would make an instruction touch 64 lines with
    // 16 bytes each.  Each 32 x 32 tile goes through a wavefront-private LDS buffer (rows of 144
    // bytes; the ring is free once everyone's copies have landed) and comes back with 8 lanes
    // along a row: a store instruction then writes 8 whole 128-byte lines.  (Same wavefront on
    // both sides of the buffer: LDS executes its accesses in order.)
    __builtin_amdgcn_s_barrier();
    float* tbuf = reinterpret_cast<float*>(smem) + wave * (32 * 36);
    const int cc = lane & 7, r0 = lane >> 3;
#pragma unroll
    for (int ni = 0; ni < NB; ++ni)
#pragma unroll
      for (int mi = 0; mi < MA; ++mi) {
        const f32x16& c = acc[mi][ni];
#pragma unroll
        for (int e = 0; e < 4; ++e)
          *reinterpret_cast<f32x4*>(tbuf + i * 36 + 16 * h + 4 * e) = f32x4{c[4 * e], c[4 * e + 1], c[4 * e + 2], c[4 * e + 3]};
        wave_lds_fence();
        const int aidx = a0 + wm * A_HALF + mi * 32 + 4 * cc;
        f32x4 o[4];  // (all four reads go out before the first store waits for its data)
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = *reinterpret_cast<const f32x4*>(tbuf + (r0 + 8 * e) * 36 + 4 * cc);
        wave_lds_fence();
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int nidx = n0 + wn * B_HALF + ni * 32 + r0 + 8 * e;
          if (nidx < Bs && aidx < a_lim) *reinterpret_cast<f32x4*>(p.dW + ((size_t)b * Bs + nidx) * d + aidx) = o[e];
        }
      }
    return;
  }
  if constexpr (MA > 1 && (OP == OP_DH || (OP == OP_UP && (ACT & 3) == 1))) {
    // Two outputs per value: likewise, two A-side tiles at a time (64 bf16 outputs of a row are a line), through rows of
    // 256 bytes whose 16-byte pieces are permuted by row, so that no pass of an access meets a bank twice.
    // us, low-rank pass of T 8192, d 2048, 4 blocks of 2048, k 2, ReLU: up-projection 171 -> 157, dH 183 -> 171; d 4096, blocks of
    // 2752, GELU: dH 396 -> 383.  Nothing gained, so stored as they lie: the up-projection with GELU (363 -> 363, 760 tokens of
    // d 3392 35 -> 36: the stores go out behind its arithmetic), the inference forward (53 -> 56), the partial rows (135).
    constexpr int MP = MA / 2;                               // pairs of A-side tiles
    const int c8 = (lane & 7) * 8, r0 = lane >> 3;           // lane's piece: rows r0 + 8 r, 8 columns from c8 on
    uint4 zsave[(OP == OP_DH) ? NB : 1][(OP == OP_DH) ? MP : 1][4];
    if (OP == OP_DH) {
#pragma unroll
      for (int ni = 0; ni < NB; ++ni)
#pragma unroll
        for (int mp = 0; mp < MP; ++mp)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int nidx = n0 + wn * B_HALF + ni * 32 + r0 + 8 * r, aidx = a0 + wm * A_HALF + mp * 64 + c8;
            if (nidx < qe && aidx < a_lim)
              zsave[ni][mp][r] = *reinterpret_cast<const uint4*>(p.Hsave + (size_t)nidx * Bs + aidx);
          }
    }
    __builtin_amdgcn_s_barrier();                            // (the ring is free, as above)
    f32x4* tbuf = reinterpret_cast<f32x4*>(smem) + wave * (32 * 16);
    auto put = [&](int ni, int mp) {
#pragma unroll
      for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const f32x16& c = acc[2 * mp + m][ni];
          tbuf[i * 16 + ((8 * m + 4 * h + e) ^ (i & 15))] = f32x4{c[4 * e], c[4 * e + 1], c[4 * e + 2], c[4 * e + 3]};
        }
    };
    put(0, 0);
#pragma unroll
    for (int ni = 0; ni < NB; ++ni) {
#pragma unroll
      for (int mp = 0; mp < MP; ++mp) {
        wave_lds_fence();
        f32x4 o[4][2];
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int e = 0; e < 2; ++e) o[r][e] = tbuf[(r0 + 8 * r) * 16 + ((2 * (lane & 7) + e) ^ ((r0 + 8 * r) & 15))];
        wave_lds_fence();
        // (the next pair goes in behind these reads)
        if (mp + 1 < MP) put(ni, mp + 1);
        else if (ni + 1 < NB) put(ni + 1, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int nidx = n0 + wn * B_HALF + ni * 32 + r0 + 8 * r, aidx = a0 + wm * A_HALF + mp * 64 + c8;
          if (nidx < qe && aidx < a_lim) {
            const size_t at = (size_t)nidx * Bs + aidx;
            float cv[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) cv[e] = o[r][e / 4][e % 4];
            if (OP == OP_UP) {
              *reinterpret_cast<uint4*>(p.Hsave + at) = pack_bf16x8(cv);
#pragma unroll
              for (int e = 0; e < 8; ++e) cv[e] = act_fn<(ACT & 1)>(cv[e]);
              *reinterpret_cast<uint4*>(p.Hact + at) = pack_bf16x8(cv);
            } else {
              const uint4 z = zsave[(OP == OP_DH) ? ni : 0][(OP == OP_DH) ? mp : 0][r];
              const uint32_t zw[4] = {z.x, z.y, z.z, z.w};
              float av[8];
#pragma unroll
              for (int e = 0; e < 8; ++e) {
                const float x = e & 1 ? hi_bf16(zw[e / 2]) : lo_bf16(zw[e / 2]);
                cv[e] *= act_grad<(ACT & 1)>(x);
                av[e] = act_fn<(ACT & 1)>(x);
              }
              *reinterpret_cast<uint4*>(p.dHpre + at) = pack_bf16x8(cv);
              *reinterpret_cast<uint4*>(p.Hact + at) = pack_bf16x8(av);
            }
          }
          __builtin_amdgcn_sched_barrier(0);  // 8 values at a time keeps the register need low
        }
      }
    }
    return;
  }
#pragma unroll
  for (int ni = 0; ni < NB; ++ni) {
    const int nidx = n0 + wn * B_HALF + ni * 32 + i;
#pragma unroll
    for (int mi = 0; mi < MA; ++mi) {
      const int aidx = a0 + wm * A_HALF + mi * 32 + 16 * h;
      const f32x16& c = acc[mi][ni];
      if (nidx < qe && aidx < a_lim) {
        if (OP == OP_UP) {
          const size_t o = (size_t)nidx * Bs + aidx;
#pragma unroll
          for (int hf = 0; hf < 2; ++hf) {  // 8 values at a time keeps the register need low
            float cv[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) cv[e] = pin_vgpr(c[8 * hf + e]);
            if (!(ACT & 2))  // bit 1 of ACT: inference forward, nothing saved for a backward pass
              reinterpret_cast<uint4*>(p.Hsave + o)[hf] = pack_bf16x8(cv);
#pragma unroll
            for (int e = 0; e < 8; ++e) cv[e] = act_fn<(ACT & 1)>(cv[e]);
            reinterpret_cast<uint4*>(p.Hact + o)[hf] = pack_bf16x8(cv);
            __builtin_amdgcn_sched_barrier(0);
          }
        } else if (OP == OP_DH) {                          // (a bucket's last rows)
          const size_t o = (size_t)nidx * Bs + aidx;
#pragma unroll
          for (int hf = 0; hf < 2; ++hf) {
            const uint4 z = reinterpret_cast<const uint4*>(p.Hsave + o)[hf];
            const uint32_t zw[4] = {z.x, z.y, z.z, z.w};
            float cv[8], av[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              const float x = e & 1 ? hi_bf16(zw[e / 2]) : lo_bf16(zw[e / 2]);
              cv[e] = c[8 * hf + e] * act_grad<(ACT & 1)>(x);
              av[e] = act_fn<(ACT & 1)>(x);
            }
            reinterpret_cast<uint4*>(p.dHpre + o)[hf] = pack_bf16x8(cv);
            reinterpret_cast<uint4*>(p.Hact + o)[hf] = pack_bf16x8(av);
          }
        } else if (OP == OP_PART) {
          uint4* dst = reinterpret_cast<uint4*>(p.part + (size_t)nidx * d + aidx);
          dst[0] = make_uint4(pack_bf16x2(c[0], c[1]), pack_bf16x2(c[2], c[3]), pack_bf16x2(c[4], c[5]),
                              pack_bf16x2(c[6], c[7]));
          dst[1] = make_uint4(pack_bf16x2(c[8], c[9]), pack_bf16x2(c[10], c[11]),
                              pack_bf16x2(c[12], c[13]), pack_bf16x2(c[14], c[15]));
        }
      }
    }
  }
}

// Up / dH / partial-row GEMMs: persistent workgroups, one per CU.  The work items -- (row tile of the
// bucket-major list, A-side tile), in groups of W_RT row tiles x all A-side tiles, A-side tile major --
// are cut into 8 equal slices, one per XCD (workgroup id modulo 8), and an XCD's 32 workgroups walk its
// slice in step.  They are then on about 4 row tiles x 8 A-side tiles at a time, so each operand slice
// pulled into that XCD's L2 serves several of them.
// What is left of a slice after its full rounds of 32 would cost another round whatever its size.  So up to
// 8 items are worked off as quarters, at 0.35 of a round, up to 16 as halves, at 0.6 (smaller pieces read more
// operand bytes per product; a second and third round of quarters gains nothing over a full one).
// Whole row tiles dealt to the XCDs before: 9 of 66 to some, 4 rounds of 11 A-side tiles each, where 2.84
// rounds' worth of items is there.  us, before and now: T 8192, d 4096, 4 blocks of 2752, k 2: up-projection 450,
// 373, its backward 499, 403 (385 since its outputs go out as whole lines), partial rows 376, 345; 3001 tokens of that 215, 168; 24 tokens 85, 46.
// (Registers: all 256 and 256 of accumulators; dH with GELU and the adapters' stages keeps one in scratch, read back once an item.)
// TAILS: buckets' last rows, where they are at most 64, are listed behind the full tiles (kd_count[1] of those) and can go out as pieces of 64 rows x
// 64 A-side indices, at about 0.12 of a round, instead of as tiles like the others: whichever is less.  For layers whose mean bucket is that small: us
// a pass, 24 tokens of d 4096, 4 blocks of 2752, 2 active 87 -> 65; 100 tokens of d 2048, 4 of 2048 54 -> 44.  Larger buckets, whose tails
// are a few of many tiles, gain nothing (8192 tokens of d 2048, 4 of 2048: 66 items on 32 CUs an XCD, or 64 and the tails, 134.5 / 134.3 -- what the chip
// saves in a last round it has spent on its clock) and pay for the longer kernel: 700 tokens of that layer 151.9 -> 152.8.
template <int OP, int ACT, bool TAILS>
__global__ __launch_bounds__(256, 1) void wide_rows_kernel(WideArgs p) {
  extern __shared__ uint4 w_smem[];
  const int xcd = blockIdx.x & 7, wg = blockIdx.x >> 3, wgs = gridDim.x >> 3;
  const int a_lim = (OP == OP_PART) ? p.d : p.Bs;
  const int n_at = (a_lim + WD - 1) / WD;
  const KdTile* list = static_cast<const KdTile*>(p.kd_list);
  int count = p.kd_count[0], first_tail = 0, pieces = 0;
  constexpr int PIECE = 64;
  const int n_pt = (a_lim + PIECE - 1) / PIECE;
  if (TAILS) {
    const int big = p.kd_count[1], grid = gridDim.x, all = (count - big) * n_pt;
    auto rounds = [&](int tiles) {                         // in hundredths, of the fullest slice
      const int64_t n = ((int64_t)tiles * n_at + 7) >> 3;
      const int left = (int)(n % wgs);
      return n / wgs * 100 + (left == 0 ? 0 : left <= wgs / 4 ? 35 : left <= wgs / 2 ? 60 : 100);
    };
    if (rounds(big) + 12 * ((all + grid - 1) / grid) < rounds(count)) {
      count = first_tail = big;
      pieces = all;
    }
  }
  const int64_t items = (int64_t)count * n_at;
  const int lo = (int)(items * xcd / 8), n = (int)(items * (xcd + 1) / 8) - lo;
  const int left = n % wgs, split = left > wgs / 2 ? 1 : (left > wgs / 4 ? 2 : 4), full = split > 1 ? n - left : n;
  auto locate = [&](int item, KdTile& t, int& a0) {
    const int grp = item / (W_RT * n_at), rem = item - grp * W_RT * n_at;
    const int rtg = (count - grp * W_RT < W_RT) ? count - grp * W_RT : W_RT;
    t = list[grp * W_RT + rem % rtg];
    a0 = (rem / rtg) * WD;
  };
  KdTile t;
  int a0;
  for (int e = wg; e < full; e += wgs) {
    locate(lo + e, t, a0);
    wide_tile<OP, ACT, 4, 4>(p, w_smem, t.bucket, a0, t.q0, 0, p.offsets[t.bucket + 1]);
  }
  if (wg < split * (n - full)) {                           // (at most one piece per workgroup)
    locate(lo + full + wg / split, t, a0);
    const int part = wg % split, n0 = t.q0 + (part & 1) * (WD / 2), qe = p.offsets[t.bucket + 1];
    a0 += (part >> 1) * (WD / 2);
    if (n0 < qe && a0 < a_lim) {
      if (split == 2) wide_tile<OP, ACT, 4, 2>(p, w_smem, t.bucket, a0, n0, 0, qe);
      else            wide_tile<OP, ACT, 2, 2>(p, w_smem, t.bucket, a0, n0, 0, qe);
    }
  }
  if (TAILS)
    for (int e = blockIdx.x; e < pieces; e += gridDim.x) {
      t = list[first_tail + e / n_pt];
      wide_tile<OP, ACT, 1, 1>(p, w_smem, t.bucket, e % n_pt * PIECE, t.q0, 0, p.offsets[t.bucket + 1]);
    }
}

// dW GEMMs: one work item (column tile, unit tile, bucket) per workgroup.  With a multiple of
// 8 column tiles an XCD keeps to the column tiles congruent to its id and takes, for each
// bucket (largest first), all unit tiles of one column tile side by side: they gather the same
// 512-byte column slab of the same activation rows.
__global__ __launch_bounds__(256, 1) void wide_dw_kernel(WideArgs p) {
  extern __shared__ uint4 w_smem[];
  const int n_ct = (p.d + WD - 1) / WD, n_ut = (p.Bs + WD - 1) / WD;
  int ct, ut, br;
  if (n_ct % 8 == 0) {
    const int xcd = blockIdx.x & 7, jj = blockIdx.x >> 3, per = n_ct / 8;
    ut = jj % n_ut;
    const int r = jj / n_ut;
    ct = xcd + 8 * (r % per);
    br = r / per;
  } else {
    ut = blockIdx.x % n_ut;
    const int r = blockIdx.x / n_ut;
    ct = r % n_ct;
    br = r / n_ct;
  }
  if (br >= p.N) return;
  const int b = p.border[br];
  wide_tile<OP_DW, 0, 4, 4>(p, w_smem, b, ct * WD, ut * WD, p.offsets[b], p.offsets[b + 1]);
}

template <int OP, int ACT>
static void launch_rows(const WideArgs& a, bool tails, hipStream_t st) {
  static const hipError_t attr[2] = {hipFuncSetAttribute(reinterpret_cast<const void*>(wide_rows_kernel<OP, ACT, false>),
                                                         hipFuncAttributeMaxDynamicSharedMemorySize, W_SMEM),
                                     hipFuncSetAttribute(reinterpret_cast<const void*>(wide_rows_kernel<OP, ACT, true>),
                                                         hipFuncAttributeMaxDynamicSharedMemorySize, W_SMEM)};
  (void)attr;
  if (tails) wide_rows_kernel<OP, ACT, true><<<8 * 32, 256, W_SMEM, st>>>(a);
  else       wide_rows_kernel<OP, ACT, false><<<8 * 32, 256, W_SMEM, st>>>(a);
}

hipError_t launch_wide(int op, const spt_shape_t& s, const WideArgs& a, hipStream_t st) {
  const bool gelu = s.act == SPT_ACT_GELU, tails = wide_tails(s);
  switch (op) {
    case OP_UP:  // the activation code's bit 1 marks the inference forward (no Hsave), bit 2
                 // the low-rank extension of the K loop
      if (a.Xe)         { if (gelu) launch_rows<OP_UP, 4>(a, tails, st); else launch_rows<OP_UP, 5>(a, tails, st); }
      else if (a.Hsave) { if (gelu) launch_rows<OP_UP, 0>(a, tails, st); else launch_rows<OP_UP, 1>(a, tails, st); }
      else              { if (gelu) launch_rows<OP_UP, 2>(a, tails, st); else launch_rows<OP_UP, 3>(a, tails, st); }
      break;
    case OP_DH:
      if (a.Xe) { if (gelu) launch_rows<OP_DH, 4>(a, tails, st); else launch_rows<OP_DH, 5>(a, tails, st); }
      else      { if (gelu) launch_rows<OP_DH, 0>(a, tails, st); else launch_rows<OP_DH, 1>(a, tails, st); }
      break;
    case OP_PART:
      launch_rows<OP_PART, 0>(a, tails, st);
      break;
    default: {
      const int n_ct = (s.d + WD - 1) / WD, n_ut = (s.Bs + WD - 1) / WD;
      static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(wide_dw_kernel),
                                                         hipFuncAttributeMaxDynamicSharedMemorySize, W_SMEM);
      (void)attr;
      wide_dw_kernel<<<n_ct * n_ut * s.N, 256, W_SMEM, st>>>(a);
    }
  }
  return hipGetLastError();
}

}  // namespace spt
