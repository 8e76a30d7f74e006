// Weight-gradient GEMMs of narrow blocks: the work of one workgroup, for the kernel that does nothing else (ffn.hip) and for the one that
// shares its launch with the K = Bs contraction (ffn_scatter.hip).
#pragma once
#include <type_traits>

#include "ffn_common.hpp"
#include "spt_host.hpp"

namespace spt {

// ------------------------------------------------------------------------------------------
// K = bucket rows GEMMs for Bs <= 128: dW1 (Act = X, Hin = dHpre) and dW2 (Act = dY, Hin = act(H)).
//   dW[b][u][c] = sum_{q in bucket b} Hin[q][u] * Act[tok[q]][c]    MFMA rows c, columns u
// K runs over the bucket's rows in sorted order, so the sum order is fixed (no split-K, no
// atomics).  A workgroup owns 256 output columns x UT hidden units of one block.  UT = 128: wavefront (wm, wn) owns 128 columns x 64 units (4 x 2 MFMA tiles);
// UT = 64, for blocks of at most 64 units (a 128-unit tile would be half padding): wavefront wm
// owns 64 columns x 64 units (2 x 2 tiles).  Two workgroups share a CU.
// Both operands are token-major in memory, i.e. K is the strided dimension for both.  They
// are copied as they are into a 6-slot LDS ring (16 tokens per stage: 16 x 512 B of gathered
// activation columns + 16 x 256 B of Hin) by global_load_lds_dwordx4, and ds_read_b64_tr_b16
// builds the K-contiguous MFMA fragments out of the token-major tiles; the column side goes
// through the rho32 row permutation, so a lane ends up with 16 consecutive columns of one
// hidden unit (64-byte runs of fp32; the epilogue regroups them into whole lines through LDS).
// Ring schedule: "issue j" copies stage min(j, nk-1) into slot j % 6 (past the last stage it
// repeats it into a slot nobody reads: the loop body has no branch and every vmcnt wait is a
// constant).  Issues 0..4 go out up front, iteration kt sends issue kt+5 (LA = 5 below).  At the top of
// iteration kt the stages kt and kt+1 are visible and the fragments of stage kt are in
// registers; the iteration multiplies them (8 MFMAs per wavefront) with, behind each MFMA, one
// piece of the other work: first the 3 DMA instructions, one behind each MFMA (two behind the first one: 2 % slower),
// then the 6 fragment reads of stage kt+1.
// Rows past the bucket's end read a zero line for Hin (so they add nothing) and any valid row
// for the activations.
// The token ids of the gathered rows are copied to LDS as well, 16 stages at a time and 16 to 32 stages ahead, each
// wavefront those of its own rows.  (As scalar loads, one cache line per stage fetched an iteration ahead, they shared a
// counter with the fragment reads: the matrix instructions of every stage waited for a load from L2, and no depth of the ring helped.
// us, both sides on one box: T 8192, d 4096, 128 blocks of 128, 32 active, one product 303 -> 283; T 16384, d 1024, 64 blocks of 64, 16
// active, both products 114 -> 89; T 8192, d 2048, 64 blocks of 128, 16 active and skewed 181 -> 157.)
// What bounds it now: for the first of these MFMAs and fragment reads without copies take 229, copies alone (L2 delivers
// them at twice that rate to loads that nothing else accompanies) less; the clock falls with the matrix units' load.  512 columns
// per workgroup, for a sixth fewer copied bytes, gains nothing any more: 296 against 294; nor do 4, 5 or 7 slots, nor four workgroups of 64-unit
// tiles per CU.
constexpr int DW_KT = 16;                          // tokens per stage
constexpr int DW_CT = 256;                         // columns of a workgroup
constexpr int DW_A_BYTES = DW_KT * DW_CT * 2;      // 8 KiB: 16 token rows x 256 columns
constexpr int DW_SLOTS = 6;                        // 72 KiB per workgroup with 256 x 128 tiles
constexpr int DW_ID_BYTES = 256;                   // token ids of a wavefront's rows of 16 stages

template <int UT>
constexpr int dw_smem_bytes() { return DW_SLOTS * (DW_A_BYTES + DW_KT * UT * 2) + 4 * 2 * DW_ID_BYTES; }

// Workgroups along the (column tile, piece) items.
inline int dw_grid(int npieces, int d) {
  const int nct = (d + DW_CT - 1) / DW_CT;
  return nct % 8 != 0 && 8 % nct == 0 ? 8 * ((npieces + 8 / nct - 1) / (8 / nct)) : nct * npieces;
}

// Workgroup wg of dw_grid's, unit tile ut.
template <int UT>
__device__ __forceinline__ void dw_tile(
    const DwOperands& ops, int wg, int ut,
    const int32_t* __restrict__ tok, const uint16_t* __restrict__ zero_row, int npieces, int Bs,
    int d, const DwPiece* __restrict__ pieces, int nblocks) {
  const uint16_t* __restrict__ Act = ops.Act;
  const uint16_t* __restrict__ Hin = ops.Hin;
  float* __restrict__ dW = ops.dW;
  float* __restrict__ stage = ops.stage;
  constexpr int MI = UT == 128 ? 4 : 2;               // 32-column tiles per wavefront
  constexpr int DW_B_BYTES = DW_KT * UT * 2;          // 4 or 2 KiB
  constexpr int DW_STAGE_BYTES = DW_A_BYTES + DW_B_BYTES;
  constexpr int CPW = UT == 128 ? 128 : 64;           // columns per wavefront
  constexpr int LA = DW_SLOTS - 1;                    // stages a copy is issued ahead of its use
  extern __shared__ uint4 dw_smem[];
  // Work item = (column tile, bucket).  An XCD (workgroup id mod 8) keeps to its own column
  // tiles and walks the buckets, largest first: the workgroups that run together on an XCD
  // then gather the same narrow column slab of the activations -- it fits that XCD's L2 and
  // every token row in it is wanted by k of the N buckets.
  const int nct = (d + DW_CT - 1) / DW_CT;
  const int xcd = wg & 7, jj = wg >> 3;
  int ct, br;
  if (nct % 8 == 0) {
    const int per = nct / 8;
    ct = xcd + 8 * (jj % per);
    br = jj / per;
  } else if (8 % nct == 0) {
    const int r = 8 / nct;
    ct = xcd % nct;
    br = xcd / nct + r * jj;
  } else {
    ct = wg % nct;
    br = wg / nct;
  }
  if (br >= npieces) return;
  const DwPiece pc = pieces[br];
  if (pc.dst < 0) return;
  const int qb = pc.lo, qe = pc.hi;
  float* const dst = pc.dst < nblocks ? dW + (size_t)pc.dst * Bs * d : stage + (size_t)(pc.dst - nblocks) * Bs * d;
  const int c0 = ct * DW_CT, u0 = ut * UT;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = UT == 128 ? wave >> 1 : wave, wn = UT == 128 ? wave & 1 : 0;
  const int i = lane & 31, h = lane >> 5;
  const uint32_t lds0 = (uint32_t)(uintptr_t)dw_smem;
  const int nk = (qe - qb + DW_KT - 1) / DW_KT;
  const int klast = nk - 1;

  // DMA lane roles.  Activations: instruction j (2 per wavefront) moves token rows
  // 4 wave + 2j, + 1 of the stage, 512 B each: lane L -> row + L/32, physical chunk L%32 =
  // logical ^ ((row&3)<<2).  Hin, UT = 128: one instruction per wavefront moves rows 4 wave .. + 3,
  // 256 B each: lane L -> row 4 wave + L/16, physical chunk L%16 = logical ^ ((row&3)<<2).  UT = 64:
  // an instruction moves 8 rows of 128 B (lane L -> row + L/8, physical chunk L%8 = logical ^
  // (((row>>1)&1)<<2)); wavefronts 2 and 3 repeat the copies of 0 and 1 -- same bytes to the same
  // place -- so that every wavefront has the same number of copies in flight.
  const int lane_half = lane >> 5;
  int a_coloff[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int row = 4 * wave + 2 * j + lane_half;
    const int col = c0 + (((lane & 31) ^ ((row & 3) << 2)) << 3);
    a_coloff[j] = (col < d) ? col : c0;  // ragged last column tile: harmless duplicate, never stored
  }
  const int b_row = UT == 128 ? 4 * wave + (lane >> 4) : 8 * (wave & 1) + (lane >> 3);
  int b_coloff = UT == 128 ? u0 + (((lane & 15) ^ ((b_row & 3) << 2)) << 3)
                           : u0 + (((lane & 7) ^ (((b_row >> 1) & 1) << 2)) << 3);
  if (b_coloff >= Bs) b_coloff = u0;
  // Token ids of this wavefront's four rows of 16 stages, 256 bytes; two such groups per wavefront.
  const uint32_t ids0 = DW_SLOTS * DW_STAGE_BYTES + wave * 2 * DW_ID_BYTES;
  auto fetch_ids = [&](int group) {
    const int q = qb + (group * 16 + (lane >> 2)) * DW_KT + 4 * wave + (lane & 3);
    dma4(tok + min(q, qe - 1), __builtin_amdgcn_readfirstlane(lds0 + ids0 + (group & 1) * DW_ID_BYTES));
  };
  auto load_ids = [&](int kt, int (&ids)[2]) {  // of the lane's row of either copy of stage kt
    const int* p = reinterpret_cast<const int*>(reinterpret_cast<const char*>(dw_smem) + ids0 + (kt & 31) * 16 + lane_half * 4);
    ids[0] = p[0];
    ids[1] = p[2];
  };
  auto issue_a = [&](int j, int slot, const int (&ids)[2]) {
    dma16(Act + (size_t)ids[j] * d + a_coloff[j],
          __builtin_amdgcn_readfirstlane(
              lds0 + (uint32_t)(slot * DW_STAGE_BYTES + (wave * 2 + j) * 1024)));
  };
  auto issue_b = [&](int slot, int kt) {
    const int q = qb + kt * DW_KT + b_row;
    const uint16_t* src = (q < qe) ? Hin + hfrag_off(q, b_coloff, Bs) : zero_row + ((lane & 15) << 3);
    dma16(src, __builtin_amdgcn_readfirstlane(
                   lds0 + (uint32_t)(slot * DW_STAGE_BYTES + DW_A_BYTES + (UT == 128 ? wave : wave & 1) * 1024)));
  };

  // Transposing fragment reads, lane (group g = lane/16, s = lane%16): token row
  // 8 (g>>1) + 4 r + (s>>2) of the stage; column group: the rho32-permuted one on the column
  // side (4 * colgrp), natural order 16 (g&1) + 4 (s&3) on the hidden-unit side.
  const int g = lane >> 4, sl = lane & 15;
  const int sw = ((sl >> 2) & 3) << 2;  // ((krow & 3) << 2): krow & 3 = (s >> 2) & 3
  const int ag = sl & 3;
  const int acol = 4 * (4 * (ag & 1) + 2 * (g & 1) + (ag >> 1));
  const int bcol = 16 * (g & 1) + 4 * (sl & 3);
  const int krow0 = 8 * (g >> 1) + (sl >> 2);
  const int swb = UT == 128 ? sw : ((krow0 >> 1) & 1) << 2;
  uint32_t a_off[MI], b_off[2];  // byte offsets of the r = 0 read inside a stage
#pragma unroll
  for (int mi = 0; mi < MI; ++mi)
    a_off[mi] = (uint32_t)(krow0 * 512 + ((((wm * MI + mi) * 4 + (acol >> 3)) ^ sw) * 16) +
                           (acol & 4) * 2);
#pragma unroll
  for (int ni = 0; ni < 2; ++ni)
    b_off[ni] = (uint32_t)(DW_A_BYTES + krow0 * (2 * UT) + ((((wn * 2 + ni) * 4 + (bcol >> 3)) ^ swb) * 16) + (bcol & 4) * 2);
  const char* ring = reinterpret_cast<const char*>(dw_smem);
  auto load_frag = [&](const char* st, int f) -> bf16x8 {  // f < MI: column tile f; else unit tile f - MI
    if (f < MI) return tr_read_frag(st + a_off[f], st + a_off[f] + 4 * 512);
    return tr_read_frag(st + b_off[f - MI], st + b_off[f - MI] + 4 * (2 * UT));
  };

  f32x16 acc[MI][2];
#pragma unroll
  for (int mi = 0; mi < MI; ++mi)
#pragma unroll
    for (int ni = 0; ni < 2; ++ni)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[mi][ni][v] = 0.f;

  bf16x8 fa[2][MI], fb[2][2];
  int ids[2] = {0, 0};
  if (nk > 0) {
    fetch_ids(0);
    fetch_ids(1);
    wait_vmcnt<0>();
#pragma unroll
    for (int st = 0; st < LA; ++st) {
      const int ks = st < klast ? st : klast;
      load_ids(ks, ids);
      issue_a(0, st, ids);
      issue_a(1, st, ids);
      issue_b(st, ks);
    }
    load_ids(LA < klast ? LA : klast, ids);
    // issues 0 and 1 have landed (the LA - 2 later ones may be out: 3 instructions each)
    wait_vmcnt<3 * (LA - 2)>();
    __builtin_amdgcn_s_barrier();
#pragma unroll
    for (int f = 0; f < MI; ++f) fa[0][f] = load_frag(ring, f);
#pragma unroll
    for (int f = 0; f < 2; ++f) fb[0][f] = load_frag(ring, f + MI);
  }
  // One iteration; cur says which fragment buffer holds stage kt (a compile-time constant, so
  // the buffers stay in registers: the loop below is unrolled by two).
  auto iteration = [&](int kt, int slot, auto cur_tag) {
    constexpr int cur = decltype(cur_tag)::value;
    const int next_slot = (slot + 1 == DW_SLOTS) ? 0 : slot + 1;
    const int fill = (slot == 0) ? DW_SLOTS - 1 : slot - 1;  // slot of stage kt-1 = that of stage kt+LA
    // after the last stage the look-ahead reads the current one again: harmless
    const char* st1 = ring + ((kt + 1 < nk) ? next_slot : slot) * DW_STAGE_BYTES;
    const int kfill = kt + LA < klast ? kt + LA : klast;
    const int kids = kt + LA + 1 < klast ? kt + LA + 1 : klast;
    int ids_next[2] = {0, 0};
#pragma unroll
    for (int m = 0; m < 2 * MI; ++m) {
      const int mi = m >> 1, ni = m & 1;
      acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[cur][mi], fb[cur][ni], acc[mi][ni], 0, 0, 0);
      if (m == 2) {
        issue_b(fill, kfill);
        if (((kt + LA + 1) & 15) == 0 && kt + LA + 1 < klast) fetch_ids((kt + LA + 1) / 16 + 1);  // (over the group that has been read to its end)
        load_ids(kids, ids_next);
      }
      if (m < 2) issue_a(m, fill, ids);
      else if (m < MI + 2) fa[cur ^ 1][m - 2] = load_frag(st1, m - 2);
      else fb[cur ^ 1][m - MI - 2] = load_frag(st1, m - 2);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (2 * MI < MI + 4) {  // 64-unit tiles: 4 MFMAs only, the hidden-unit fragments follow them
      fb[cur ^ 1][0] = load_frag(st1, MI);
      fb[cur ^ 1][1] = load_frag(st1, MI + 1);
      __builtin_amdgcn_sched_barrier(0);
    }
    ids[0] = ids_next[0];
    ids[1] = ids_next[1];
    // own copies of stage kt+2 have landed: only issues kt+3 .. kt+LA (3 instructions each) may
    // be outstanding; the barrier makes everyone's visible and ends all reads of stage kt
    wait_vmcnt<3 * (LA - 2)>();
    __builtin_amdgcn_s_barrier();
  };
  int slot = 0;
  for (int kt = 0; kt < nk; kt += 2) {
    iteration(kt, slot, std::integral_constant<int, 0>{});
    slot = (slot + 1 == DW_SLOTS) ? 0 : slot + 1;
    if (kt + 1 < nk) {
      iteration(kt + 1, slot, std::integral_constant<int, 1>{});
      slot = (slot + 1 == DW_SLOTS) ? 0 : slot + 1;
    }
  }
  wait_vmcnt<0>();  // the trailing copies (repeats of the last stage) are done too
  __builtin_amdgcn_s_barrier();  // ... everyone's: the ring is free

  // Lane (i, h) holds, for hidden unit u0 + 64 wn + 32 ni + i, the columns
  // c0 + 32 MI wm + 32 mi + 16 h + (0..15): stored as they are, an instruction would touch 64
  // lines with 16 bytes each.  Each 32 x 32 tile goes through a wavefront-private LDS buffer
  // (rows of 144 bytes) instead, and comes back with 8 lanes along a row, so a store instruction
  // writes 8 whole 128-byte lines.  (Same wavefront on both sides: LDS executes its accesses in order.)
  float* tbuf = reinterpret_cast<float*>(dw_smem) + wave * (32 * 36);
  const int cc = lane & 7, r0 = lane >> 3;
#pragma unroll
  for (int mi = 0; mi < MI; ++mi)
#pragma unroll
    for (int ni = 0; ni < 2; ++ni) {
      const f32x16& v = acc[mi][ni];
#pragma unroll
      for (int e = 0; e < 4; ++e)
        *reinterpret_cast<f32x4*>(tbuf + i * 36 + 16 * h + 4 * e) = f32x4{v[4 * e], v[4 * e + 1], v[4 * e + 2], v[4 * e + 3]};
      wave_lds_fence();
      const int c = c0 + wm * CPW + mi * 32 + 4 * cc;
      f32x4 o[4];  // (all four reads go out before the first store waits for its data)
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = *reinterpret_cast<const f32x4*>(tbuf + (r0 + 8 * e) * 36 + 4 * cc);
      wave_lds_fence();
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int u = u0 + wn * 64 + ni * 32 + r0 + 8 * e;
        if (u < Bs && c < d) *reinterpret_cast<f32x4*>(dst + (size_t)u * d + c) = o[e];
      }
    }
}

}  // namespace spt
