// Low-rank adapted routed FFN (paper section 2.2: a projection Y = XW becomes X(W + BC) with W
// frozen; section 4.2 routing on top): the small kernels around the big GEMMs.
//
// With rank r <= 32 every adapter term is a product through a 32-wide bottleneck, so it is kept
// out of the big GEMMs' way instead of being merged into the weights:
//   inner projection   hpre += C1_b^T (A1^T x):  U = X A1 is computed once per token
//                      (lora_proj) and enters the K = d GEMM as 64 more K-values (each of the
//                      32 padded ranks as a bf16 value plus a bf16 remainder);
//   outer projection   y += C2^T (sum_b B2_b^T h_b): per pair Sp = H B2_b (lora_pair_gemm); the
//                      sum over a token's pairs, times C2, is added where the token's partial rows
//                      are combined (wide blocks) or written as one row more to add (lora_expand);
//   backward           the transposes of the same three steps, and the four adapter gradients,
//                      contractions over rows with a 32-wide side, in one launch (lora_grads).
// All adapter operands are first copied into zero-padded bf16 panels with 32 in place of r
// (lora_setup), so no kernel below has a ragged rank dimension.
//
// Every kernel here reads an activation-sized tensor once and does little with it: bandwidth is the
// bound, and what keeps one away from it is too few loads in flight and the launches themselves.
#include "ffn_common.hpp"
#include "spt_host.hpp"
#include "profile.hpp"

namespace spt {

// Panels: dst[a][b] (drows x dcols, bf16) = transpose ? src[b'][a] : src[a][b'] with b' = b, or b % 32
// when dup is set (a 32-wide panel repeated in columns 32..63); zero outside src (srows x scols).
// frag: the panel (drows = 32 ranks, a K axis of dcols) in the order its readers' lanes want it, [dcols / 32][rank / 16]
// [lane][8], lane (rank % 16, K-group lane / 16): an operand of v_mfma_f32_16x16x32_bf16 is then one contiguous kilobyte.
// Pieces (blockIdx.y past the panels): buckets cut into pieces of at most `piece` rows, so that the
// K = bucket rows adapter gradients run as many short contractions instead of a few long ones.
// first[b] = index of b's first piece (first[N] = total), off[p] / off[p+1] = the row range of piece p;
// unused pieces up to max_pieces are empty ranges at the end.
__global__ __launch_bounds__(256) void lora_setup_kernel(PadJobs jobs, int njobs, PieceTable pt) {
  if ((int)blockIdx.y == njobs) {
    if (blockIdx.x > 0) return;
    __shared__ int32_t wtot[16];
    int base = 0;
    for (int b0 = 0; b0 < pt.N; b0 += 256) {
      const int b = b0 + (int)threadIdx.x;
      const int o0 = b < pt.N ? pt.offsets[b] : 0;
      const int m = b < pt.N ? pt.offsets[b + 1] - o0 : 0;
      const int np = (m + pt.piece - 1) / pt.piece;
      int total;
      const int begin = base + block_inclusive_sum(np, wtot, total) - np;
      if (b < pt.N) {
        pt.first[b] = begin;
        for (int p = 0; p < np; ++p) pt.off[begin + p] = o0 + p * pt.piece;
      }
      base += total;
    }
    if (threadIdx.x == 0) pt.first[pt.N] = base;
    const int last_row = pt.offsets[pt.N];
    for (int p = base + (int)threadIdx.x; p <= pt.max_pieces; p += 256) pt.off[p] = last_row;
    return;
  }
  const PadJob j = jobs.job[blockIdx.y];
  const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (id >= (int64_t)j.drows * j.dcols) return;
  int a = (int)(id / j.dcols), b = (int)(id % j.dcols);
  if (j.frag) {
    const int e = (int)(id & 7), ln = (int)(id >> 3) & 63, n = (int)(id >> 9) & 1;
    a = 16 * n + (ln & 15);
    b = (int)(id >> 10) * 32 + 8 * (ln >> 4) + e;
  }
  if (j.dup) b &= 31;
  const int sr = j.transpose ? b : a, sc = j.transpose ? a : b;
  j.dst[id] = (sr < j.srows && sc < j.scols) ? j.src[(size_t)sr * j.scols + sc] : (uint16_t)0;
}

// S[t][rho] = sum_i Act[t][i] * panel[rho][i], rho < 32, written as TWO bf16 numbers: the rounded
// value in column rho and the rounded remainder in column 32 + rho of the 64-wide row, so the
// pair carries about 16 mantissa bits.  (With one bf16 the 2^-9 rounding of this term would be
// enough to flip the sign of pre-activations near zero, which ReLU's derivative turns into
// visible gradient errors.)  The row goes to [token] and / or to the sorted positions of the token's pairs.
// A workgroup owns 32 tokens; its eight wavefronts split d eight ways (both operands straight from global memory,
// sixteen 16-byte loads in flight per lane) and add their parts through LDS in wave order.  v_mfma_f32_16x16x32_bf16
// rather than 32x32x16: a load then takes 64 bytes of each of 16 rows instead of 32 bytes of 32.
// (Four wavefronts with eight loads: 12.2 us for 8192 x 2048 values, and one launch for each of the backward
// pass's two products.)
__global__ __launch_bounds__(512, 4) void lora_proj_kernel(ProjJob j0, ProjJob j1, const int32_t* __restrict__ inv,
                                                           int T, int d, int k) {
  __shared__ f32x4 red[8][4][64];
  __shared__ uint4 rows4[32 * 8];
  const ProjJob job = blockIdx.y ? j1 : j0;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int i = lane & 15, g = lane >> 4;
  const int t0 = blockIdx.x * 32;
  const int steps = d / 32, per = (steps + 7) / 8;
  const int s0 = wave * per, s1 = s0 + per < steps ? s0 + per : steps;
  const uint16_t* arow[2];
#pragma unroll
  for (int m = 0; m < 2; ++m)   // (rows past the end are computed but never stored)
    arow[m] = job.act + (size_t)min(t0 + 16 * m + i, T - 1) * d + 8 * g;
  const uint16_t* prow = job.panel + lane * 8;
  f32x4 acc[2][2];
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int n = 0; n < 2; ++n) acc[m][n] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int s = s0; s < s1; s += 4) {
    uint4 a[4][2], b[4][2];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const bool ok = s + e < s1;
#pragma unroll
      for (int m = 0; m < 2; ++m) {
        a[e][m] = ok ? *reinterpret_cast<const uint4*>(arow[m] + (s + e) * 32) : make_uint4(0, 0, 0, 0);
        b[e][m] = ok ? *reinterpret_cast<const uint4*>(prow + (size_t)((s + e) * 2 + m) * 512) : make_uint4(0, 0, 0, 0);
      }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int n = 0; n < 2; ++n)
          acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(b[e][n]), as_bf16x8(a[e][m]), acc[m][n], 0, 0, 0);
  }
  // lane (token i of 16, g) holds ranks 16 n + 4 g + e of token 16 m + i in acc[m][n][e]
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int n = 0; n < 2; ++n) red[wave][2 * m + n][lane] = acc[m][n];
  __syncthreads();
  uint16_t* rows = reinterpret_cast<uint16_t*>(rows4);
  if (tid < 256) {
    const int mn = tid >> 6;
    f32x4 sum = red[0][mn][lane];
#pragma unroll
    for (int w = 1; w < 8; ++w) sum += red[w][mn][lane];
    uint16_t* at = rows + (16 * (mn >> 1) + i) * 64 + 16 * (mn & 1) + 4 * g;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t hi = f32_to_bf16_bits(sum[e]);
      at[e] = (uint16_t)hi;
      at[32 + e] = (uint16_t)f32_to_bf16_bits(sum[e] - bf16_to_f32((uint16_t)hi));
    }
  }
  __syncthreads();
  const int nrow = T - t0 < 32 ? T - t0 : 32;
  if (job.by_token)
    for (int e = tid; e < nrow * 8; e += 512) reinterpret_cast<uint4*>(job.by_token + (size_t)t0 * 64)[e] = rows4[e];
  if (job.by_pair)
    for (int e = tid; e < nrow * k * 8; e += 512) {
      const int pr = e >> 3, row = pr / k;
      reinterpret_cast<uint4*>(job.by_pair + (size_t)inv[(size_t)t0 * k + pr] * 64)[e & 7] = rows4[row * 8 + (e & 7)];
    }
}

// Per pair: Sp[q][rho] = sum_u Hin[q][u] * panel[rho][b*Bs + u], b the bucket of sorted position q.
// Where a group of positions straddles buckets it makes one masked pass per bucket.
// Narrow blocks (fragment order): a wavefront takes 32 positions, whose at most four K-steps are contiguous half
// kilobytes.  Wide blocks: a workgroup takes 64 positions, its eight wavefronts an eighth of the block's
// hidden units each, added through LDS in wave order.  (Four wavefronts on 32 positions, one load of each operand in
// flight: 28 us for 16384 pairs x 2048 units.)
__device__ __forceinline__ int bucket_of(const int32_t* __restrict__ offsets, int N, int q) {
  int lo = 0, hi = N;  // the largest b with offsets[b] <= q
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (offsets[mid] <= q) lo = mid; else hi = mid;
  }
  return lo;
}

__global__ __launch_bounds__(256) void lora_pair_narrow_kernel(PairJob j0, PairJob j1,
                                                               const int32_t* __restrict__ offsets, int N, int Bs,
                                                               int P) {
  const PairJob job = blockIdx.y ? j1 : j0;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, i = lane & 15, g = lane >> 4;
  const int qbase = (blockIdx.x * 4 + wave) * 32;
  const int qstop = (qbase + 32 < P) ? qbase + 32 : P;
  for (int q = qbase; q < qstop;) {
    const int b = bucket_of(offsets, N, q);
    const int qe = min(qstop, offsets[b + 1]);
    const uint16_t* prow = job.panel + (size_t)b * (Bs / 32) * 1024 + lane * 8;
    uint4 hv[4][2], wv[4][2];
#pragma unroll
    for (int s = 0; s < 4; ++s) {   // (Bs is at most 128)
      const bool ok = 32 * s < Bs;
#pragma unroll
      for (int m = 0; m < 2; ++m) {
        const int row = qbase + 16 * m + i, hq = row >= q && row < qe ? row : q;
        hv[s][m] = ok ? *reinterpret_cast<const uint4*>(job.hin + hfrag_off(hq, 32 * s + 8 * g, Bs)) : make_uint4(0, 0, 0, 0);
        wv[s][m] = ok ? *reinterpret_cast<const uint4*>(prow + (size_t)(2 * s + m) * 512) : make_uint4(0, 0, 0, 0);
      }
    }
    // A operand: rows rho (panel), B operand: columns = sorted positions (Hin); lane (position i of 16, g) gets
    // rho = 16 n + 4 g + e
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      const int row = qbase + 16 * m + i;
#pragma unroll
      for (int n = 0; n < 2; ++n) {
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < 4; ++s)
          acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(wv[s][n]), as_bf16x8(hv[s][m]), acc, 0, 0, 0);
        if (row >= q && row < qe) *reinterpret_cast<f32x4*>(job.out + (size_t)row * 32 + 16 * n + 4 * g) = acc;
      }
    }
    q = qe;
  }
}

__global__ __launch_bounds__(512, 4) void lora_pair_wide_kernel(PairJob j0, PairJob j1,
                                                                const int32_t* __restrict__ offsets, int N, int Bs,
                                                                int P) {
  __shared__ f32x4 red[8][8][64];
  const PairJob job = blockIdx.y ? j1 : j0;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, i = lane & 15, g = lane >> 4;
  const int qbase = blockIdx.x * 64;
  const int qstop = (qbase + 64 < P) ? qbase + 64 : P;
  const int steps = Bs / 32, per = (steps + 7) / 8;
  const int s0 = wave * per, s1 = s0 + per < steps ? s0 + per : steps;
  for (int q = qbase; q < qstop;) {
    const int b = bucket_of(offsets, N, q);
    const int qe = min(qstop, offsets[b + 1]);
    const uint16_t* hrow[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const int row = qbase + 16 * m + i;
      hrow[m] = job.hin + (size_t)(row >= q && row < qe ? row : q) * Bs + 8 * g;
    }
    const uint16_t* prow = job.panel + (size_t)b * steps * 1024 + lane * 8;
    f32x4 acc[4][2];
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
      for (int n = 0; n < 2; ++n) acc[m][n] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int s = s0; s < s1; s += 2) {
      uint4 hv[2][4], wv[2][2];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const bool ok = s + e < s1;
#pragma unroll
        for (int n = 0; n < 2; ++n)
          wv[e][n] = ok ? *reinterpret_cast<const uint4*>(prow + (size_t)((s + e) * 2 + n) * 512) : make_uint4(0, 0, 0, 0);
#pragma unroll
        for (int m = 0; m < 4; ++m)
          hv[e][m] = ok ? *reinterpret_cast<const uint4*>(hrow[m] + (s + e) * 32) : make_uint4(0, 0, 0, 0);
      }
#pragma unroll
      for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
          for (int n = 0; n < 2; ++n)
            acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(wv[e][n]), as_bf16x8(hv[e][m]), acc[m][n], 0, 0, 0);
    }
    __syncthreads();  // the previous pass has been read out
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
      for (int n = 0; n < 2; ++n) red[wave][2 * m + n][lane] = acc[m][n];
    __syncthreads();
    // lane (position i of 16, g) holds rho = 16 n + 4 g + e of position 16 m + i: wavefront 2 m + n adds its tile
    const int row = qbase + 16 * (wave >> 1) + i;
    if (row >= q && row < qe) {
      f32x4 sum = red[0][wave][lane];
#pragma unroll
      for (int w = 1; w < 8; ++w) sum += red[w][wave][lane];
      *reinterpret_cast<f32x4*>(job.out + (size_t)row * 32 + 16 * (wave & 1) + 4 * g) = sum;
    }
    q = qe;
  }
}

// Low-rank term of an outer projection: S[t] = sum_j Sp[inv[t*k + j]], j ascending, rounded to bf16, times
// panel[c][rho] (rho < 32).  COMBINE: added to the sum of the token's k partial rows (j ascending, as the plain
// combine adds them) and written as the result; else written by itself, one more row for the token-range kernel
// to add.  Sb (optional) keeps the rounded S for the weight gradients, and Sb2 that of a second tensor Sp2.
// A wavefront takes 16 tokens x 128 columns: v_mfma_f32_16x16x32_bf16 has K = 32, the whole rank; the columns are
// its rows, two products interleaved so that a lane ends up with 8 consecutive columns of its token: partial rows and
// result are then read and written 64 bytes per token and instruction.  (Two passes with a token-sum launch between,
// lanes holding 16-byte pieces 32 bytes apart: 19 + 28 + 5 us for 8192 x 2048 values, k = 2.)
template <bool COMBINE>
__global__ __launch_bounds__(256) void lora_expand_kernel(const float* __restrict__ Sp, const uint16_t* __restrict__ panel,
                                                          const int32_t* __restrict__ inv, int T, int d, int k,
                                                          const uint16_t* __restrict__ part, uint16_t* __restrict__ out,
                                                          uint16_t* __restrict__ Sb, const float* __restrict__ Sp2,
                                                          uint16_t* __restrict__ Sb2) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int tl = lane & 15, g = lane >> 4;
  const int t0 = blockIdx.x * 16, c0 = (blockIdx.y * 4 + wave) * 128;
  if (c0 >= d) return;
  const bool live = t0 + tl < T;
  const int32_t* iv = inv + (size_t)(live ? t0 + tl : T - 1) * k;
  auto token_sum = [&](const float* src) -> uint4 {
    f32x4 lo = {0.f, 0.f, 0.f, 0.f}, hi = lo;
#pragma unroll 4
    for (int j = 0; j < k; ++j) {
      const f32x4* row = reinterpret_cast<const f32x4*>(src + (size_t)iv[j] * 32 + 8 * g);
      lo += row[0];
      hi += row[1];
    }
    return make_uint4(pack_bf16x2(lo[0], lo[1]), pack_bf16x2(lo[2], lo[3]), pack_bf16x2(hi[0], hi[1]),
                      pack_bf16x2(hi[2], hi[3]));
  };
  float a[4][8];
#pragma unroll
  for (int ct = 0; ct < 4; ++ct)
#pragma unroll
    for (int e = 0; e < 8; ++e) a[ct][e] = 0.f;
  if (COMBINE) {
    const uint16_t* pc = part + c0 + 8 * g;
    auto add = [&](const u32x4 (&v)[4]) {
#pragma unroll
      for (int ct = 0; ct < 4; ++ct)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          a[ct][2 * e] += lo_bf16(v[ct][e]);
          a[ct][2 * e + 1] += hi_bf16(v[ct][e]);
        }
    };
    auto load = [&](int j, u32x4 (&v)[4]) {
      const uint16_t* row = pc + (size_t)iv[j] * d;
#pragma unroll
      for (int ct = 0; ct < 4; ++ct)
        v[ct] = c0 + 32 * ct < d ? __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(row + 32 * ct)) : u32x4{0, 0, 0, 0};
    };
    u32x4 v0[4], v1[4];
    int j = 0;
    for (; j + 2 <= k; j += 2) {
      load(j, v0);
      load(j + 1, v1);
      add(v0);
      add(v1);
    }
    if (j < k) {
      load(j, v0);
      add(v0);
    }
  }
  const uint4 s = token_sum(Sp);
  const bool keeper = blockIdx.y == 0 && wave == 0 && live;
  if (Sb && keeper) reinterpret_cast<uint4*>(Sb + (size_t)(t0 + tl) * 32)[g] = s;
  if (Sb2 && keeper) reinterpret_cast<uint4*>(Sb2 + (size_t)(t0 + tl) * 32)[g] = token_sum(Sp2);
#pragma unroll
  for (int ct = 0; ct < 4; ++ct) {
    const int c = c0 + ct * 32;
    if (c >= d) break;  // d is a multiple of 64, tiles are 32 wide: whole tiles only
    // MFMA row r of product m is column c + 8 (r >> 2) + 4 m + (r & 3): lane (token tl, g) gets c + 8 g + 4 m + e
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      const uint16_t* prow = panel + (size_t)(c + 8 * (tl >> 2) + 4 * m + (tl & 3)) * 32 + 8 * g;
      f32x4 z = {0.f, 0.f, 0.f, 0.f};
      z = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(*reinterpret_cast<const uint4*>(prow)), as_bf16x8(s), z, 0, 0, 0);
#pragma unroll
      for (int e = 0; e < 4; ++e) a[ct][4 * m + e] += z[e];
    }
    if (live)
      *reinterpret_cast<uint4*>(out + (size_t)(t0 + tl) * d + c + 8 * g) =
          make_uint4(pack_bf16x2(a[ct][0], a[ct][1]), pack_bf16x2(a[ct][2], a[ct][3]), pack_bf16x2(a[ct][4], a[ct][5]),
                     pack_bf16x2(a[ct][6], a[ct][7]));
  }
}

// Contractions over rows with a narrow side: out[piece][u][rho] = sum over the piece's rows q of H[q][u] * R[q][rho],
// u up to an activation's width, rho 32 or 64 wide (FOLD: the two 32-wide halves of a value | remainder panel are
// added).  Bound by reading H once; the matrix cores have little to do.  A workgroup takes 128 units, its four
// wavefronts a quarter of the piece's rows each, and every wavefront runs a ring of its own -- 16 rows a stage, three
// stages, filled by LDS DMA, read back with the transposing ds_read_b64_tr_b16 -- so no barrier stands between the
// stages; two workgroups per CU keep 96 KiB in flight.  The four sums are added through LDS in wave order.
// (As weight-gradient GEMMs with a 256-column side, of which 64 were wanted, or 128 workgroups: 2 x 35 and
// 2 x 19 us for 16384 pairs x 2048 units and 8192 tokens x 2048 columns.)
constexpr int GR_UNITS = 128;
constexpr int GR_WAVE = GR_UNITS * 36 * 4;     // bytes of a wavefront: the ring, then its sums as rows of 36 words
constexpr int GR_SMEM = 4 * GR_WAVE;           // 72 KiB

template <bool FRAG, int RT, bool FOLD>
__device__ __forceinline__ void grad_tile(const GradJob& jb, int piece, int u0, int r0, char* smem,
                                          const uint16_t* __restrict__ zero_row) {
  constexpr int STAGE = 4096 + RT * 1024;      // 16 rows x 128 units, 16 rows x 32 RT ranks
  constexpr int NI = 4 + RT;                   // copies per stage
  static_assert(3 * STAGE <= GR_WAVE, "the ring fits the wavefront's LDS");
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i = lane & 31, h = lane >> 5, g = lane >> 4, sl = lane & 15;
  const int qb = jb.off ? jb.off[piece] : piece * jb.piece;
  const int qe = jb.off ? jb.off[piece + 1] : (qb + jb.piece < jb.rows ? qb + jb.piece : jb.rows);
  if (qb >= qe) return;                        // (an unused piece: nobody reads its slot)
  const int per = ((qe - qb + 63) / 64) * 16;
  const int wb = qb + wave * per, we = wb + per < qe ? wb + per : qe;
  const int nk = wb < we ? (we - wb + 15) / 16 : 0;
  char* ring = smem + wave * GR_WAVE;
  const uint32_t lds0 = (uint32_t)(uintptr_t)ring;

  auto issue = [&](int kt, int slot) {         // stage min(kt, nk - 1): the number of copies in flight stays the same
    const int q0 = wb + (kt < nk ? kt : nk - 1) * 16;
    const uint32_t dst = __builtin_amdgcn_readfirstlane(lds0 + (uint32_t)(slot * STAGE));
#pragma unroll
    for (int j = 0; j < 4; ++j) {              // rows 4 j + lane / 16, chunk lane % 16 ^ swizzle
      const int row = 4 * j + (lane >> 4), q = q0 + row;
      int col = u0 + (((lane & 15) ^ ((row & 3) << 2)) << 3);
      if (col >= jb.units) col = u0;           // past the end: harmless duplicate, never stored
      dma16(q < we ? jb.H + hval_off<FRAG>(q, col, jb.units) : zero_row + ((lane & 15) << 3), dst + j * 1024);
    }
#pragma unroll
    for (int j = 0; j < RT; ++j) {
      const int row = RT == 2 ? 8 * j + (lane >> 3) : lane >> 2;
      int col = r0 + (RT == 2 ? ((lane & 7) ^ (((row >> 1) & 1) << 2)) << 3 : (lane & 3) << 3);
      if (col >= jb.ldr) col = r0;
      const int q = q0 + row < we ? q0 + row : we - 1;   // (past the end: times a zero row of H)
      dma16(jb.R + (size_t)q * jb.ldr + col, dst + 4096 + j * 1024);
    }
  };

  // Fragment addresses: rank side through the permuted columns (a lane then holds 16 consecutive ranks of its
  // unit), unit side in natural order.
  const int krow = 8 * (g >> 1) + (sl >> 2), ag = sl & 3;
  const int acol = 4 * (4 * (ag & 1) + 2 * (g & 1) + (ag >> 1)), bcol = 16 * (g & 1) + 4 * ag;
  constexpr int RROW = RT * 64;                // bytes of a row of the rank side
  const int sw_r = RT == 2 ? ((krow >> 1) & 1) << 2 : 0, sw_u = (krow & 3) << 2;
  f32x16 acc[RT][4];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int ut = 0; ut < 4; ++ut)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[rt][ut][v] = 0.f;
  if (nk > 0) {
#pragma unroll
    for (int s = 0; s < 3; ++s) issue(s, s);
    int slot = 0;
    for (int kt = 0; kt < nk; ++kt) {
      wait_vmcnt<2 * NI>();                    // stage kt is in, the two after it may be out
      const char* st = ring + slot * STAGE;
      bf16x8 fr[RT], fu[4];
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        const char* at = st + 4096 + krow * RROW + (((rt * 4 + (acol >> 3)) ^ sw_r) * 16) + (acol & 4) * 2;
        fr[rt] = tr_read_frag(at, at + 4 * RROW);
      }
#pragma unroll
      for (int ut = 0; ut < 4; ++ut) {
        const char* at = st + krow * 256 + (((ut * 4 + (bcol >> 3)) ^ sw_u) * 16) + (bcol & 4) * 2;
        fu[ut] = tr_read_frag(at, at + 4 * 256);
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // read before the slot is filled again
      issue(kt + 3, slot);
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int ut = 0; ut < 4; ++ut)
          acc[rt][ut] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[rt], fu[ut], acc[rt][ut], 0, 0, 0);
      slot = slot == 2 ? 0 : slot + 1;
    }
    wait_vmcnt<0>();                           // the trailing copies are done before the sums take their place
  }
  float* mine = reinterpret_cast<float*>(ring);
  constexpr int OUT = FOLD ? 1 : RT;
#pragma unroll
  for (int rt = 0; rt < OUT; ++rt) {
    if (rt > 0) __syncthreads();
#pragma unroll
    for (int ut = 0; ut < 4; ++ut)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        f32x4 o;
#pragma unroll
        for (int x = 0; x < 4; ++x)
          o[x] = FOLD && RT == 2 ? acc[0][ut][4 * e + x] + acc[RT - 1][ut][4 * e + x] : acc[rt][ut][4 * e + x];
        *reinterpret_cast<f32x4*>(mine + (ut * 32 + i) * 36 + 16 * h + 4 * e) = o;
      }
    __syncthreads();
    if (r0 + 32 * rt >= jb.ldo) continue;      // (workgroup-uniform)
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const int id = tid + 256 * m, unit = id >> 3, c4 = id & 7;
      const float* p = reinterpret_cast<const float*>(smem) + unit * 36 + 4 * c4;
      f32x4 s = *reinterpret_cast<const f32x4*>(p);
#pragma unroll
      for (int w = 1; w < 4; ++w) s += *reinterpret_cast<const f32x4*>(p + w * (GR_WAVE / 4));
      if (u0 + unit < jb.units)
        *reinterpret_cast<f32x4*>(jb.out + ((size_t)piece * jb.units + u0 + unit) * jb.ldo + r0 + 32 * rt + 4 * c4) = s;
    }
  }
}

// All four adapter gradients: jobs 0, 1 over the pairs of each bucket (value | remainder panels), 2, 3 over the tokens.
template <bool FRAG>
__global__ __launch_bounds__(256, 2) void lora_grads_kernel(GradJobs jobs, const uint16_t* __restrict__ zero_row) {
  extern __shared__ uint4 gr_smem[];
  int id = blockIdx.x, j = 0;
  while (j < 3 && id >= jobs.job[j].npieces * jobs.job[j].tiles) {
    id -= jobs.job[j].npieces * jobs.job[j].tiles;
    ++j;
  }
  const GradJob jb = jobs.job[j];
  const int piece = id % jb.npieces, u0 = id / jb.npieces * GR_UNITS;
  char* smem = reinterpret_cast<char*>(gr_smem);
  if (j < 2) grad_tile<FRAG, 2, true>(jb, piece, u0, 0, smem, zero_row);
  else       grad_tile<false, 1, true>(jb, piece, u0, 0, smem, zero_row);
}

// One such contraction with a rank side of any width, 64 columns per workgroup (the route network's weight gradient).
__global__ __launch_bounds__(256, 2) void row_contraction_kernel(GradJob jb, const uint16_t* __restrict__ zero_row) {
  extern __shared__ uint4 gr_smem[];
  grad_tile<false, 2, false>(jb, blockIdx.x % jb.npieces, blockIdx.x / jb.npieces * GR_UNITS, blockIdx.y * 64,
                             reinterpret_cast<char*>(gr_smem), zero_row);
}

// The staged pieces added in order: for unit u of block b and rank rho the sum over b's pieces (first[b] ..
// first[b+1], or all of them) of stage[.][u][rho], written as out[rho][b*units + u] (transpose) or out[b*units + u][rho].
__global__ __launch_bounds__(256) void lora_reduce_kernel(GradJobs jobs, int r) {
  const GradJob jb = jobs.job[blockIdx.y];
  const int64_t id = (int64_t)blockIdx.x * 256 + threadIdx.x, total = (int64_t)jb.nblocks * jb.units;
  const int rho = (int)(id & 31);
  const int64_t unit = id >> 5;
  if (unit >= total || rho >= r) return;
  const int b = (int)(unit / jb.units), u = (int)(unit % jb.units);
  const int p0 = jb.first ? jb.first[b] : 0, p1 = jb.first ? jb.first[b + 1] : jb.npieces;
  const float* src = jb.out + (size_t)u * 32 + rho;
  const size_t stride = (size_t)jb.units * 32;
  float s = 0.f;
  int p = p0;
  for (; p + 8 <= p1; p += 8) {   // eight values are requested before the first is added
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = src[(size_t)(p + e) * stride];
#pragma unroll
    for (int e = 0; e < 8; ++e) s += v[e];
  }
#pragma unroll 4
  for (; p < p1; ++p) s += src[(size_t)p * stride];
  if (jb.transpose) jb.result[(size_t)rho * total + unit] = s;
  else jb.result[(size_t)unit * r + rho] = s;
}

hipError_t lora_setup(const PadJobs& jobs, int njobs, const PieceTable* pieces, hipStream_t st) {
  int64_t n = 0;
  for (int j = 0; j < njobs; ++j) {
    const int64_t m = (int64_t)jobs.job[j].drows * jobs.job[j].dcols;
    if (m > n) n = m;
  }
  lora_setup_kernel<<<dim3((unsigned)((n + 255) / 256), njobs + (pieces ? 1 : 0)), 256, 0, st>>>(
      jobs, njobs, pieces ? *pieces : PieceTable{});
  return hipGetLastError();
}

hipError_t lora_proj(const ProjJob* jobs, int njobs, const int32_t* inv, int T, int d, int k, hipStream_t st) {
  lora_proj_kernel<<<dim3((T + 31) / 32, njobs), 512, 0, st>>>(jobs[0], jobs[njobs - 1], inv, T, d, k);
  return hipGetLastError();
}

hipError_t lora_pair_gemm(const PairJob* jobs, int njobs, bool narrow, const int32_t* offsets, int N, int Bs, int P,
                          hipStream_t st) {
  const int64_t p = P;
  if (narrow) lora_pair_narrow_kernel<<<dim3((unsigned)((p + 127) / 128), njobs), 256, 0, st>>>(jobs[0], jobs[njobs - 1], offsets, N, Bs, P);
  else lora_pair_wide_kernel<<<dim3((unsigned)((p + 63) / 64), njobs), 512, 0, st>>>(jobs[0], jobs[njobs - 1], offsets, N, Bs, P);
  return hipGetLastError();
}

hipError_t lora_expand(const float* Sp, const uint16_t* panel, const int32_t* inv, int T, int d, int k,
                       const uint16_t* part, uint16_t* out, uint16_t* Sb, const float* Sp2, uint16_t* Sb2, hipStream_t st) {
  const dim3 grid((T + 15) / 16, (d + 511) / 512);
  if (part) lora_expand_kernel<true><<<grid, 256, 0, st>>>(Sp, panel, inv, T, d, k, part, out, Sb, Sp2, Sb2);
  else lora_expand_kernel<false><<<grid, 256, 0, st>>>(Sp, panel, inv, T, d, k, nullptr, out, Sb, Sp2, Sb2);
  return hipGetLastError();
}

hipError_t lora_grads(const GradJobs& jobs, bool frag, int r, const uint16_t* zero_row, hipStream_t st) {
  static const hipError_t attr[2] = {
      hipFuncSetAttribute(reinterpret_cast<const void*>(lora_grads_kernel<false>), hipFuncAttributeMaxDynamicSharedMemorySize, GR_SMEM),
      hipFuncSetAttribute(reinterpret_cast<const void*>(lora_grads_kernel<true>), hipFuncAttributeMaxDynamicSharedMemorySize, GR_SMEM)};
  if (attr[frag] != hipSuccess) return attr[frag];
  unsigned grid = 0;
  int64_t most = 0;
  for (int j = 0; j < 4; ++j) {
    const GradJob& jb = jobs.job[j];
    grid += (unsigned)(jb.npieces * jb.tiles);
    if ((int64_t)jb.nblocks * jb.units > most) most = (int64_t)jb.nblocks * jb.units;
  }
  if (frag) lora_grads_kernel<true><<<grid, 256, GR_SMEM, st>>>(jobs, zero_row);
  else lora_grads_kernel<false><<<grid, 256, GR_SMEM, st>>>(jobs, zero_row);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  lora_reduce_kernel<<<dim3((unsigned)((most * 32 + 255) / 256), 4), 256, 0, st>>>(jobs, r);
  return hipGetLastError();
}

hipError_t row_contraction(const GradJob& jb, const uint16_t* zero_row, hipStream_t st) {
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(row_contraction_kernel),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, GR_SMEM);
  if (attr != hipSuccess) return attr;
  row_contraction_kernel<<<dim3(jb.npieces * jb.tiles, (jb.ldr + 63) / 64), 256, GR_SMEM, st>>>(jb, zero_row);
  return hipGetLastError();
}

// Rows per piece: as few as 128, more while the pieces would be more than a round and a quarter of the chip at two
// workgroups per CU (longer pieces cost less staging).
int grad_piece_rows(int64_t rows, int blocks, int units) {
  const int tiles = (units + GR_UNITS - 1) / GR_UNITS;
  int64_t piece = 128;
  while ((rows / piece + blocks) * tiles > 640 && piece < rows) piece *= 2;
  return (int)piece;
}

}  // namespace spt
