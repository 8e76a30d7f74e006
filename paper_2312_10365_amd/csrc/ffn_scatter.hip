// K = Bs contraction of the routed FFN for blocks of at most 128 hidden units, with the
// write-back of Algorithm 4 (line 5, block outputs ADDED per token) folded into the GEMM:
//
//   out[t][:] = sum over the blocks b that token t activates, ascending b, of
//               Hin[position of (t, b)][:] * W[b]            (+ Z[t][:], the low-rank term)
//
// forward: Hin = act(H), W = W2, out = Y;  backward: Hin = dHpre, W = W1, out = dX.
//
// The GEMM is token-range stationary.  A workgroup owns R consecutive tokens x 64 output columns
// as an fp32 slab in LDS.  Inside a bucket the sorted positions ascend with the token id, so the
// rows of block b that belong to the workgroup's tokens are one contiguous run
// [rstart[r][b], rstart[r+1][b]) -- about R k / N of them.  A run (cut into records of at most
// 16 NT rows) is one WAVEFRONT's work, and the wavefronts of a workgroup are at different runs:
// wavefront w takes records w, w + 4, ...  It turns the block's 64 weight columns into matrix
// operands once, streams the run's rows past them in tiles of 16 (v_mfma_f32_16x16x32_bf16, rows on
// the register axis) and adds every finished tile into the slab rows of its tokens.  Nothing is
// shared between wavefronts but the slab, so there is no barrier in the loop.
//
// A token occurs at most once per block, and its sums have a fixed order (no atomics, no partial rows
// in HBM, one rounding to bf16 when the slab is written out):
//   one slab (OWN = false)  blocks in order.  Each wavefront says in LDS up to which token its record is done; a
//                           tile is added once the three records before it are past its last token.  Tokens
//                           ascend in every run, so the four wavefronts follow one another through the slab a
//                           tile or two apart.  A wait is for lower records only and for no more than their end (tokens
//                           are clamped to the range), so it ends, also with a table that is not sorted.  (Looking at the
//                           one record before it alone, the second piece of a long run held up the next block:
//                           blocks of 96 +- 7 rows in records of 96 761 us, now 635.)
//   four slabs (OWN = true) every wavefront has its own, nobody waits, and the four are added at the end,
//                           0 + 1 + 2 + 3.  For ranges of at most 159 tokens: few records to follow one
//                           another, and shorter than what they would wait.
//
// Slab rows are 256 bytes.  Lane (g, i) = (lane / 16, lane % 16) of a tile holds rows 4 g .. + 3 of columns
// 4 i .. + 3 (W columns 4 i + t go to tile t), so a 16-byte access of the wavefront is four whole slab rows:
// no bank conflict whatever the tokens are (with the lanes on the row axis a third of the LDS cycles were).
// LDS writes are what the slab costs: 79 B/clk per CU against 256 for reads, one ds_write_b128 of all four
// SIMDs per 52 clk.  So the weight slice does not pass through LDS: 8-byte loads of 4 columns x 8 units per lane and
// byte permutes make the operand (16 b128 writes and 32 transposing reads per slice instead: 515 -> 497 us).
// Hin is stored in fragment order (ffn_common.hpp): the 16 bytes per K-step of 16 consecutive
// rows are two contiguous half kilobytes, which go straight from global memory into the lanes that own the rows.
//
// Measured, us a launch, the kernel this replaces (four wavefronts at one run, a barrier per run) -> this one: 7B-like
// (T 8192, d 4096, N 128, Bs 128, k 32) 590 -> 497; BERT-large-like (16384, 1024, 64, 64, 16) 124 -> 82; the
// OPT-1.3B-like layer (8192, 2048, 64, 128, 16) 195 -> 165; BERT-base-like (2048, 768, 32, 96, 8) 25 -> 18.
// Then tiles that a record does not hold left out, and the slab's new values written and published earlier (`ALL`, `WRITE` below), us of a
// launch in turn on one box: 7B-like 513 -> 484; the OPT-1.3B-like layer, skewed routing, 162 -> 147; 3001 tokens of the 7B-like layer
// 236 -> 223; 16384 tokens, d 4096, 64 blocks of 96, 12 each 396 -> 378; BERT-large-like as it was.
// What bounds it (8 K-steps): one wavefront per SIMD, because its registers hold the operands of a run and the next one's loads in flight.  It issues
// in 54 % of the cycles, waits for loads, LDS or its turn in 28 % and for a unit in 18 %; the matrix cores are busy in 27 %.  Without the order
// of the records a launch takes 7 % less (7B-like), 19 % (3001 tokens) and 22 % less (BERT-large-like, 4.6 tiles a run: four wavefronts
// that stay nearly two tiles apart do not fit in it), without the slab 15, 19 and 32 %, with all rows in one line of L1 4, 11 and 4 %.
#include <math.h>
#include <stdlib.h>
#include <type_traits>
#include <utility>

#include "ffn_common.hpp"
#include "ffn_dw.hpp"
#include "spt_host.hpp"
#include "profile.hpp"

namespace spt {

constexpr int SC_C = 64;                 // output columns per workgroup
constexpr int SC_STRIDE = SC_C * 4;      // bytes per slab row
constexpr int SC_WAVES = 4;
constexpr int SC_THREADS = 64 * SC_WAVES;
constexpr int SC_CODE = 1024;            // progress codes per record; more than the rows of a slab
constexpr int SC_NONE = -(1 << 29);      // a code that is always reached
constexpr int SC_RSRC = 0x00027000;      // last word of a raw buffer descriptor

__device__ __forceinline__ void sc_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// One wavefront per token range: see compact_runs.
__global__ __launch_bounds__(64) void scatter_runs_kernel(const int32_t* __restrict__ starts, int N, int cap, int run_rows,
                                                          RunRec* __restrict__ runs,
                                                          int32_t* __restrict__ nruns) {
  compact_runs(starts, N, cap, run_rows, runs, nruns, blockIdx.x, threadIdx.x);
}

typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

// Work item of workgroup `wg`: a part of the range's records, a token range and a slab; slab < 0: none.  An XCD (workgroup id mod
// 8) takes an eighth of all items in order, parts included: part after part, in it groups of `inner` slabs, range after
// range of a group, so that what it runs together is a few ranges x inner slabs, which share weight slices and runs of Hin
// rows in its L2.  (With an eighth of the ranges and slabs and all parts of each, 85 of them in three parts were 33 workgroups
// for the 32 CUs of seven XCDs, and a second round: 2100 tokens, d 320, 60 blocks of 128, 24 each 49 us a launch, now 30.)
struct ScatterItem { int part, r, slab; };
__host__ __device__ __forceinline__ ScatterItem scatter_item(int wg, int nslab, int nr, int parts, int inner) {
  const int each = nslab * nr, per = (each * parts + 7) >> 3, item = (wg & 7) * per + (wg >> 3);
  if ((wg >> 3) >= per || item >= each * parts) return ScatterItem{0, 0, -1};
  const int part = parts > 1 ? item / each : 0, in_part = item - part * each;
  const int grp = in_part / (inner * nr), rem = in_part % (inner * nr);
  const int size = nslab - grp * inner < inner ? nslab - grp * inner : inner;
  return ScatterItem{part, rem / size, grp * inner + rem % size};
}
inline int scatter_grid(const ScatterPlan& p) { return 8 * ((p.nslab * p.nr * p.splits + 7) / 8); }

template <class F, int... I>
__device__ __forceinline__ void for_each_index(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}

// KS = Bs / 16.  NT tiles of 16 rows per record, each a slot of the unrolled loop; rows are requested RH tiles ahead.
// LATE: the next weight slice is requested in a record's last slot, not behind its first (64 registers less).
// OWN: a slab per wavefront.
template <int KS, int NT, int RH, bool LATE, bool OWN>
__device__ __forceinline__ void scatter_tile(
    int wg, const uint16_t* __restrict__ Hin, const uint16_t* __restrict__ W, const RunRec* __restrict__ runs,
    const int32_t* __restrict__ nruns, const int32_t* __restrict__ tok, int N, int d, int T, int R,
    int nr, int nslab, int parts, int inner, int cap, uint16_t* __restrict__ out, const uint16_t* __restrict__ Z,
    float* __restrict__ split) {
  constexpr int Bs = KS * 16;
  constexpr int KT = KS / 2;                   // K-steps of 32 hidden units
  // Slots that are gone through whatever the record holds; of the others those without a tile only request the rows that
  // fall to them.  (All loads stay in common code, in one order: the compiler's waits count them.)  Rows requested behind the products and not
  // between them cost less than the empty slots of records of 8 and 10 tiles, but where two workgroups share a CU, and fill each other's gaps, as much or
  // more, us with and without: 4 tiles, 32768 tokens, d 1024, 128 blocks of 32, 16 each 287 / 246; 65536, 512, 32 of 64, 4 95 / 87; 6 tiles,
  // 4000, 1024, 100 of 128, 30 70 / 64; 3000, 256, 100 of 96, 30 24.3 / 22.7; BERT-large-like 92 / 90.
  constexpr int ALL = NT > 6 ? 4 : NT;
  static_assert(ALL == NT || !LATE, "weights are requested in slots that are gone through");
  constexpr int THREADS = SC_THREADS;
  
  extern __shared__ uint4 sc_smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i = lane & 15, g = lane >> 4;

  const ScatterItem item = scatter_item(wg, nslab, nr, parts, inner);
  if (item.slab < 0) return;
  const int slab = item.slab, r = item.r;
  const int t0 = r * R, c0 = slab * SC_C;
  const int rows = (T - t0 < R) ? T - t0 : R;

  const int slab_bytes = (R + 1) * SC_STRIDE;                  // (the last row is the dummy)
  char* const slabs = reinterpret_cast<char*>(sc_smem);
  char* const slab_lds = slabs + (OWN ? wave * slab_bytes : 0);
  // how far each wavefront is: SC_CODE x record + first token of it that is not done, a word per lane
  typedef __attribute__((address_space(3))) int* lds_int_ptr;
  const lds_int_ptr prog = (lds_int_ptr)(uintptr_t)(slabs + slab_bytes);

  typedef const __attribute__((address_space(4))) RunRec* const_run_ptr;
  // (few tokens: a workgroup takes a part of the range's records and leaves fp32 sums to be added)
  const int Mall = __builtin_amdgcn_readfirstlane(nruns[r]);
  const int jfirst = (int)((int64_t)Mall * item.part / parts);
  const int M = (int)((int64_t)Mall * (item.part + 1) / parts) - jfirst;
  const const_run_ptr rl = (const_run_ptr)(uintptr_t)(runs + (size_t)r * cap + jfirst);
  struct Run { int b, lo, hi, piece; };
  auto run_at = [&](int j) {  // wave-uniform scalar load; past the end: the last run again
    const int jj = j < M ? j : M - 1;
    return Run{rl[jj].b, rl[jj].lo, rl[jj].hi, rl[jj].piece};
  };

  // (every token activates k >= 1 blocks, so a range always has records; M = 0 means a caller's table that lists nothing for
  // these tokens: zeros)
  if (M == 0 && split) {
    for (int it = tid; it < rows * (SC_C / 4); it += THREADS)
      *reinterpret_cast<uint4*>(split + ((size_t)item.part * T + t0 + it / (SC_C / 4)) * d + c0 + (it % (SC_C / 4)) * 4) =
          make_uint4(0u, 0u, 0u, 0u);
    return;
  }
  if (M == 0) {
    for (int it = tid; it < rows * (SC_C / 8); it += THREADS) {
      const size_t o = (size_t)(t0 + it / (SC_C / 8)) * d + c0 + (it % (SC_C / 8)) * 8;
      *reinterpret_cast<uint4*>(out + o) = Z ? *reinterpret_cast<const uint4*>(Z + o) : make_uint4(0u, 0u, 0u, 0u);
    }
    return;
  }

  // Weight slice: lane (g, i) takes columns 4 i .. 4 i + 3 of units 32 s + 8 g + e.
  u32x2 wraw[KT][8];
  const int w_off = (8 * g * d + 4 * i) * 2;
  auto w_rsrc = [&](int b) {
    return __builtin_amdgcn_make_buffer_rsrc((void*)(W + (size_t)b * Bs * d + c0), 0,
                                             (int)(((unsigned)(Bs - 1) * d + SC_C) * 2), SC_RSRC);
  };
  auto load_w = [&](int s, int e, __amdgpu_buffer_rsrc_t rs) {
    wraw[s][e] = __builtin_amdgcn_raw_buffer_load_b64(rs, w_off, (32 * s + e) * d * 2, 0);
  };
  // MFMA operand of K-step s, columns 4 i + t
  bf16x8 wf[KT][4];
  auto make_w = [&](int s, int t) {
    const uint32_t sel = (t & 1) ? 0x07060302u : 0x05040100u;
    u32x4 f;
#pragma unroll
    for (int e = 0; e < 4; ++e) f[e] = __builtin_amdgcn_perm(wraw[s][2 * e + 1][t >> 1], wraw[s][2 * e][t >> 1], sel);
    wf[s][t] = as_bf16x8(f);
  };

  static_assert(NT % RH == 0, "a run ends where the ring does");
  bf16x8 hb[RH][KT];
  int tokv[RH];
  // Where a record lies: byte offsets of the lane's rows from 32 aligned positions on (the tiles start at a multiple of four:
  // whole cache lines), even and odd tiles, and of its last row, whose repetition stands for rows past the end.
  struct Where { int even, odd, last, tok; __amdgpu_buffer_rsrc_t h, t, w; };
  auto where = [&](const Run& q) {
    Where x;
    const int first = q.lo & ~31, st = (q.lo & ~3) - first, last = q.hi - 1 - first;
    auto off = [&](int p) { return (p >> 5) * (KS * 1024) + (p & 31) * 32; };
    const int part = (g >> 1) * 1024 + (g & 1) * 16;
    x.even = off(st + i) + part;
    x.odd = off(st + 16 + i) + part;
    x.last = off(last) + part;
    x.tok = (st + 4 * g + (i & 3)) * 4;
    x.h = __builtin_amdgcn_make_buffer_rsrc((void*)(reinterpret_cast<const char*>(Hin) + (size_t)(first >> 5) * (KS * 1024)), 0,
                                            0x40000000, SC_RSRC);
    x.t = __builtin_amdgcn_make_buffer_rsrc((void*)(tok + first), 0, (last + 1) * 4, SC_RSRC);   // (past the run: zeros)
    x.w = w_rsrc(q.b);
    return x;
  };
  // What slot ti of a run requests for the wavefront's next run (the prologue in the same order: the compiler's waits
  // count the loads behind the one they are for).
  auto request_h = [&](auto tag, const Where& x, int s) {
    constexpr int ti = decltype(tag)::value;
    const int o = min((ti & 1 ? x.odd : x.even) + (ti >> 1) * (KS * 1024), x.last);
    hb[ti % RH][s] = as_bf16x8(__builtin_bit_cast(
        u32x4, __builtin_amdgcn_raw_buffer_load_b128(x.h, o + (s & 1) * 2048, (s >> 1) * 4096, 0)));
  };
  auto request_t = [&](auto tag, const Where& x) {
    constexpr int ti = decltype(tag)::value;
    tokv[ti % RH] = (int)__builtin_amdgcn_raw_buffer_load_b32(x.t, x.tok + ti * 64, 0, 0);
  };
  // The share of the next slice that slot ti requests.  (Slot 0 turns the present one into operands; early, because the wait
  // for it there is a wait for everything requested before it.)
  auto request_w = [&](auto tag, const Where& x) {
    constexpr int ti = decltype(tag)::value, n = 8 * KT, WS = NT > 4 ? 3 : 1;
    constexpr int lo = ti == 0 ? 0 : ti > WS ? n : (ti - 1) * n / WS, hi = ti > WS ? n : ti * n / WS;
#pragma unroll
    for (int u = lo; u < hi; ++u) load_w(u >> 3, u & 7, x.w);
  };
  auto request_late = [&](auto tag, const Where& x, int s) {
    constexpr int ti = decltype(tag)::value;
    if (ti == NT - 1) {
#pragma unroll
      for (int e = 0; e < 8; ++e) load_w(s, e, x.w);
    }
  };

  // Accumulators: of the tile in hand, and of the one before it until it is in the slab.
  static_assert(NT % 2 == 0, "a record leaves them as it found them");
  f32x4 acc[2][4];
  int xprev = R * SC_STRIDE, need_prev = SC_NONE;     // (before the first: nothing, to the dummy row)
#pragma unroll
  for (int t = 0; t < 4; ++t) acc[1][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  f32x4 sl[4];
  const lds_int_ptr prog_in = prog + (lane & (SC_WAVES - 1)) * 64 + lane;     // lane l looks at wavefront l mod 4
  const lds_int_ptr prog_out = prog + wave * 64 + lane;
  auto progress = [&] { return OWN ? 0 : __hip_atomic_load(prog_in, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); };
  auto slab_at = [&](int v, int x) -> f32x4* {
    int a;
    switch (v) {
      case 0: a = __builtin_amdgcn_mov_dpp(x, 0x00, 0xf, 0xf, true); break;
      case 1: a = __builtin_amdgcn_mov_dpp(x, 0x55, 0xf, 0xf, true); break;
      case 2: a = __builtin_amdgcn_mov_dpp(x, 0xaa, 0xf, 0xf, true); break;
      default: a = __builtin_amdgcn_mov_dpp(x, 0xff, 0xf, 0xf, true); break;
    }
    return reinterpret_cast<f32x4*>(slab_lds + (a + 16 * i));
  };
  auto behind = [&](int f) { return __builtin_amdgcn_ballot_w64(f < need_prev) != 0; };
  auto may_go = [&](int& f) {
    if (!OWN && behind(f))
      do f = progress(); while (behind(f));
    wave_lds_fence();
  };
  auto rmw_read = [&](int v) { sl[v] = *slab_at(v, xprev); };
  auto rmw_write = [&](int v, const f32x4 (&a)[4]) {
#pragma unroll
    for (int t = 0; t < 4; ++t) sl[v][t] += a[t][v];
    *slab_at(v, xprev) = sl[v];
  };
  auto publish = [&](int done) {
    wave_lds_fence();
    if (!OWN) __hip_atomic_store(prog_out, done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  };

  Run q = run_at(wave), qn = run_at(wave + SC_WAVES);
  const int iters = M > wave ? (M - wave + SC_WAVES - 1) / SC_WAVES : 0;
  if (iters > 0) {
    const Where x = where(q);
    auto first = [&](auto tag) {     // in the loop's order: tile ti's slot requests tile ti + RH
      constexpr int tr = decltype(tag)::value, ti = tr + NT - RH;
      if (!LATE && RH < NT && tr == 0) {
#pragma unroll
        for (int u = 0; u < 8 * KT; ++u) load_w(u >> 3, u & 7, x.w);
      }
#pragma unroll
      for (int s = 0; s < KT; ++s) {
        request_h(tag, x, s);
        if (LATE) request_late(std::integral_constant<int, ti>{}, x, s);
        else if (s == 0 && RH == NT) request_w(std::integral_constant<int, ti>{}, x);
        __builtin_amdgcn_sched_barrier(0);
      }
      request_t(tag, x);
      __builtin_amdgcn_sched_barrier(0);
    };
    for_each_index(first, std::make_integer_sequence<int, RH>{});
  }
  for (int o = tid * 16; o < (OWN ? SC_WAVES * slab_bytes : slab_bytes + SC_WAVES * 256); o += THREADS * 16)
    *reinterpret_cast<uint4*>(slabs + o) = make_uint4(0u, 0u, 0u, 0u);
  sc_barrier();

  int code = wave * SC_CODE;
  Where xc = where(q);
  // The lane looks at the record `ahead` places before this wavefront's.  A tile may be added once the records before it are past
  // its last token; the pieces before it of its own run have other tokens, so of those only the start is waited
  // for, which says that what their wavefronts did before is done.
  const int ahead = (wave - lane) & (SC_WAVES - 1);
  int need_base = ahead == 0 ? SC_NONE : code - ahead * SC_CODE;
  int f = 0;                 // how far that was when last looked at
  for (int it = 0; it < iters; ++it, code += SC_WAVES * SC_CODE, need_base += SC_WAVES * SC_CODE) {
    const int st = q.lo & ~3;
    const int ntile = (q.hi - st + 15) >> 4;    // 1 .. NT
    const int len = q.hi - q.lo;
    const int rel = st - q.lo + 4 * g + (i & 3);
    const int last_row = (q.hi - 1 - st) & 15, last_lane = (last_row >> 2) * 16 + (last_row & 3);
    const bool other_run = ahead > q.piece;
    const Run qnn = run_at(wave + SC_WAVES * (it + 2));
    const Where x = where(qn);
    auto slot = [&](auto tag) {
      constexpr int ti = decltype(tag)::value, par = ti & 1, before = par ^ 1;
      constexpr bool may_skip = ti >= ALL;
      auto mfma1 = [&](int s, int t) {
        acc[par][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hb[ti % RH][s], wf[s][t],
                                                              s == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : acc[par][t], 0, 0, 0);
      };
      constexpr std::integral_constant<int, (ti + RH) % NT> ask{};
      const Where& xa = ti + RH < NT ? xc : x;
      constexpr int G = 4 * KT;
      // Where the slab's rows are read and written behind the products, and where the others' progress is looked at again.  What lies between
      // reading and publishing is time that the records behind this one wait: reading earlier makes this one wait for its own turn
      // (READ 1, 2, 4: 507, 495, 484 us 7B-like), writing in the last four gaps and publishing behind them 3001 tokens 231, from the middle on 223.
      constexpr int READ = G / 4, WRITE = G > 8 ? G / 2 : G - 4, LOOK = G - 4;
      int tk = 0, xcur = 0, last_token = 0, first_token = 0;
      // Everything but the products, dealt to the gaps behind them (n: 0 .. G - 1): a vector instruction or two in the shadow of
      // every product cost nothing, bunched they cost 4 clk each.
      auto gap = [&](int n) {
        // (the table's tokens are the caller's: one outside the range, where a bucket's are not ascending, is the dummy's too.  What
        // a wait needs is then at most R + 1 into a record, which its wavefront reaches whatever the table says.)
        if (n == 0) tk = (int)min((unsigned)(tokv[ti % RH] - t0), (unsigned)R);
        if (n == (G > 4 ? 1 : 0)) {    // the lane's row of this tile: its token's slab row, or the dummy
          tk = (ti == 0 ? (unsigned)rel < (unsigned)len : rel < len - 16 * ti) ? tk : R;
          xcur = tk * SC_STRIDE;
          asm volatile("" : "+v"(xcur));
        }
        if (n == READ) { rmw_read(0); rmw_read(1); }
        if (n == READ + (G > 4 ? 1 : 0)) { rmw_read(2); rmw_read(3); }
        if (n == READ + 2) last_token = __builtin_amdgcn_readlane(tk, ti + 1 < ntile ? 63 : last_lane);
        if (n == READ + 2) first_token = __builtin_amdgcn_readlane(tk, ti == 0 ? q.lo & 3 : 0);
        if (!may_skip) {
          if (n >= 4 && n % 4 == 0) request_h(ask, xa, n / 4 - 1);
          if (LATE && n % 4 == 1 && n > 4) request_late(tag, x, n / 4 - 1);
          if (!LATE && n == (G > 4 ? 6 : 2)) request_w(tag, x);
        }
        if (n == LOOK) f = progress();
        if (G > 4 && n >= WRITE && n < WRITE + 4) rmw_write(n - WRITE, acc[before]);
        if (G > 8 && n == WRITE + 3) publish(code + (may_skip || ti < ntile ? first_token : SC_CODE));
        if (G == 4 && n == 3) {
#pragma unroll
          for (int v = 0; v < 4; ++v) rmw_write(v, acc[before]);
        }
        __builtin_amdgcn_sched_barrier(0);
      };
      auto products = [&] {
#pragma unroll
        for (int n = 0; n < G; ++n) {
          if (ti == 0) make_w(n / 4, n % 4);
          if (n == READ) may_go(f);
          mfma1(n / 4, n % 4);
          gap(n);
        }
        if (G <= 8) publish(code + (may_skip || ti < ntile ? first_token : SC_CODE));
        xprev = xcur;
        need_prev = may_skip || ti < ntile ? need_base + (other_run ? last_token + 1 : 0) : SC_NONE;
      };
      if (!may_skip) {
        products();
        request_h(ask, xa, KT - 1);
        if (LATE) request_late(tag, x, KT - 1);
      } else {
        if (ti < ntile) {
          products();
        } else if (par == 1 && ti == ntile) {     // (the last tile waits where the next record's first slot adds it from)
#pragma unroll
          for (int t = 0; t < 4; ++t) acc[1][t] = acc[0][t];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < KT; ++s) request_h(ask, xa, s);
      }
      request_t(ask, xa);
      __builtin_amdgcn_sched_barrier(0);
    };
    for_each_index(slot, std::make_integer_sequence<int, NT>{});
    q = qn; qn = qnn;
    xc = x;
  }
  if (iters > 0) {
    may_go(f);
#pragma unroll
    for (int v = 0; v < 4; ++v) rmw_read(v);
#pragma unroll
    for (int v = 0; v < 4; ++v) rmw_write(v, acc[1]);
    publish(code);
  }
  sc_barrier();

  auto sum_at = [&](int o) {
    f32x4 a = *reinterpret_cast<const f32x4*>(slabs + o);
    if (OWN) {
#pragma unroll
      for (int w = 1; w < SC_WAVES; ++w) a += *reinterpret_cast<const f32x4*>(slabs + w * slab_bytes + o);
    }
    return a;
  };
  // Write the slab out, one rounding to bf16: eight columns of a row at a time (fp32 sums of a part: four).
  if (split) {
    for (int it = tid; it < rows * (SC_C / 4); it += THREADS)
      *reinterpret_cast<f32x4*>(split + ((size_t)item.part * T + t0 + it / (SC_C / 4)) * d + c0 + (it % (SC_C / 4)) * 4) =
          sum_at((it / (SC_C / 4)) * SC_STRIDE + (it % (SC_C / 4)) * 16);
    return;
  }
  constexpr int CG = SC_C / 8;  // 16-byte output pieces per row
  for (int it = tid; it < rows * CG; it += THREADS) {
    const int at = (it / CG) * SC_STRIDE + (it % CG) * 32;
    f32x4 lo4 = sum_at(at), hi4 = sum_at(at + 16);
    const size_t o = (size_t)(t0 + it / CG) * d + c0 + (it % CG) * 8;
    if (Z) {                    // the low-rank row of the token
      const uint4 z = *reinterpret_cast<const uint4*>(Z + o);
      lo4 += f32x4{lo_bf16(z.x), hi_bf16(z.x), lo_bf16(z.y), hi_bf16(z.y)};
      hi4 += f32x4{lo_bf16(z.z), hi_bf16(z.z), lo_bf16(z.w), hi_bf16(z.w)};
    }
    *reinterpret_cast<uint4*>(out + o) =
        make_uint4(pack_bf16x2(lo4[0], lo4[1]), pack_bf16x2(lo4[2], lo4[3]), pack_bf16x2(hi4[0], hi4[1]),
                   pack_bf16x2(hi4[2], hi4[3]));
  }
}

// WG: workgroups a CU is to hold.
template <int KS, int NT, int RH, bool LATE, int WG, bool OWN>
__global__ __launch_bounds__(SC_THREADS, WG) void ffn_scatter_kernel(
    const uint16_t* __restrict__ Hin, const uint16_t* __restrict__ W, const RunRec* __restrict__ runs,
    const int32_t* __restrict__ nruns, const int32_t* __restrict__ tok, int N, int d, int T, int R,
    int nr, int nslab, int parts, int inner, int cap, uint16_t* __restrict__ out, const uint16_t* __restrict__ Z,
    float* __restrict__ split) {
  scatter_tile<KS, NT, RH, LATE, OWN>(blockIdx.x, Hin, W, runs, nruns, tok, N, d, T, R, nr, nslab, parts, inner, cap, out, Z, split);
}

// dX and both weight gradients of a backward pass, which need nothing of one another, in one launch: the first `mine` workgroups are
// those of the contraction (two tiles a record), the others those of the weight gradients' kernel.  For the layers whose launches leave CUs empty or are not much
// longer than their own latency.
template <int KS, int UT>
__global__ __launch_bounds__(SC_THREADS, 2) void ffn_scatter_dw_kernel(
    const uint16_t* __restrict__ Hin, const uint16_t* __restrict__ W, const RunRec* __restrict__ runs,
    const int32_t* __restrict__ nruns, const int32_t* __restrict__ tok, int N, int d, int T, int R,
    int nr, int nslab, int inner, int cap, uint16_t* __restrict__ out, int mine, DwOperands ops0, DwOperands ops1, int each,
    const uint16_t* __restrict__ zero_row, int npieces, const DwPiece* __restrict__ pieces) {
  static_assert(SC_THREADS == 256, "both kernels' workgroups");
  const int wg = blockIdx.x;
  if (wg < mine) {
    scatter_tile<KS, 2, 2, false, true>(wg, Hin, W, runs, nruns, tok, N, d, T, R, nr, nslab, 1, inner, cap, out, nullptr, nullptr);
    return;
  }
  const int rest = wg - mine;
  dw_tile<UT>(rest < each ? ops0 : ops1, rest < each ? rest : rest - each, 0, tok, zero_row, npieces, KS * 16, d, pieces, N);
}

// out = the parts' sums added in order (+ the low-rank row), rounded once.
__global__ __launch_bounds__(256) void scatter_sum_kernel(const float* __restrict__ split, int splits, int64_t total,
                                                          uint16_t* __restrict__ out, const uint16_t* __restrict__ Z) {
  const int64_t at = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
  if (at >= total) return;
  f32x4 s = *reinterpret_cast<const f32x4*>(split + at);
#pragma unroll 4
  for (int z = 1; z < splits; ++z) s += *reinterpret_cast<const f32x4*>(split + (size_t)z * total + at);
  if (Z) {
    const uint2 z = *reinterpret_cast<const uint2*>(Z + at);
    s += f32x4{lo_bf16(z.x), hi_bf16(z.x), lo_bf16(z.y), hi_bf16(z.y)};
  }
  *reinterpret_cast<uint2*>(out + at) = make_uint2(pack_bf16x2(s[0], s[1]), pack_bf16x2(s[2], s[3]));
}

// ------------------------------------------------------------------------------------------
// host side
// The kernel's forms: tiles per record, a slab per wavefront, workgroups of a CU that the registers allow and us per four records of
// a workgroup that has its CU to itself, both by K-steps (Bs / 32).  A record of up to 6 tiles takes them whatever it holds, so few rows per block
// and range want few tiles; a record's start (the slice of weights) is the larger part of a short one.  Records of 8 and 10 tiles stop behind their
// last one; `rec` is of full ones (below).
struct ScatterForm { int nt; bool own; int wg[4]; double rec[4]; };
static const ScatterForm kScatterForms[] = {
    {2, true, {4, 3, 2, 2}, {.68, .80, 1.16, 1.52}},
    {4, false, {4, 2, 2, 2}, {1.40, 1.60, 1.96, 2.08}},
    {6, false, {3, 2, 2, 2}, {1.80, 1.88, 2.20, 2.52}},
    {8, false, {3, 2, 1, 1}, {2.24, 2.36, 2.76, 3.16}},
    {10, false, {3, 2, 1, 1}, {2.72, 2.80, 3.28, 3.76}},
};

// us that a launch takes with `nr` ranges of R tokens and the block list in `sp` parts, the same for even and for skewed routing.
// Fitted to the time of 858 shapes (1 to 65536 tokens, 1 to 1024 blocks, 64 to 4096 columns, all block sizes) under even and under
// skewed routing, 40 thousand plans timed, when records of 8 and 10 tiles still went through all their slots: the plan of least cost took 0.5 % more
// than the quickest timed one on average, 3.8 % at the 95th percentile, 13 % at most.  With the present kernel it is 1.0, 7 and 12 % over 248 of those
// shapes and 1.3, 7 and 38 % over 700 others (5668 plans; at most: 5.6 against 7.8 us, one block).  Constants fitted anew to half of these 948 shapes do little
// better on the other half: 1.2 % as it is, 1.0 with a price of 8- and 10-tile records that falls with the tiles they hold, 0.9 with all constants free,
// a launch above 40 us 2.0, 1.7 and 1.7 %: left as they are.
// (What does not depend on the plan is in ScatterWork.  `best`: the least so far; a plan whose workgroups or bytes alone take longer, by what
// they take at least, is not looked at further, and the records' error functions, two thirds of the search, are left out.)
struct ScatterWork {
  double share, rows, weights, once, sums;
  int ks, nslab;
  explicit ScatterWork(const spt_shape_t& s)
      : share((double)s.k / s.N), rows((double)s.T * s.k * s.Bs * 2), weights((double)s.N * s.Bs * s.d * 2),
        sums((double)s.T * s.d * 8.0 / 9.5e6), ks(s.Bs / 32 - 1), nslab(s.d / SC_C) {
    // from memory: rows and weights once, at 6.6 TB/s (fitted)
    const double total = s.T * share;
    once = (rows + weights * (total < 30.0 ? 1.0 - exp(-total) : 1.0) + (double)s.T * s.d * 2) / 6.6e6;
  }
};
static double scatter_cost(const spt_shape_t& s, const ScatterWork& w, const ScatterForm& f, int R, int nr, int sp, double best) {
  const int run = 16 * f.nt;
  // Workgroups per CU, as many at once as registers and LDS allow; each one more makes the others slower by `beside`.
  static const double kBeside[4] = {.27, .32, .37, .42};
  const double beside = kBeside[w.ks];
  const int lds = 160 * 1024 / (f.own ? SC_WAVES * (R + 1) * SC_STRIDE : (R + 1) * SC_STRIDE + SC_WAVES * 256);
  const int at_once = lds < f.wg[w.ks] ? lds : f.wg[w.ks];
  const int each = (int)(((int64_t)nr * w.nslab * sp + 255) / 256), full = each / at_once, rest = each % at_once;
  const double times = full * (1.0 + (at_once - 1) * beside) + (rest ? 1.0 + (rest - 1) * beside : 0.0);
  const double rec = f.rec[w.ks] / (4.0 * sp) * s.N, fixed = R * (f.own ? 0.0187 : 0.0098) + 0.6 * f.rec[w.ks];
  const double added = sp > 1 ? 2.0 + 0.2 * sp + sp * w.sums : 0.0;             // the parts' sums, added by another launch
  const double mean = R * w.share, some_least = mean / (1.0 + mean), full_least = 0.9 * mean / run;
  const double rec_least = rec * (some_least > full_least ? some_least : full_least);
  // (more ranges are more records and more bytes: -1)
  const double shared = (1.0 + (f.wg[w.ks] - 1) * beside) / f.wg[w.ks];
  if ((double)nr * w.nslab * (sp / 256.0) * shared * rec * some_least + added >= best) return -1.0;
  if (times * (fixed + rec_least) + added >= best || w.once + added >= best) return best;
  // Bytes into the CUs: rows once per column slab and weights once per range, at 17.8 TB/s (fitted).
  const double some = mean < 30.0 ? 1.0 - exp(-mean) : 1.0;
  const double in = (w.rows * w.nslab + w.weights * nr * some) / 17.8e6;
  if (in + added >= best) return -1.0;
  // Records of a block in a range: its rows are about Binomial(R, k / N); 1 + P(rows > run) + P(rows > 2 run) + .. if it has any.
  const double sd = sqrt(mean * (1.0 - w.share) + 1e-9), by = 1.0 / (sd * 1.41421356);
  double records = some;
  for (int c = 1; c * run < mean + 4.0 * sd + 2.0; ++c) records += 0.46 * erfc((c * run - 1.5 - mean) * by);
  const double work = times * (fixed + rec * records), bytes = in > w.once ? in : w.once;
  const double more = work > bytes ? work : bytes, less = work > bytes ? bytes : work;
  return more + 0.26 * less * less * less / (more * more) + added;
}

static ScatterPlan plan_scatter_once(const spt_shape_t& s) {
  ScatterPlan p = {};
  const ScatterWork w(s);
  p.nslab = w.nslab;
  // Per form and number of parts (16 blocks or more in each) the range counts that give every CU one workgroup, two, ...; more than
  // five are too short for parts.  Both sides, us a launch, again and again on the same rows: 7B-like, 16 ranges in 10 tiles 457, 28 in 6 tiles 484, 20 in 8 tiles
  // 497; 3001 tokens of it, 8 in 8 tiles 198, 12 in 6 tiles 203, 8 in 10 tiles 209; BERT-large-like, 64 ranges in 6 tiles 98, 32 in 10 tiles 101, 64 in 8 tiles
  // 103; 10956 tokens, d 512, 92 blocks of 96, 19 each: 32 ranges in 6 tiles 59, in 8 tiles 67, in 10 tiles 70; 32768, 1024, 128 of 32, 16: 112 ranges in 4 tiles
  // 234, 64 in 6 tiles 250, 52 in 8 tiles 297.
  double best = 1e300;
  int fits = 0;
  for (const ScatterForm& f : kScatterForms) {
    const int rmax = f.own ? 160 * 1024 / SC_WAVES / SC_STRIDE - 1 : (160 * 1024 - SC_WAVES * 256) / SC_STRIDE - 1;   // (one slab row is the dummy)
    if (s.T <= fits) break;      // (no run is longer than the records of the form before)
    fits = 16 * f.nt - 4;        // (a run may start in the last place of four)
    const int nr_min = (s.T + rmax - 1) / rmax, nr_max = (s.T + 31) / 32 > nr_min ? (s.T + 31) / 32 : nr_min;
    for (int sp = 1; sp == 1 || (sp <= 8 && sp * 16 <= s.N); sp += sp < 4 ? 1 : 2) {
      int last = 0;
      for (int each = 0; each <= (sp == 1 ? 24 : 5) && last < nr_max; ++each) {
        const int count = each == 0 ? nr_min : each * 256 / (p.nslab * sp);
        if (sp > 1 && (int64_t)count * p.nslab * sp > 5 * 256) break;   // (also the fewest there can be: 84857 tokens, 3.3 GB of sums)
        if (count <= last || count < nr_min) continue;
        last = count > nr_max ? nr_max : count;
        const int R = (s.T + last - 1) / last, nr = (s.T + R - 1) / R;
        const double cost = scatter_cost(s, w, f, R, nr, sp, best);
        if (cost < 0.0) break;
        if (cost < best) {
          best = cost; p.R = R; p.nr = nr; p.splits = sp; p.nt = f.nt;
          p.smem = f.own ? SC_WAVES * (R + 1) * SC_STRIDE : (R + 1) * SC_STRIDE + SC_WAVES * 256;
        }
      }
    }
  }
  p.run_rows = 16 * p.nt;
  // Slabs side by side on an XCD: of a ranges x b slabs that run together (a b = 32 workgroups per place on a CU) it fetches a
  // runs of `mean` rows and b slices of 64 columns per block, least at b^2 = a b mean / 64; all ranges where there are few.
  // (47 slabs, 32 ranges of one slab side by side instead of four by eight: 346 us, 312.  Two places also for the other forms that have them:
  // within 0.3 % over 270 layers.)
  const int together = 32 * (p.nt == 6 ? 2 : 1);
  p.inner = (int)(sqrt(together * ((double)p.R * s.k / s.N) / 64.0) + 0.5);
  if (p.inner < (together + p.nr - 1) / p.nr) p.inner = (together + p.nr - 1) / p.nr;
  if (p.inner < 1) p.inner = 1;
  if (p.inner > p.nslab) p.inner = p.nslab;
  p.split_bytes = p.splits > 1 ? align256((size_t)p.splits * s.T * s.d * 4) : 0;
  p.cap = s.N + (int)(((int64_t)p.R * s.k + 3 * s.N + p.run_rows - 1) / p.run_rows);
  p.runs_bytes = align256((size_t)p.nr * p.cap * sizeof(RunRec));
  p.counts_bytes = align256((size_t)p.nr * 4);
  p.table_bytes = p.runs_bytes + p.counts_bytes + align256((size_t)(p.nr + 1) * s.N * 4);
  return p;
}

// (The search takes 0.4 microseconds for 24 tokens, 2.5 for 3001 or 8192 of the 7B-like layer, and every call of the path asks several
// times: each thread keeps the plans of the last few shapes, which are functions of the shape alone.)
ScatterPlan plan_scatter(const spt_shape_t& s) {
  struct Kept { int32_t T, d, N, Bs, k; ScatterPlan plan; };
  static thread_local Kept kept[8] = {};
  static thread_local int next = 0;
  for (const Kept& e : kept)
    if (e.T == s.T && e.d == s.d && e.N == s.N && e.Bs == s.Bs && e.k == s.k) return e.plan;
  Kept& e = kept[next++ & 7];
  e = Kept{s.T, s.d, s.N, s.Bs, s.k, plan_scatter_once(s)};
  return e.plan;
}

int32_t* scatter_starts(const ScatterPlan& p, int32_t* table) {
  return reinterpret_cast<int32_t*>(reinterpret_cast<char*>(table) + p.runs_bytes + p.counts_bytes);
}

RunRec* scatter_runs(const ScatterPlan&, int32_t* table) { return reinterpret_cast<RunRec*>(table); }
int32_t* scatter_counts(const ScatterPlan& p, int32_t* table) {
  return reinterpret_cast<int32_t*>(reinterpret_cast<char*>(table) + p.runs_bytes);
}

hipError_t run_scatter_ranges(const spt_shape_t& s, const ScatterPlan& p, int32_t* table, hipStream_t st) {
  scatter_runs_kernel<<<p.nr, 64, 0, st>>>(scatter_starts(p, table), s.N, p.cap, p.run_rows, scatter_runs(p, table),
                                           scatter_counts(p, table));
  return hipGetLastError();
}

template <int KS, int NT, int RH, bool LATE, int WG, bool OWN>
static hipError_t launch_scatter_t(const spt_shape_t& s, const ScatterPlan& p, const uint16_t* Hin,
                                   const uint16_t* W, const int32_t* table, const int32_t* tok,
                                   uint16_t* out, const uint16_t* Z, float* split, hipStream_t st) {
  static bool attr_set = false;
  if (!attr_set) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(ffn_scatter_kernel<KS, NT, RH, LATE, WG, OWN>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  const RunRec* runs = reinterpret_cast<const RunRec*>(table);
  const int32_t* nruns = reinterpret_cast<const int32_t*>(reinterpret_cast<const char*>(table) + p.runs_bytes);
  const bool parts = p.splits > 1;
  ffn_scatter_kernel<KS, NT, RH, LATE, WG, OWN><<<scatter_grid(p), SC_THREADS, p.smem, st>>>(
      Hin, W, runs, nruns, tok, s.N, s.d, s.T, p.R, p.nr, p.nslab, p.splits, p.inner, p.cap, out, Z, parts ? split : nullptr);
  if (!parts) return hipGetLastError();
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int64_t total = (int64_t)s.T * s.d;
  scatter_sum_kernel<<<(unsigned)((total / 4 + 255) / 256), 256, 0, st>>>(split, p.splits, total, out, Z);
  return hipGetLastError();
}

hipError_t launch_scatter(const spt_shape_t& s, const ScatterPlan& p, const uint16_t* Hin, const uint16_t* W,
                          const int32_t* table, const int32_t* tok, uint16_t* out, const uint16_t* Z,
                          float* split, hipStream_t st) {
  // (four and six tiles, two workgroups per CU, leave a lane 256 registers: rows requested fewer tiles ahead, and with eight K-steps
  // of 16 the weight slice later)
#define SPT_SC_ARGS s, p, Hin, W, table, tok, out, Z, split, st
#define SPT_SC(KS)                                                                                                      \
  (p.nt == 2   ? launch_scatter_t<KS, 2, 2, false, 1, true>(SPT_SC_ARGS)                                                \
   : p.nt == 4 ? launch_scatter_t<KS, 4, (KS > 6 ? 2 : 4), (KS > 6), 2, false>(SPT_SC_ARGS)                             \
   : p.nt == 6 ? launch_scatter_t<KS, 6, (KS > 4 ? 3 : 6), (KS > 6), 2, false>(SPT_SC_ARGS)                             \
   : p.nt == 8 ? launch_scatter_t<KS, 8, 8, false, 1, false>(SPT_SC_ARGS)                                               \
               : launch_scatter_t<KS, 10, 10, false, 1, false>(SPT_SC_ARGS))
  switch (s.Bs / 16) {
    case 2: return SPT_SC(2);
    case 4: return SPT_SC(4);
    case 6: return SPT_SC(6);
    case 8: return SPT_SC(8);
    default: return hipErrorInvalidValue;
  }
#undef SPT_SC_ARGS
#undef SPT_SC
}

// Where two workgroups share a CU, so that the launch holds as much at once as the two it replaces.  us a pass, two launches and one, unless said otherwise 4 to 8
// less over 60 layers: 512 tokens, d 256, 16 blocks of 64, 4 each (34 KB of slabs) 42 / 37; 2287, 512, 28 of 96, 12 (74 KB) 106 / 98; with one
// workgroup per CU 573, 2752, 151 of 32, 17 (119 KB) 186 / 193; 829, 2304, 35 of 32, 6 (123 KB) 86.0 / 87.3; 1304, 1024, 40 of 32, 4 (85 KB) 73 / 73.
// The gradients' 62 or 72 KB of LDS leave room for two of the contraction's workgroups where short ranges and narrow blocks would put three or four on a CU.  With
// more than two for each, up to 20000 rows: 4670 tokens, d 512, 3 of 32, 1 69 / 66; 5202 rows of 1734, 1024, 6 of 32, 3 69 / 67; but 4589,
// 448, 19 of 32, 10 103 / 108; 9775, 192, 14 of 32, 8 138 / 144; 4369, 576, 16 of 32, 9 102 / 106; and in six rounds and more the contraction is nearly all there
// is: 10472, 512, 99 of 32, 1 141 / 145; 13494, 960, 197 of 32, 2 461 / 490.
bool scatter_takes_dw(const spt_shape_t& s, const ScatterPlan& p) {
  if (p.nt != 2 || p.splits != 1 || p.smem > 80 * 1024) return false;
  const int grid = p.nr * p.nslab, regs = kScatterForms[0].wg[s.Bs / 32 - 1], lds = 160 * 1024 / p.smem;
  return grid <= 2 * 256 || (regs < lds ? regs : lds) <= 2 || (grid <= 6 * 256 && (int64_t)s.T * s.k <= 20000);
}

template <int KS>
static hipError_t launch_scatter_dw_t(const spt_shape_t& s, const ScatterPlan& p, const uint16_t* Hin, const uint16_t* W,
                                      const Schedule& sc, uint16_t* out, const DwOperands* ops, hipStream_t st) {
  constexpr int UT = KS > 4 ? 128 : 64;
  static bool attr_set = false;
  if (!attr_set) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(ffn_scatter_dw_kernel<KS, UT>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  const RunRec* runs = reinterpret_cast<const RunRec*>(sc.rstart);
  const int32_t* nruns = reinterpret_cast<const int32_t*>(reinterpret_cast<const char*>(sc.rstart) + p.runs_bytes);
  const int mine = scatter_grid(p), each = dw_grid(sc.dw_cap, s.d), lds = p.smem > dw_smem_bytes<UT>() ? p.smem : dw_smem_bytes<UT>();
  ffn_scatter_dw_kernel<KS, UT><<<mine + 2 * each, SC_THREADS, lds, st>>>(
      Hin, W, runs, nruns, sc.tok, s.N, s.d, s.T, p.R, p.nr, p.nslab, p.inner, p.cap, out, mine, ops[0], ops[1], each, sc.zero_row,
      sc.dw_cap, sc.dw_pieces);
  return hipGetLastError();
}

hipError_t launch_scatter_dw(const spt_shape_t& s, const ScatterPlan& p, const uint16_t* Hin, const uint16_t* W, const Schedule& sc,
                             uint16_t* out, const DwOperands* ops, hipStream_t st) {
  switch (s.Bs / 16) {
    case 2: return launch_scatter_dw_t<2>(s, p, Hin, W, sc, out, ops, st);
    case 4: return launch_scatter_dw_t<4>(s, p, Hin, W, sc, out, ops, st);
    case 6: return launch_scatter_dw_t<6>(s, p, Hin, W, sc, out, ops, st);
    case 8: return launch_scatter_dw_t<8>(s, p, Hin, W, sc, out, ops, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace spt

// For tests, not declared in the header: the plan of a shape (tiles of 16 rows per record, tokens per range, ranges, parts, column
// slabs, grid) and what the grid's first `count` workgroups do (part, range, slab each).  0 if the shape has no such launch.
extern "C" int spt_internal_scatter_layout(const spt_shape_t* s, int32_t* plan, int32_t* items, int count) {
  using namespace spt;
  if (!s || !plan || s->T < 1 || s->N < 1 || s->k < 1 || s->k > s->N || s->d < SC_C || s->d % SC_C || s->Bs % 32 || s->Bs < 32 || s->Bs > 128) return 0;
  const ScatterPlan p = plan_scatter(*s);
  const int out[6] = {p.nt, p.R, p.nr, p.splits, p.nslab, scatter_grid(p)};
  for (int e = 0; e < 6; ++e) plan[e] = out[e];
  for (int wg = 0; wg < count && wg < out[5]; ++wg) {
    const ScatterItem x = scatter_item(wg, p.nslab, p.nr, p.splits, p.inner);
    items[3 * wg] = x.part; items[3 * wg + 1] = x.r; items[3 * wg + 2] = x.slab;
  }
  return 1;
}
