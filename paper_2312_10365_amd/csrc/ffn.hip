// Grouped bf16 MFMA GEMMs of the routed FFN.
//
// Algorithm 4 of the paper runs, per weight block, a gather, two dense GEMMs and a scatter.
// Here every stage is ONE launch over all blocks: a row tile knows its bucket from a small
// prefix table built on the device, the gather is fused into the operand loads, and block
// outputs are added per token in a fixed order (in LDS for narrow blocks; through per-pair
// partial rows and a combine for wide ones).
//
// This file: the schedule tables, the K = d GEMMs of narrow blocks (up-projection + activation,
// dH * act'), the weight-gradient GEMMs (K = bucket rows), the combine used by the wide-block
// path, and the host-side sequencing of all stages.  The K = Bs contraction of narrow blocks
// (down-projection, dX) with Alg. 4's write-back folded in lives in ffn_scatter.hip; blocks
// wider than 128 units in ffn_wide.hip.
#include <stdlib.h>
#include <type_traits>

#include "ffn_common.hpp"
#include "ffn_dw.hpp"
#include "spt_host.hpp"
#include "profile.hpp"

namespace spt {

// ------------------------------------------------------------------------------------------
// Schedule tables, built on the device from `offsets` (plan_kernel: the row lists by one workgroup, thread b = bucket b).
//
// The chip has 8 XCDs with a private L2 each, and workgroups are handed to XCDs round-robin
// by workgroup id, so "which XCD runs which tile, and when" decides what is served from L2
// and what has to come over the fabric.  Two tables:
//   border[N]         buckets by size, largest first (dW GEMMs start the long ones first);
//   kd_list[8][cap], kd_count[8]   per XCD, the row tiles of the K = d GEMMs in the order
//                     the XCD should run them.  With N >= 16 the buckets are dealt to the
//                     XCDs by size rank (boustrophedon, so the loads balance), and an XCD's
//                     list is ordered by tile level first (the i-th tile of every bucket it
//                     owns, which all cover the same window of token ids), bucket second:
//                     tiles that run together then share both the activation rows (each
//                     token sits in k of the N buckets) and, level after level, the same few
//                     weight blocks.  With fewer buckets the bucket-major tile sequence is
//                     cut into 8 contiguous runs of equal length (weight reuse only).
//                     Wide blocks have one list, bucket-major, and its length in kd_count[0]: there
//                     the kernel itself cuts the (row tile, A-side tile) items into 8 equal slices.
//                     Where the mean bucket is small (wide_tails) the buckets' last tiles, if they are of
//                     at most 64 rows, are behind all others, and kd_count[1] is how many are in front of them.

constexpr int FU_ROWS = 256;      // rows of a K = d tile of narrow blocks
// A round of K = d tiles of 256, 128 or 64 rows, one per CU of an XCD, takes as long as a tile that has the memory path for itself,
// or as all of them together by the rows and weight rows they fetch (the kernel is bound by those): kPartAlone, and
// kPartShare per tile; 640 = a full round of 256-row tiles.  us a launch, up / dH, whole tiles on their bucket's XCD -> this:
// the OPT-1.3B-like layer with the skewed router (63 to 83 tiles an XCD) 102 / 114 -> 86 / 95; 7B-like (nine tiles for most
// buckets of 2048 + 39 rows) 305 / 314 -> 287 / 296; BERT-large-like 76 / 84 -> 72 / 80; with rounds counted alone
// (a half tile 0.6 of a whole one) 3000 tokens of the 7B-like layer were cut into halves for nothing (121, 121).
constexpr int kPartAlone[3] = {12 * 32, 7 * 32, 5 * 32}, kPartShare[3] = {20, 13, 10};

struct PlanArgs {
  const int32_t* offsets;
  const int32_t* perm;
  int N, QT, cap, P, k, wide, tails, spread;
  int32_t *border, *kd_count;
  KdTile* kd_list;
  uint32_t* zero_row;
  int32_t* tok;
  int R, nr;               // narrow blocks: token ranges of the K = Bs kernel (R = 0: none)
  int32_t* starts;
  RunRec* runs;
  int32_t* nruns;
  int run_cap, run_rows;
  int dw_rows, dw_cap;
  DwPiece* dw_pieces;
  int32_t* dw_xlist;
};

// Sorted position q: tok[q] = its token and, for narrow blocks (R > 0), its entries of the table
// starts[r][b] = first sorted position of bucket b whose token is >= r R (r = 0 .. nr): position q is
// that first position for every range after its predecessor's and up to its own, and the bucket's
// end for the ranges behind its last row -- every entry is written exactly once, no search, no atomics.
__device__ __forceinline__ void plan_position(const PlanArgs& p, const int32_t* off_sh, int q) {
  const int t = p.perm[q] / p.k;
  p.tok[q] = t;
  if (p.R <= 0) return;
  int lo = 0, hi = p.N;   // bucket of q: the largest b with offsets[b] <= q
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (off_sh[mid] <= q) lo = mid; else hi = mid;
  }
  const int b = lo;
  const int rq = t / p.R;
  const int rprev = (q > off_sh[b]) ? (p.perm[q - 1] / p.k) / p.R : -1;
  for (int r = rprev + 1; r <= rq; ++r) p.starts[(size_t)r * p.N + b] = q;
  if (q + 1 == off_sh[b + 1])
    for (int r = rq + 1; r <= p.nr; ++r) p.starts[(size_t)r * p.N + b] = q + 1;
}

// The same for all positions of a batch of few pairs by one workgroup, Q per thread (products below 2^31: quotients by a multiplication
// are exact), and the run records of the K = Bs kernel, for which the table stays in LDS if it fits.
constexpr int kAllPairs = 4096, kAllTable = 10240;
template <int Q>
__device__ __forceinline__ void plan_positions(const PlanArgs& p, int32_t* off_sh) {
  __shared__ int32_t sm_table[kAllTable];
  auto over = [](uint32_t x, uint32_t y_inv) { return (int)((uint64_t)x * y_inv >> 31); };
  const uint32_t k_inv = (0x80000000u + p.k - 1) / p.k, r_inv = p.R > 0 ? (0x80000000u + p.R - 1) / p.R : 0u;
  const int N = p.N, q0 = threadIdx.x;
  int at[Q], before[Q], lo[Q];
#pragma unroll
  for (int x = 0; x < Q; ++x) {
    const int q = min(q0 + x * 1024, p.P - 1);
    at[x] = p.perm[q];
    before[x] = p.perm[max(q - 1, 0)];
    lo[x] = 0;
  }
  for (int e = q0; e <= N; e += 1024) off_sh[e] = p.offsets[e];
#pragma unroll
  for (int x = 0; x < Q; ++x) {
    at[x] = over(at[x], k_inv);
    before[x] = over(before[x], k_inv);
    if (q0 + x * 1024 < p.P) p.tok[q0 + x * 1024] = at[x];
  }
  if (p.R <= 0) return;
  __syncthreads();
  for (int step = 1 << (31 - __clz(N)); step; step >>= 1)   // bucket of q: the largest b with offsets[b] <= q
#pragma unroll
    for (int x = 0; x < Q; ++x) {
      const int mid = lo[x] + step;
      if (off_sh[min(mid, N)] <= q0 + x * 1024 && mid < N) lo[x] = mid;
    }
  auto runs = [&](int32_t* table) {
    for (int e = q0; e < N; e += 1024)        // an empty bucket has no row to write its table column
      if (off_sh[e] == off_sh[e + 1])
        for (int r = 0; r <= p.nr; ++r) table[r * N + e] = off_sh[e];
#pragma unroll
    for (int x = 0; x < Q; ++x) {
      const int q = q0 + x * 1024, b = lo[x];
      if (q >= p.P) break;
      const int rq = over(at[x], r_inv), rprev = q > off_sh[b] ? over(before[x], r_inv) : -1;
      for (int r = rprev + 1; r <= rq; ++r) table[r * N + b] = q;
      if (q + 1 == off_sh[b + 1])
        for (int r = rq + 1; r <= p.nr; ++r) table[r * N + b] = q + 1;
    }
    __syncthreads();
    for (int r = q0 >> 6; r < p.nr; r += 16) compact_runs(table, N, p.run_cap, p.run_rows, p.runs, p.nruns, r, q0 & 63);
  };
  if ((p.nr + 1) * N <= kAllTable) runs(sm_table);
  else runs(p.starts);
}

// Workgroup 0 builds the row tiles' lists over the buckets, workgroup 1 the pieces of the weight gradients (one after the
// other in one workgroup they were the length of the launch; us: 8192 tokens, 128 blocks, 32 each 10.8 -> 8.8; 16384, 64, 16
// 9.6 -> 7.7; 2048, 32, 8 6.1 -> 5.1), the others take 1024 sorted positions each; kAll: one workgroup takes them all, and the
// run lists of the K = Bs kernel after them (few pairs: a launch of the path then costs more than the work in it).
template <int Q>
__global__ __launch_bounds__(1024) void plan_kernel(PlanArgs p) {
  constexpr bool kAll = Q > 0;
  __shared__ int32_t off_sh[1025];
  const int N = p.N;
  if constexpr (kAll) {
    if (blockIdx.x == 2) {
      plan_positions<Q>(p, off_sh);
      return;
    }
  }
  for (int e = threadIdx.x; e <= N; e += 1024) off_sh[e] = p.offsets[e];
  __syncthreads();
  if (!kAll && blockIdx.x == 0 && p.R > 0)     // an empty bucket has no row to write its table column
    for (int e = threadIdx.x; e < N; e += 1024)
      if (off_sh[e] == off_sh[e + 1])
        for (int r = 0; r <= p.nr; ++r) p.starts[(size_t)r * N + e] = off_sh[e];
  if (!kAll && blockIdx.x > 1) {
    const int q = (blockIdx.x - 2) * 1024 + threadIdx.x;
    if (q < p.P) plan_position(p, off_sh, q);
    return;
  }
  const bool lists = blockIdx.x == 0, cuts = p.dw_pieces && blockIdx.x == 1;
  if (!lists && !cuts) return;
  __shared__ int32_t wtot[16];
  if (lists && threadIdx.x < 64) p.zero_row[threadIdx.x] = 0u;  // 256 bytes of zeros for padded K rows
  __shared__ __align__(16) int32_t sm_m[1024];
  __shared__ int32_t sm_ntq_by_rank[1024];
  const int b = threadIdx.x;
  const int off = (b < N) ? off_sh[b] : 0;
  const int m = (b < N) ? off_sh[b + 1] - off : 0;

  auto inclusive_scan = [&](int v) {
    int total;
    return block_inclusive_sum(v, wtot, total);
  };

  __shared__ int32_t own[8], shorts[8][2];                      // per XCD: its group's tiles, and bucket ends listed apart (parts)
  if (b < 8) { own[b] = 0; shorts[b][0] = 0; shorts[b][1] = 0; }
  sm_m[b] = m;
  __syncthreads();
  // rank by size: as many threads per bucket as there are, at most a wavefront's, each with a share of the others, four at a time
  // (a thread per bucket: 8.2 -> 7.0 us for the whole kernel with 24 tokens and 128 buckets, 14.6 -> 10.6 with 131072 pairs in 64)
  const int tlog = 10 - (32 - __clz(N - 1)), tpb = 1 << tlog, tb = b >> tlog;
  __shared__ int16_t sm_rank[1024];
  int rank = 0;
  if (N < 16) {                 // (not worth the barrier: 4.8 -> 4.5 us with 6 buckets)
    if (b < N)
      for (int o = 0; o < N; ++o) rank += (sm_m[o] > m) || (sm_m[o] == m && o < b);
  } else {
    const int need = (N + 3) >> 2, step = min(min(tpb, 64), need > 1 ? 1 << (32 - __clz(need - 1)) : 1);
    const int share = b & (tpb - 1), tm = sm_m[min(tb, 1023)];
    int r = 0;
    if (share < step)
      for (int o = 4 * share; o < N; o += 4 * step) {            // (sizes past the last bucket are 0, their ids above every bucket's)
        const int4 q = *reinterpret_cast<const int4*>(sm_m + o);
        r += (q.x > tm || (q.x == tm && o < tb)) + (q.y > tm || (q.y == tm && o + 1 < tb)) +
             (q.z > tm || (q.z == tm && o + 2 < tb)) + (q.w > tm || (q.w == tm && o + 3 < tb));
      }
    for (int o = 1; o < step; o <<= 1) r += __shfl_xor(r, o);
    if (share == 0 && tb < N) sm_rank[tb] = (int16_t)r;
    __syncthreads();
    rank = b < N ? sm_rank[b] : 0;
  }
  // Tiles of p.QT rows; with 256 a bucket's last rows, if they are at most 128, are listed apart (1: up to 64, 2: up to 128).
  __shared__ uint8_t sm_short_by_rank[1024];
  const bool parts = p.QT == FU_ROWS && N >= 16 && !p.wide;
  const int end_rows = m & (p.QT - 1), mine_short = !parts || end_rows == 0 || end_rows > 128 ? 0 : end_rows > 64 ? 2 : 1;
  const int ntq = (m >> (31 - __clz(p.QT))) + (end_rows > 0 && !mine_short);   // (64 or 256: a power of two)
  // rank r goes to group r%16 (<8) or 15 - r%16: position pg = r/8 inside the group; the
  // member at position p of group g has rank 8p + (p even ? g : 7 - g); sizes fall with p.
  auto group_of = [&](int r) { return (r >> 3 & 1) ? 7 - (r & 7) : (r & 7); };
  if (b < N) {
    if (p.spread && N >= 16) {
      atomicAdd(&own[group_of(rank)], ntq);
      if (mine_short) atomicAdd(&shorts[group_of(rank)][mine_short - 1], 1);
    }
    if (lists) p.border[rank] = b;
    sm_ntq_by_rank[rank] = ntq;
    sm_short_by_rank[rank] = (uint8_t)mine_short;
  }
  __syncthreads();

  // Weight-gradient work items (backward, narrow blocks): a bucket of m rows becomes
  // ceil(m / p.dw_rows) pieces of equal size (an empty bucket one empty piece: its gradient block
  // is written as zeros), listed largest bucket first.  A bucket's first piece goes straight
  // into its gradient block, the others into staging slots that are added afterwards in order.
  if (cuts) {
    __shared__ int32_t sm_np_rank[1024];
    __shared__ int32_t sm_wstart[1024];
    const int np = (b < N) ? (m > p.dw_rows ? (m + p.dw_rows - 1) / p.dw_rows : 1) : 0;
    if (b < N) sm_np_rank[rank] = np;
    else sm_np_rank[b] = 0;
    // one sum for both: staging slots, in bucket order (there are fewer than N of them: a piece holds 1.5 times the mean bucket),
    // and, above, buckets with staged pieces
    const int both = inclusive_scan(np > 1 ? (np - 1) | 1 << 16 : 0);
    const int x_end = both & 0xFFFF, l_end = both >> 16;
    if (b < N && np > 1) {
      p.dw_xlist[1 + 3 * (l_end - 1)] = b;
      p.dw_xlist[2 + 3 * (l_end - 1)] = x_end - (np - 1);
      p.dw_xlist[3 + 3 * (l_end - 1)] = x_end;
    }
    if (b == N - 1) p.dw_xlist[0] = l_end;
    const int mine = sm_np_rank[b];                            // (the sum's barriers lie between)
    const int w_end = inclusive_scan(mine);                    // work order: by rank
    sm_wstart[b] = w_end - mine;
    __shared__ int32_t total_pieces;
    if (b == 1023) total_pieces = w_end;
    __syncthreads();
    if (b < N) {
      const int at = sm_wstart[rank], base = m / np, rem = m % np;
      for (int pc = 0; pc < np; ++pc) {
        const int lo = off + pc * base + (pc < rem ? pc : rem);
        p.dw_pieces[at + pc] = DwPiece{lo, lo + base + (pc < rem ? 1 : 0), pc == 0 ? b : N + x_end - (np - 1) + pc - 1, 0};
      }
    }
    for (int e = total_pieces + b; e < p.dw_cap; e += 1024) p.dw_pieces[e] = DwPiece{0, 0, -1, 0};
  }
  if (!lists) return;

  if (p.wide) {
    // (p.tails: a bucket's last rows, if they are at most 64, behind everything else.  P is small then: one sum for both)
    const int small = p.tails && end_rows > 0 && end_rows <= 64, big = ntq - small;
    const int both = inclusive_scan(small << 20 | big), inc = p.tails ? both & 0xFFFFF : both, tails = p.tails ? both >> 20 : 0;
    __shared__ int32_t bigs;
    if (b == N - 1) {
      bigs = inc;
      p.kd_count[0] = inc + tails;
      p.kd_count[1] = inc;
    }
    if (p.tails) __syncthreads();
    if (b < N) {
      for (int lvl = 0; lvl < big; ++lvl) p.kd_list[inc - big + lvl] = KdTile{(uint16_t)b, (uint16_t)p.QT, off + lvl * p.QT};
      if (small) p.kd_list[bigs + tails - 1] = KdTile{(uint16_t)b, (uint16_t)p.QT, off + big * p.QT};
    }
    return;
  }
  // Into how many parts (1 << c) the `left` tiles of an unfilled last round go: what takes least, with s2 ends of up to 128 rows and s1 of
  // up to 64 behind them.
  auto cheapest_cut = [](int left, int s1, int s2) {
    int best = 0, least = 0;
    for (int c = 0; (left || s2) && c < 3; ++c) {
      const int big = left << c, mid = c == 2 ? 0 : s2, n = big + (c == 2 ? 2 * s2 : s2) + s1;
      int cost = 0;
      for (int at = 0; at < n; at += 32) {
        const int cls = at < big ? c : at < big + mid ? 1 : 2;
        cost += max(kPartAlone[cls], kPartShare[cls] * min(32, n - at));
      }
      if (c == 0 || cost < least) { least = cost; best = c; }
    }
    return best;
  };
  if (N >= 16) {
    auto member_rank = [&](int grp, int pos) { return 8 * pos + ((pos & 1) ? 7 - grp : grp); };
    // The same number of tiles for every XCD (spread: see run_plan), and for lists that one workgroup per CU walks in rounds (parts) how those
    // of a last, unfilled round are cut.
    __shared__ int32_t surplus0[8], gap0[9], have[8], cut[8];
    int most = 0;                 // tiles of an XCD
    if (!p.spread) {
      if (b < 8) {
        int total = 0;
        for (int pos = 0; 8 * pos < N; ++pos) {
          const int r = member_rank(b, pos);
          total += r < N ? sm_ntq_by_rank[r] : 0;
        }
        p.kd_count[b] = total;
      }
    } else {
#pragma unroll
      for (int x = 0; x < 8; ++x) most += own[x];
      most = (most + 7) / 8;
      if (b < 8) {
        int sur = 0, gap = 0, all = 0;
#pragma unroll
        for (int x = 0; x < 8; ++x) {
          const int o = own[x];
          all += max(o - most, 0);
          if (x < b) { sur += max(o - most, 0); gap += max(most - o, 0); }
        }
        const int mine = own[b];
        surplus0[b] = sur; gap0[b] = gap;
        if (b == 7) gap0[8] = 0x7FFFFFFF;
        const int hv = mine >= most ? most : mine + max(0, min(all - gap, most - mine));
        const int left = parts ? hv % 32 : 0, s1 = shorts[b][0], s2 = shorts[b][1], best = cheapest_cut(left, s1, s2);
        have[b] = hv;
        cut[b] = best;
        p.kd_count[b] = hv - left + (left << best) + (best == 2 ? 2 * s2 : s2) + s1;
      }
      __syncthreads();
    }
    const int members = (N + 7) / 8;
    auto place = [&](int o, int lvl) {                     // the tile of bucket o at a level
      const int orank = sm_rank[o], g = group_of(orank);
      int at = orank >> 3;          // members with a tile at this level are a prefix; before them: all tiles of lower levels
#pragma unroll 4
      for (int pos = 0; pos < members; ++pos) {
        const int r = member_rank(g, pos);
        at += min(r < N ? (int)sm_ntq_by_rank[r] : 0, lvl);
      }
      int x = g;
      const int q = off_sh[o] + lvl * p.QT;
      if (!p.spread) {
        p.kd_list[(size_t)x * p.cap + at] = KdTile{(uint16_t)o, (uint16_t)p.QT, q};
        return;
      }
      if (at >= most) {           // more than its share: the next free place of the XCDs that have less
        const int e = surplus0[g] + at - most;
        for (x = 0; gap0[x + 1] <= e; ++x) {}
        at = own[x] + e - gap0[x];
      }
      KdTile* list = p.kd_list + (size_t)x * p.cap;
      const int full = parts ? have[x] / 32 * 32 : have[x], c = cut[x], rows = p.QT >> c;
      if (at < full) {
        list[at] = KdTile{(uint16_t)o, (uint16_t)p.QT, q};
      } else {
        for (int e = 0; e < 1 << c; ++e)
          list[full + ((at - full) << c) + e] = KdTile{(uint16_t)o, (uint16_t)(q + e * rows < off_sh[o + 1] ? rows : 0), q + e * rows};
      }
    };
    // As many threads per bucket as there are, a level each.  Where that would be many levels for the threads of the largest, a tile each, its bucket
    // searched for: every level is a walk through the members, one after the other.  us a training pass, threads per bucket and 64-row tiles on their bucket's
    // XCD -> this, skewed routing: 8416 tokens, d 640, 526 blocks of 64, 1 each 729 -> 367; 3692, 576, 568 of 64, 2 469 -> 274; 12288, 1024, 256 of 64, 1
    // 490 -> 401; 6981, 448, 107 of 32, 4 184 -> 154; 256-row tiles in their place, listed so, 377, 283, 398, 158.  (One loop for both: written twice, a pass of the
    // BERT-base-like layer took 96.8 where this takes 96.6.)
    const bool by_tile = sm_ntq_by_rank[0] > 4 * tpb;
    __shared__ int32_t tiles_to[1024];                     // tiles up to and with those of bucket b
    int first = b & (tpb - 1), step = tpb, end = tb < N ? (int)sm_ntq_by_rank[sm_rank[tb]] : 0;
    if (by_tile) {
      tiles_to[b] = inclusive_scan(ntq);
      __syncthreads();
      first = b; step = 1024; end = tiles_to[N - 1];
    }
    for (int t = first; t < end; t += step) {
      int o = tb, before = 0;
      if (by_tile) {
        o = 0;                                             // the first bucket with more
        for (int by = 512; by; by >>= 1)
          if (o + by <= N - 1 && tiles_to[o + by - 1] <= t) o += by;
        before = o ? tiles_to[o - 1] : 0;
      }
      place(o, t - before);
    }
    if (b < N && mine_short) {      // a bucket's end, behind the tiles: those of up to 128 rows, then of up to 64
      const int g = group_of(rank), pg = rank >> 3;
      int same = 0;
#pragma unroll 4
      for (int pos = 0; pos < pg; ++pos) same += sm_short_by_rank[member_rank(g, pos)] == mine_short;
      const int left = have[g] % 32, c = cut[g], q = off + ntq * p.QT;
      KdTile* list = p.kd_list + (size_t)g * p.cap + (have[g] - left) + (left << c);
      const int s2_entries = c == 2 ? 2 * shorts[g][1] : shorts[g][1];
      if (mine_short == 1) list[s2_entries + same] = KdTile{(uint16_t)b, 64, q};
      else if (c < 2) list[same] = KdTile{(uint16_t)b, 128, q};
      else
        for (int e = 0; e < 2; ++e) list[2 * same + e] = KdTile{(uint16_t)b, 64, q + 64 * e};
    }
  } else {
    const int inc = inclusive_scan(ntq);
    __shared__ __align__(16) int32_t tiles_to[16];   // tiles up to and with those of bucket b (past the last bucket: all)
    __shared__ int32_t part_cut[8];
    if (b < 16) tiles_to[b] = inc;
    __syncthreads();
    const int total = tiles_to[N - 1];
    // XCD x has tiles total x / 8 .. total (x + 1) / 8 - 1; of 256-row tiles, those of its last, unfilled round in parts (above; a bucket's end counts
    // as a whole tile).  us a training pass, whole tiles dealt by one thread per bucket -> this: 8832 tokens, d 2048, 4 blocks of 128, 1 each 180 -> 151;
    // 4352, 1024, 8 of 128, 2 113 -> 94; 2491, 2048, 15 of 64, 7 130 -> 118; 51168, 2048, 1 of 32 980 -> 963.
    // (Products of 32 bits: below 2^25 + 16 tiles.)
    const bool in_parts = p.QT == FU_ROWS;
    if (b < 8) {
      const int n = total * (b + 1) / 8 - total * b / 8, left = in_parts ? n % 32 : 0, c = in_parts ? cheapest_cut(left, 0, 0) : 0;
      part_cut[b] = c;
      p.kd_count[b] = n - left + (left << c);
    }
    if (in_parts) __syncthreads();
    for (int t = b; t < total; t += 1024) {
      int o = 0, before = 0;                        // the tile's bucket, and the tiles in front of it
#pragma unroll
      for (int y = 0; y < 15; ++y) {
        const int to = tiles_to[y];
        o += to <= t;
        before = to <= t ? to : before;
      }
      const int x = (int)((8u * t + 7u) / (uint32_t)total), first = total * x / 8, at = t - first;
      const int q = off_sh[o] + (t - before) * p.QT;
      const int full = in_parts ? (total * (x + 1) / 8 - first) / 32 * 32 : total;
      KdTile* list = p.kd_list + (size_t)x * p.cap;
      if (at < full) {
        list[at] = KdTile{(uint16_t)o, (uint16_t)p.QT, q};
      } else {
        const int c = part_cut[x], rows = p.QT >> c, end = off_sh[o + 1];
        for (int e = 0; e < 1 << c; ++e)
          list[full + ((at - full) << c) + e] = KdTile{(uint16_t)o, (uint16_t)(q + e * rows < end ? rows : 0), q + e * rows};
      }
    }
  }
}

// ------------------------------------------------------------------------------------------
// K = d GEMM of one row tile of one bucket for Bs <= 128, activation in the epilogue.
//   MODE 0 (forward, Alg. 4 line 4):  Hsave = Xg W1_b^T,  Hact = act(Hsave)
//   MODE 1 (backward):  dHpre = (dYg W2_b^T) * act'(Hsave),  Hact = act(Hsave)
// Hsave is row-major [P, Bs] (it crosses the ABI); Hact and dHpre are in fragment order (hfrag_off).
// C[u][q] is computed with hidden units as MFMA rows, so a lane holds hidden units of ITS bucket row q.  The K = Bs contraction that
// follows (down-projection, dX) is the token-range-stationary kernel of ffn_scatter.hip.
// Two kernels: tiles of 256 rows, eight wavefronts, one workgroup per CU, the gathered rows and the weight block through an LDS ring
// (global_load_lds_dwordx4, the gather folded into the copy addresses), bound by bytes entering the CU
// (ffn_up_pair_kernel); and, where those would leave CUs without a tile, 32 hidden units x 64 rows a workgroup, operands straight into
// registers (ffn_up_few_rows_kernel).
constexpr int FU_ROWS_FEW = 64;   // rows of a tile where 256-row tiles would leave CUs without one

// Epilogue of a 32-row tile whose hidden units went through rho32: units 32 (first + mi) + 16 h + (0..15) in c[mi], stored as 32-byte
// runs; only the first `many` of the tiles are (all of them where that is a constant, which costs nothing).
template <int MODE, int ACT, int MI>
__device__ __forceinline__ void up_store_runs(const f32x16 (&c)[MI], int q, int q0, int qend, int first, int many, int h,
                                              int Bs, uint16_t* __restrict__ Hsave, uint16_t* __restrict__ Hact,
                                              uint16_t* __restrict__ dHpre) {
  const bool live = q < qend;
  const int ql = live ? q : q0;
  uint4* hs = reinterpret_cast<uint4*>(Hsave + (size_t)ql * Bs + 32 * first + 16 * h);   // 32 units further: 4 words
  const size_t f0 = hfrag_off(ql, 32 * first + 16 * h, Bs);                              // 32 units further: 1024 values
  uint4 z[MODE ? MI : 1][2];
  if (MODE)
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) {
      if (mi >= many) break;
      z[mi][0] = hs[4 * mi];
      z[mi][1] = hs[4 * mi + 1];
    }
#pragma unroll
  for (int mi = 0; mi < MI; ++mi) {
    if (mi >= many) break;
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
      if (MODE == 0) {
        uint32_t hw[4], aw[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          hw[e] = pack_bf16x2(c[mi][8 * hf + 2 * e], c[mi][8 * hf + 2 * e + 1]);
          aw[e] = pack_bf16x2(act_fn<ACT>(c[mi][8 * hf + 2 * e]), act_fn<ACT>(c[mi][8 * hf + 2 * e + 1]));
        }
        if (live) {
          if (Hsave) hs[4 * mi + hf] = make_uint4(hw[0], hw[1], hw[2], hw[3]);
          reinterpret_cast<uint4*>(Hact + f0 + 1024 * mi)[hf] = make_uint4(aw[0], aw[1], aw[2], aw[3]);
        }
      } else {
        const uint4 zq = z[MODE ? mi : 0][hf];
        const uint32_t zw[4] = {zq.x, zq.y, zq.z, zq.w};
        uint32_t gw[4], aw[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float zl = lo_bf16(zw[e]), zh = hi_bf16(zw[e]);
          gw[e] = pack_bf16x2(c[mi][8 * hf + 2 * e] * act_grad<ACT>(zl), c[mi][8 * hf + 2 * e + 1] * act_grad<ACT>(zh));
          aw[e] = pack_bf16x2(act_fn<ACT>(zl), act_fn<ACT>(zh));
        }
        if (live) {
          reinterpret_cast<uint4*>(dHpre + f0 + 1024 * mi)[hf] = make_uint4(gw[0], gw[1], gw[2], gw[3]);
          reinterpret_cast<uint4*>(Hact + f0 + 1024 * mi)[hf] = make_uint4(aw[0], aw[1], aw[2], aw[3]);
        }
      }
      // keep the scheduler from interleaving the groups: their erf evaluations would otherwise all be in
      // flight at once and spill
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// The K = d GEMM of a 256-row tile with eight wavefronts, one workgroup per CU, in stages of 64 K-values.
// A row then contributes 128 contiguous bytes to a stage, a whole line: an LDS copy of 64-byte pieces reaches
// 64-80 bytes per ns and CU out of L2, one of 128-byte pieces 125, and the tile wants 48 KiB per 1024 matrix-core
// cycles.  (With 64-byte pieces, two workgroups of four wavefronts: 364 us on the 7B-like shape, 326 with every
// operand in L2.)  Wavefronts w and w + 4 share a SIMD and 64 bucket rows; each takes half of every stage's K-steps
// (the two sums are added through LDS at the end), and they work in opposite phases: while one reads its fragments
// of a stage the other multiplies, a barrier between the phases, so neither the matrix cores nor LDS wait for the
// other.  Ring of three stages: the slot of stage kt - 1 is filled again (stage kt + 2) as soon as both have
// read it.
template <int KS>
struct UpPair {
  static constexpr int UNITS = KS * 16, ROWS = UNITS + FU_ROWS;
  static constexpr int STAGE = ROWS * 128;        // bytes: 48 KiB at 128 units
  static constexpr int SLOTS = KS <= 4 ? 4 : 3;
  static constexpr int SMEM = SLOTS * STAGE;
};
// 16-byte chunk c of a 128-byte row lies at physical chunk c ^ up_swz(row): one chunk of the 16 rows that are read together
// -- consecutive bucket rows, hidden units in rho32 order -- then covers all banks.
__device__ __forceinline__ int up_swz_row(int row) { return (row >> 1) & 7; }
__device__ __forceinline__ int up_swz_unit(int row) { return ((row >> 1) & 3) | ((row >> 2) & 4); }

// A tile of R rows: 256 (the rule), 128 or 64 (what is left over, see plan_kernel).  A pair of wavefronts then shares R / 4 rows
// of all units; at 64 rows 32 rows of half the 32-unit tiles.
template <int KS, int R>
struct UpPart {
  static constexpr int MI = KS / 2;                                 // 32-unit tiles of the block
  static constexpr int NI = R == 256 ? 2 : 1;                       // 32-row tiles of a wavefront
  static constexpr int MW = R == 64 ? (MI + 1) / 2 : MI;            // ... and its 32-unit tiles
  static constexpr int STAGE = (KS * 16 + R) * 128;                 // bytes
  static constexpr int FIT = UpPair<KS>::SMEM / STAGE;
  static constexpr int SLOTS = FIT < 8 ? FIT : 8;                   // (what a small stage leaves free: copies further ahead)
};

// One tile of R rows, from q0, of bucket b.
template <int MODE, int ACT, int KS, bool EXT, int R>
__device__ __forceinline__ void up_pair_tile(
    const uint16_t* __restrict__ Wa, const uint16_t* __restrict__ Act, int b, int q0, int qend,
    const int32_t* __restrict__ tok, int Bs, int d, uint16_t* __restrict__ Hsave, uint16_t* __restrict__ Hact,
    uint16_t* __restrict__ dHpre, const uint16_t* __restrict__ Xe, const uint16_t* __restrict__ We) {
  typedef UpPart<KS, R> Part;
  constexpr int UNITS = KS * 16, MI = Part::MI, NI = Part::NI, MW = Part::MW, SLOTS = Part::SLOTS, STAGE = Part::STAGE;
  constexpr int PA = 2 * KS;                           // copies of the weight rows of a stage (8 rows each)
  constexpr int NA = (PA + 7) / 8, NB = R / 64, NP = NA + NB;   // copies of a wavefront per stage
  extern __shared__ uint4 fu_smem[];
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int grp = wave >> 2, rw = wave & 3;
  const int row0 = R == 64 ? (rw & 1) * 32 : rw * (R / 4);      // first row of the pair
  const int mi0 = R == 64 ? (rw >> 1) * MW : 0;                 // its first unit tile
  const uint32_t lds0 = (uint32_t)(uintptr_t)fu_smem;
  const char* ring = reinterpret_cast<const char*>(fu_smem);
  const int nkd = d / 64, nk = nkd + (EXT ? 1 : 0), klast = nk - 1;   // (EXT, low-rank adapters: one stage more)
  // (lane roles from an opaque thread id: as loop invariants they would be kept, spilled, across the tiles)
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int lane = tid & 63, i = lane & 31, h = lane >> 5;
  // fragment addresses: chunk 2 s + h of the lane's hidden unit / bucket row (and 32, 64, ... further); this
  // wavefront's K-steps are s = 2 grp, 2 grp + 1
  uint32_t foff_a[2], foff_b[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const int ch = 2 * (2 * grp + s) + h;
    foff_a[s] = (uint32_t)(rho32(i) * 128 + ((ch ^ up_swz_unit(rho32(i))) << 4));
    foff_b[s] = (uint32_t)(i * 128 + ((ch ^ up_swz_row(i)) << 4));
  }
  // DMA: instruction p of a stage fills rows 8 p .. 8 p + 7; lane L row L / 8, physical chunk L % 8.
  const uint16_t* arow[NA];
  const uint16_t* brow[NB];
  int urow[NA], apiece[NA], tq[NB];
#pragma unroll
  for (int j = 0; j < NA; ++j) {
    apiece[j] = (wave * NA + j) % PA;   // (surplus instructions repeat one: same bytes to the same place)
    const int row = apiece[j] * 8 + (lane >> 3);
    urow[j] = b * Bs + row;
    arow[j] = Wa + (size_t)urow[j] * d + (((lane & 7) ^ up_swz_unit(row)) << 3);
  }
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int row = (wave * NB + j) * 8 + (lane >> 3);
    tq[j] = tok[(q0 + row < qend) ? q0 + row : q0];
    brow[j] = Act + (size_t)tq[j] * d + (((lane & 7) ^ up_swz_row(row)) << 3);
  }
  auto issue_piece = [&](int slot, int kt, int piece) {
    const uint32_t base = lds0 + (uint32_t)(slot * STAGE);
    const bool ext = EXT && kt >= nkd;
    if (piece < NA) {
      const int j = piece;
      const int ch8 = ((lane & 7) ^ up_swz_unit(apiece[j] * 8 + (lane >> 3))) << 3;
      dma16(ext ? We + (size_t)urow[j] * 64 + ch8 : arow[j] + kt * 64,
            __builtin_amdgcn_readfirstlane(base + (uint32_t)(apiece[j] * 1024)));
    } else {
      const int j = piece - NA;
      const int ch8 = ((lane & 7) ^ up_swz_row((wave * NB + j) * 8 + (lane >> 3))) << 3;
      dma16(ext ? Xe + (size_t)tq[j] * 64 + ch8 : brow[j] + kt * 64,
            __builtin_amdgcn_readfirstlane(base + (uint32_t)(UNITS * 128 + (wave * NB + j) * 1024)));
    }
  };
  bf16x8 a[2][MW], bb[2][NI];
  auto read_frags = [&](int slot) {
    const char* st = ring + slot * STAGE;
    const char* bt = st + UNITS * 128 + row0 * 128;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
#pragma unroll
      for (int mi = 0; mi < MW; ++mi) {
        const int at = R == 64 ? min(mi0 + mi, MI - 1) : mi;   // (odd count of unit tiles: the second half repeats the last)
        a[s][mi] = *reinterpret_cast<const bf16x8*>(st + foff_a[s] + at * 4096);
      }
#pragma unroll
      for (int ni = 0; ni < NI; ++ni) bb[s][ni] = *reinterpret_cast<const bf16x8*>(bt + foff_b[s] + ni * 4096);
    }
  };
  f32x16 acc[MW][NI];
#pragma unroll
  for (int mi = 0; mi < MW; ++mi)
#pragma unroll
    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[mi][ni][v] = 0.f;
  // the products of the fragments in registers, with stage min(kf, klast) copied into `slot` behind them
  auto multiply = [&](bool fill, int slot, int kf) {
    constexpr int M = 2 * MW * NI;                  // MFMAs
    constexpr int C0 = M >= NP + 4 ? 4 : 0;         // first one with a copy behind it
    const int kfill = kf < klast ? kf : klast;
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int mi = 0; mi < MW; ++mi)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) {
          acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[s][mi], bb[s][ni], acc[mi][ni], 0, 0, 0);
          const int m = (s * MW + mi) * NI + ni;
          if (fill && m >= C0 && m < C0 + NP) {
            issue_piece(slot, kfill, m - C0);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
    if (fill)
#pragma unroll
      for (int p = M - C0; p < NP; ++p) issue_piece(slot, kfill, p);   // (small tiles: fewer MFMAs than copies)
    __builtin_amdgcn_sched_barrier(0);
  };

  __builtin_amdgcn_s_barrier();  // LDS of the previous tile is free
#pragma unroll
  for (int st = 0; st < SLOTS - 1; ++st)
#pragma unroll
    for (int p = 0; p < NP; ++p) issue_piece(st, klast < st ? klast : st, p);
  wait_vmcnt<(SLOTS - 2) * NP>();
  // Phase A of stage kt (after the first barrier): wavefronts 0-3 read it, 4-7 multiply stage kt - 1; phase B: the
  // other way round.  Each sends its copies of stage kt + SLOTS - 1 behind its own products; at the end of
  // phase B its copies of stage kt + 1 have landed.
  int slot = 0, fill = SLOTS - 1;
  auto step = [&] {
    slot = slot + 1 == SLOTS ? 0 : slot + 1;
    fill = fill + 1 == SLOTS ? 0 : fill + 1;
  };
  if (grp == 0) {
    for (int kt = 0; kt < nk; ++kt) {
      __builtin_amdgcn_s_barrier();
      read_frags(slot);
      __builtin_amdgcn_sched_barrier(0);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_s_barrier();
      multiply(true, fill, kt + SLOTS - 1);
      wait_vmcnt<(SLOTS - 2) * NP>();
      step();
    }
  } else {
    for (int kt = 0; kt < nk; ++kt) {
      __builtin_amdgcn_s_barrier();
      if (kt > 0) {
        multiply(true, fill, kt + SLOTS - 1);
      } else {
#pragma unroll
        for (int p = 0; p < NP; ++p) issue_piece(fill, klast < SLOTS - 1 ? klast : SLOTS - 1, p);
      }
      __builtin_amdgcn_s_barrier();
      read_frags(slot);
      __builtin_amdgcn_sched_barrier(0);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      wait_vmcnt<(SLOTS - 2) * NP>();
      step();
    }
    multiply(false, 0, 0);
  }
  wait_vmcnt<0>();               // the trailing copies (repeats of the last stage) are done too
  __builtin_amdgcn_s_barrier();  // ... everyone's: the ring is free
  // The two sums of a pair are added: wavefront w finishes the first KEEP of its 32 x 32 tiles (R = 256: all units of rows
  // 0-31; else the first half of the unit tiles), w + 4 the rest; each hands the other its sums of the other's.
  f32x4* xch = reinterpret_cast<f32x4*>(fu_smem) + lane;
  constexpr int TILES = MW * NI, KEEP = (TILES + 1) / 2;
  // tile t: R = 256 unit tile t % MW of rows 32 (t / MW); else unit tile t
#pragma unroll
  for (int t = 0; t < KEEP; ++t) {
    constexpr int last = TILES - 1;
    const int give0 = KEEP + t < TILES ? KEEP + t : last, give1 = t;   // what wavefronts w / w + 4 hand over
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      f32x4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = grp ? acc[give1 % MW][give1 / MW][4 * g + e] : acc[give0 % MW][give0 / MW][4 * g + e];
      xch[((rw * 2 + (grp ^ 1)) * KEEP * 4 + t * 4 + g) * 64] = o;
    }
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  f32x16 c[KEEP];
#pragma unroll
  for (int t = 0; t < KEEP; ++t) {
    constexpr int last = TILES - 1;
    const int mine0 = t, mine1 = KEEP + t < TILES ? KEEP + t : last;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const f32x4 o = xch[((rw * 2 + grp) * KEEP * 4 + t * 4 + g) * 64];
#pragma unroll
      for (int e = 0; e < 4; ++e)
        c[t][4 * g + e] = (grp ? acc[mine1 % MW][mine1 / MW][4 * g + e] : acc[mine0 % MW][mine0 / MW][4 * g + e]) + o[e];
    }
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  if (R == 256) {
    up_store_runs<MODE, ACT, KEEP>(c, q0 + row0 + grp * 32 + i, q0, qend, 0, MI, h, Bs, Hsave, Hact, dHpre);
  } else {
    // (an odd count of tiles: what is listed behind the last one is not stored)
    const int mine = mi0 + (grp ? KEEP : 0), many = min((grp ? TILES - KEEP : KEEP), MI - mine);
    up_store_runs<MODE, ACT, KEEP>(c, q0 + row0 + i, q0, min(qend, q0 + R), mine, many, h, Bs, Hsave, Hact, dHpre);
  }
}

// Registers: 198 to 200 of 256 at 128 units, 219 to 221 with the adapters' stage (EXT); nothing spills.
template <int MODE, int ACT, int KS, bool EXT>
__global__ __launch_bounds__(512, 2) void ffn_up_pair_kernel(
    const uint16_t* __restrict__ Wa, const uint16_t* __restrict__ Act, const int32_t* __restrict__ offsets,
    const int32_t* __restrict__ kd_count, const KdTile* __restrict__ kd_list, int cap, const int32_t* __restrict__ tok,
    int Bs, int d, uint16_t* __restrict__ Hsave, uint16_t* __restrict__ Hact, uint16_t* __restrict__ dHpre,
    const uint16_t* __restrict__ Xe, const uint16_t* __restrict__ We) {
  const int xcd = blockIdx.x & 7, wg_per_xcd = gridDim.x >> 3;
  const int count = kd_count[xcd];
  for (int slot_id = blockIdx.x >> 3; slot_id < count; slot_id += wg_per_xcd) {
    const KdTile tile = kd_list[(size_t)xcd * cap + slot_id];
    const int b = tile.bucket, q0 = tile.q0, qend = offsets[b + 1];
#define SPT_TILE(R) up_pair_tile<MODE, ACT, KS, EXT, R>(Wa, Act, b, q0, qend, tok, Bs, d, Hsave, Hact, dHpre, Xe, We)
    if (tile.rows == FU_ROWS) SPT_TILE(256);
    else if (tile.rows == 128) SPT_TILE(128);
    else if (tile.rows == 64) SPT_TILE(64);        // (0: an entry without rows)
#undef SPT_TILE
  }
}

// ------------------------------------------------------------------------------------------
// The same GEMMs where 256-row tiles would leave CUs without one: decoding batches, where every weight is read for few
// multiply-adds, and small layers, where a tile's K loop is a chain of memory latencies.  Both want bytes in flight on all
// CUs.  A workgroup owns 32 hidden units of one block and one row tile of at most 64 rows of its bucket, 32 RT rows at a time; its four
// wavefronts split d in chunks of 64 values and load both operands straight into registers, a chunk ahead.  The
// wavefronts' sums are added through LDS in order.
// A lane multiplies values of one row, but four lanes in a row, which want four rows, request 64 adjacent bytes of each of them
// in turn and exchange the 16-byte pieces afterwards (quad_transpose): four pieces of one line cost what one piece of each of four lines
// costs four times.  us, 24 and 100 tokens of the 7B-like layer (6 and 25 rows a bucket): each lane its own row 25, 51; this 17, 28.
// (Which layers take it, and both sides of the line: few_rows.)
// The row tiles come from the schedule's lists, as those of the tile kernel do: the mean says little about a single
// bucket.  8192 tokens, 256 blocks of 128 units, d 2048, k 1, half of the tokens in one block: 220 us, with a
// workgroup per bucket and 32 units 2834.
template <int MODE, int ACT, int RT, bool EXT>
__global__ __launch_bounds__(256) void ffn_up_few_rows_kernel(
    const uint16_t* __restrict__ Wa, const uint16_t* __restrict__ Act, const int32_t* __restrict__ offsets,
    const int32_t* __restrict__ kd_count, const KdTile* __restrict__ kd_list, int cap,
    const int32_t* __restrict__ tok, int Bs, int d, uint16_t* __restrict__ Hsave, uint16_t* __restrict__ Hact,
    uint16_t* __restrict__ dHpre, const uint16_t* __restrict__ Xe, const uint16_t* __restrict__ We) {
  constexpr int DEPTH = 2;                       // chunks in registers, one of them in flight (3 or 4, less of them on a CU: 17 -> 18, 28 -> 31)
  __shared__ float red[4][RT][16][64];
  // (the unit slices of a tile side by side; workgroups that find the list at its end are the last ones handed out)
  const int slices = Bs / 32, xcd = blockIdx.x & 7, per_xcd = (int)(gridDim.x >> 3) / slices, count = kd_count[xcd];
  const int u0 = (int)(blockIdx.x >> 3) % slices * 32;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i = lane & 31, h = lane >> 5, at = 32 * h + 8 * (lane & 3);   // the lane's piece of a chunk
  const int chunks = d / 64, cbeg = wave * chunks / 4, cend = (wave + 1) * chunks / 4, clast = cend - 1;
  for (int slot = (int)(blockIdx.x >> 3) / slices; slot < count; slot += per_xcd) {
    const KdTile tile = kd_list[(size_t)xcd * cap + slot];
    const int qe = min(tile.q0 + tile.rows, offsets[tile.bucket + 1]);
    const size_t unit0 = (size_t)tile.bucket * Bs + u0;
    const uint16_t* wrow[4];                     // rows of the lane's group of four
#pragma unroll
    for (int j = 0; j < 4; ++j) wrow[j] = Wa + (unit0 + rho32((i & ~3) + j)) * d + at;
    for (int q0 = tile.q0; q0 < qe; q0 += 32 * RT) {
      int tokens[RT][4];
      const uint16_t* xrow[RT][4];
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int j = 0; j < 4; ++j) tokens[rt][j] = tok[min(q0 + rt * 32 + (i & ~3) + j, qe - 1)];
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int j = 0; j < 4; ++j) xrow[rt][j] = Act + (size_t)tokens[rt][j] * d + at;
      f32x16 acc[RT];
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[rt][v] = 0.f;
      bf16x8 wq[DEPTH][4], xq[DEPTH][RT][4];
      auto fetch = [&](int st, int c) {
        const int k0 = min(c, clast) * 64;       // (requests past the last chunk repeat it: no branch around a load)
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          wq[st][s] = as_bf16x8(*reinterpret_cast<const uint4*>(wrow[s] + k0));
#pragma unroll
          for (int rt = 0; rt < RT; ++rt) xq[st][rt][s] = as_bf16x8(*reinterpret_cast<const uint4*>(xrow[rt][s] + k0));
        }
      };
      auto consume = [&](int st) {
        quad_transpose(wq[st], lane);
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) quad_transpose(xq[st][rt], lane);
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
          for (int rt = 0; rt < RT; ++rt)
            acc[rt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wq[st][s], xq[st][rt][s], acc[rt], 0, 0, 0);
      };
      if (cbeg < cend) {
#pragma unroll
        for (int s = 0; s < DEPTH - 1; ++s) fetch(s, cbeg + s);
        int c = cbeg;
        for (; c + DEPTH <= cend; c += DEPTH) {
#pragma unroll
          for (int s = 0; s < DEPTH; ++s) {
            fetch((s + DEPTH - 1) % DEPTH, c + s + DEPTH - 1);
            consume(s);
          }
        }
#pragma unroll
        for (int s = 0; s < DEPTH - 1; ++s)
          if (c + s < cend) consume(s);
      }
      if (EXT && wave == 3) {                    // low-rank adapters: 64 more values of every row, and one chunk more
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          wq[0][s] = as_bf16x8(*reinterpret_cast<const uint4*>(We + (unit0 + rho32((i & ~3) + s)) * 64 + at));
#pragma unroll
          for (int rt = 0; rt < RT; ++rt) xq[0][rt][s] = as_bf16x8(*reinterpret_cast<const uint4*>(Xe + (size_t)tokens[rt][s] * 64 + at));
        }
        consume(0);
      }
      // wavefront w finishes accumulators 4 w .. 4 w + 3: hidden units u0 + 16 h + 4 w .. + 3 of the lane's row
      const int u = u0 + 16 * h + 4 * wave;
      uint2 zsave[RT];
      if (MODE)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) zsave[rt] = *reinterpret_cast<const uint2*>(Hsave + (size_t)min(q0 + rt * 32 + i, qe - 1) * Bs + u);
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int v = 0; v < 16; ++v) red[wave][rt][v][lane] = acc[rt][v];
      __syncthreads();
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        const int q = q0 + rt * 32 + i;
        float z[4];
#pragma unroll
        for (int e = 0; e < 4; ++e)
          z[e] = ((red[0][rt][4 * wave + e][lane] + red[1][rt][4 * wave + e][lane]) + red[2][rt][4 * wave + e][lane]) +
                 red[3][rt][4 * wave + e][lane];
        if (q < qe) {
          if (MODE) {
            const float h0 = lo_bf16(zsave[rt].x), h1 = hi_bf16(zsave[rt].x), h2 = lo_bf16(zsave[rt].y), h3 = hi_bf16(zsave[rt].y);
            *reinterpret_cast<uint2*>(dHpre + hfrag_off(q, u, Bs)) =
                make_uint2(pack_bf16x2(z[0] * act_grad<ACT>(h0), z[1] * act_grad<ACT>(h1)),
                           pack_bf16x2(z[2] * act_grad<ACT>(h2), z[3] * act_grad<ACT>(h3)));
            z[0] = h0; z[1] = h1; z[2] = h2; z[3] = h3;
          } else if (Hsave) {
            *reinterpret_cast<uint2*>(Hsave + (size_t)q * Bs + u) = make_uint2(pack_bf16x2(z[0], z[1]), pack_bf16x2(z[2], z[3]));
          }
          *reinterpret_cast<uint2*>(Hact + hfrag_off(q, u, Bs)) =
              make_uint2(pack_bf16x2(act_fn<ACT>(z[0]), act_fn<ACT>(z[1])), pack_bf16x2(act_fn<ACT>(z[2]), act_fn<ACT>(z[3])));
        }
      }
      __syncthreads();
    }
  }
}

// ------------------------------------------------------------------------------------------
// The weight-gradient GEMMs (ffn_dw.hpp).  blockIdx.z picks the product: both weight gradients of a step can go out in one launch.
template <int UT>
__global__ __launch_bounds__(256, 2) void kq_gemm_kernel(
    DwOperands ops0, DwOperands ops1,
    const int32_t* __restrict__ tok, const uint16_t* __restrict__ zero_row, int npieces, int Bs,
    int d, const DwPiece* __restrict__ pieces, int nblocks) {
  dw_tile<UT>(blockIdx.z ? ops1 : ops0, blockIdx.x, blockIdx.y, tok, zero_row, npieces, Bs, d, pieces, nblocks);
}

// dW[b] += stage[first] + ... + stage[end - 1] (in that order) for every bucket b that was cut
// into more than one piece; xlist = (count, then (bucket, first slot, end slot) triples).
__global__ __launch_bounds__(256) void dw_reduce_kernel(DwOperands ops0, DwOperands ops1,
                                                        const int32_t* __restrict__ xlist, int Bs, int d) {
  float* __restrict__ dW = blockIdx.y ? ops1.dW : ops0.dW;
  const float* __restrict__ stage = blockIdx.y ? ops1.stage : ops0.stage;
  const int count = xlist[0];
  const size_t e4 = (size_t)Bs * d / 4;   // 16-byte groups per block
  for (size_t it = (size_t)blockIdx.x * 256 + threadIdx.x; it < (size_t)count * e4;
       it += (size_t)gridDim.x * 256) {
    const int l = (int)(it / e4);
    const size_t e = it % e4;
    const int b = xlist[1 + 3 * l], first = xlist[2 + 3 * l], end = xlist[3 + 3 * l];
    f32x4* acc = reinterpret_cast<f32x4*>(dW + (size_t)b * Bs * d) + e;
    f32x4 v = *acc;
    for (int x = first; x < end; ++x) v += reinterpret_cast<const f32x4*>(stage + (size_t)x * Bs * d)[e];
    *acc = v;
  }
}

// ------------------------------------------------------------------------------------------
// Combine: out[t][:] = sum_{j<k} part[inv[t*k+j]][:], j ascending, fp32, one rounding to bf16.
// This is Alg. 4's write-back with block outputs added (k > 1 blocks per token).
__global__ __launch_bounds__(256) void combine_kernel(const uint16_t* __restrict__ part,
                                                      const int32_t* __restrict__ inv, int T, int d, int k,
                                                      uint16_t* __restrict__ out) {
  const int cpr = d >> 3;  // 16-byte groups per row
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= (int64_t)T * cpr) return;
  const int t = (int)(gid / cpr), cg = (int)(gid % cpr);
  float a[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) a[e] = 0.f;
  const int32_t* iv = inv + (size_t)t * k;
  part += cg * 8;
  int j = 0;
  for (; j + 8 <= k; j += 8) {
    u32x4 v[8];
#pragma unroll
    for (int jj = 0; jj < 8; ++jj)
      v[jj] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(part + (size_t)iv[j + jj] * d));
#pragma unroll
    for (int jj = 0; jj < 8; ++jj) {
      a[0] += lo_bf16(v[jj].x); a[1] += hi_bf16(v[jj].x);
      a[2] += lo_bf16(v[jj].y); a[3] += hi_bf16(v[jj].y);
      a[4] += lo_bf16(v[jj].z); a[5] += hi_bf16(v[jj].z);
      a[6] += lo_bf16(v[jj].w); a[7] += hi_bf16(v[jj].w);
    }
  }
  for (; j < k; ++j) {
    const uint4 v = *reinterpret_cast<const uint4*>(part + (size_t)iv[j] * d);
    a[0] += lo_bf16(v.x); a[1] += hi_bf16(v.x);
    a[2] += lo_bf16(v.y); a[3] += hi_bf16(v.y);
    a[4] += lo_bf16(v.z); a[5] += hi_bf16(v.z);
    a[6] += lo_bf16(v.w); a[7] += hi_bf16(v.w);
  }
  *reinterpret_cast<uint4*>(out + (size_t)t * d + cg * 8) =
      make_uint4(pack_bf16x2(a[0], a[1]), pack_bf16x2(a[2], a[3]), pack_bf16x2(a[4], a[5]),
                 pack_bf16x2(a[6], a[7]));
}

// ------------------------------------------------------------------------------------------
// host side
static int max_row_tiles(const spt_shape_t& s, int rows) {
  const int64_t P = (int64_t)s.T * s.k;
  return (int)((P + rows - 1) / rows) + s.N;
}

static bool use_narrow(const spt_shape_t& s) { return s.Bs <= TILE; }

// Narrow blocks: tiles of 64 rows, and the kernel that loads its operands straight into registers, where those are about two workgroups (32 hidden
// units each) per CU at most, or a bucket has few rows and the weights are what is read.  us a pass on inputs that change, 256-row tiles (and their
// parts) / this: training 1024 tokens, d 2048, 16 blocks of 128, 4 each (288 workgroups) 99.3 / 96.8; 300, 4096, 64 of 128, 16 (428) 211 / 202; 1000,
// 3008, 24 of 96, 8 (411) 150 / 146; 2048, 4096, 16 of 128, 4 (544) 182 / 189; 1500, 768, 32 of 96, 8 (611) 84 / 86; 2048 of those (816) 96 / 102.
// Fewer than 16 blocks: 2240 tokens, d 2048, 4 of 128, 1 each (148) 84 / 79; 3712, 2048, 8 of 128, 2 (480) 111 / 111; 7648, 1024, 1 of 128 (480)
// 187 / 187; 4384, 512, 12 of 64, 4 (560) 80 / 85; 8832, 2048, 4 of 128, 1 (560) 151 / 160.
// From 128 blocks on, of more than 32 units, their 256-row tiles fill half the CUs themselves: up to 40 rows a bucket.  Even routing: 3840 tokens, d 4096,
// 128 of 128, 1 each (30 rows) 537 / 532; 640, 4096, 128 of 128, 8 (40) 354 / 346; 768 of those (48) 364 / 369; 768, 1024, 128 of 64, 8 (48) 100 / 103; 7686,
// 1024, 183 of 96, 1 (42) 326 / 334; 32 units: 897, 1664, 129, 22 161 / 155.  Skewed: 1920, 2048, 128 of 128, 2 (30) 259 / 265; 1536, 1024, 256 of 64, 8 (48)
// 200 / 200; 790, 1600, 129 of 64, 8 (48) 143 / 148.  Prefill of the 7B-like layer, 192 tokens (48) 117 / 115, 256 tokens 126 / 131.
static bool few_rows(const spt_shape_t& s) {
  const int64_t P = (int64_t)s.T * s.k;
  if (!use_narrow(s)) return false;
  return P <= 40 * (int64_t)s.N ||
         ((s.N < 128 || s.Bs == 32) && (P + FU_ROWS_FEW / 2 * (int64_t)s.N) / FU_ROWS_FEW * (s.Bs / 32) <= 512);
}
static int kd_rows(const spt_shape_t& s) { return few_rows(s) ? FU_ROWS_FEW : FU_ROWS; }

static size_t carve_schedule(const spt_shape_t& s, char* p, size_t o0, Schedule& sc, bool weight_grads = false) {
  const size_t P = (size_t)s.T * s.k;
  size_t o = o0;
  sc.kd_cap = max_row_tiles(s, kd_rows(s));
  if (kd_rows(s) == FU_ROWS && use_narrow(s)) sc.kd_cap += 4 * 32 + (s.N + 7) / 8 * 2;   // (a last round cut into quarters, two entries per bucket's end)
  sc.border = reinterpret_cast<int32_t*>(p + o);      o += align256((size_t)s.N * 4);
  sc.kd_count = reinterpret_cast<int32_t*>(p + o);    o += align256(8 * 4);
  sc.kd_list = p + o;                                 o += align256((size_t)8 * sc.kd_cap * sizeof(KdTile));
  sc.tok = reinterpret_cast<int32_t*>(p + o);         o += align256(P * 4);
  sc.zero_row = reinterpret_cast<uint16_t*>(p + o);   o += 256;
  sc.rstart = nullptr;
  if (use_narrow(s)) {
    sc.rstart = reinterpret_cast<int32_t*>(p + o);    o += plan_scatter(s).table_bytes;
  }
  sc.dw_pieces = nullptr; sc.dw_xlist = nullptr; sc.dw_cap = 0; sc.dw_rows = 0;
  if (use_narrow(s) && weight_grads) {
    // pieces of at most 1.5 x the mean bucket (never below 256 rows): balanced routing is left
    // alone, a bucket several times the mean no longer holds up the whole launch.  Up to 512 tokens a bucket stays whole, whatever
    // the routing: the sum of the pieces is a launch more.  us a pass, in pieces and whole: 512 tokens, d 256, 16 blocks of 64, 4 each, even
    // 50.1 / 47.1, skewed 51.2 / 49.9; d 2048, 64 of 128, 16, skewed 162 / 157.
    const int64_t mean15 = (3 * (int64_t)P / s.N + 1) / 2;
    sc.dw_rows = (int)((mean15 < 256 ? 256 : mean15) + 15) / 16 * 16;
    if (s.T <= 512 || s.T <= sc.dw_rows) sc.dw_rows = (int)P + 1;   // (each token at most once in a bucket: T rows)
    sc.dw_cap = s.N + (int)(P / sc.dw_rows);
    sc.dw_pieces = reinterpret_cast<DwPiece*>(p + o);  o += align256((size_t)sc.dw_cap * sizeof(DwPiece));
    sc.dw_xlist = reinterpret_cast<int32_t*>(p + o);   o += align256((size_t)(1 + 3 * s.N) * 4);
  }
  return o - o0;
}

static size_t hrows(size_t P) { return (P + 31) / 32 * 32; }  // rows of a tensor in fragment order

// Partial rows exist only on the wide-block path.
static size_t carve_part(const spt_shape_t& s, char* p, size_t o0, uint16_t*& part) {
  part = nullptr;
  if (use_narrow(s)) return 0;
  part = reinterpret_cast<uint16_t*>(p + o0);
  return align256((size_t)s.T * s.k * (size_t)s.d * 2);
}

FwdWorkspace plan_fwd(const spt_shape_t& s, void* ws) {
  const size_t P = (size_t)s.T * s.k;
  char* p = static_cast<char*>(ws);
  size_t o = 0;
  FwdWorkspace w;
  o += carve_schedule(s, p, o, w.sched);
  w.Hact = reinterpret_cast<uint16_t*>(p + o);       o += align256(hrows(P) * s.Bs * 2);
  o += carve_part(s, p, o, w.part);
  w.split = use_narrow(s) ? reinterpret_cast<float*>(p + o) : nullptr;
  o += use_narrow(s) ? plan_scatter(s).split_bytes : 0;
  w.bytes = o;
  return w;
}

BwdWorkspace plan_bwd(const spt_shape_t& s, void* ws, bool weight_grads) {
  const size_t P = (size_t)s.T * s.k;
  char* p = static_cast<char*>(ws);
  size_t o = 0;
  BwdWorkspace w;
  o += carve_schedule(s, p, o, w.sched, weight_grads);
  w.Hact = reinterpret_cast<uint16_t*>(p + o);       o += align256(hrows(P) * s.Bs * 2);
  w.dHpre = reinterpret_cast<uint16_t*>(p + o);      o += align256(hrows(P) * s.Bs * 2);
  o += carve_part(s, p, o, w.part);
  w.split = use_narrow(s) ? reinterpret_cast<float*>(p + o) : nullptr;
  o += use_narrow(s) ? plan_scatter(s).split_bytes : 0;
  w.dw_stage = w.dw_stage2 = nullptr;
  if (w.sched.dw_cap > 0) {
    // Both gradients go out in one launch, with staging slots of their own, unless those are large:
    // where a launch has thousands of work items there is no half-empty last round to share.
    const size_t bytes = align256((size_t)(w.sched.dw_cap - s.N) * s.Bs * s.d * 4);
    w.dw_stage = reinterpret_cast<float*>(p + o);
    o += bytes;
    if (bytes <= ((size_t)64 << 20)) {
      w.dw_stage2 = reinterpret_cast<float*>(p + o);
      o += bytes;
    }
  }
  w.bytes = o;
  return w;
}

size_t schedule_bytes(const spt_shape_t& s) {
  Schedule sc;
  return carve_schedule(s, nullptr, 0, sc, true);
}

Schedule plan_schedule(const spt_shape_t& s, void* buf) {
  Schedule sc;
  carve_schedule(s, static_cast<char*>(buf), 0, sc, true);
  return sc;
}

#define SPT_LAUNCH_CHECK()                 \
  do {                                     \
    hipError_t e_ = hipGetLastError();     \
    if (e_ != hipSuccess) return e_;       \
  } while (0)

static hipError_t run_plan(const spt_shape_t& s, const int32_t* offsets, const int32_t* perm,
                           const Schedule& sc, hipStream_t st) {
  const int P = s.T * s.k;
  const ScatterPlan sp = sc.rstart ? plan_scatter(s) : ScatterPlan{};
  PlanArgs a = {};
  a.offsets = offsets; a.perm = perm;
  a.wide = !use_narrow(s);
  a.tails = a.wide && wide_tails(s);
  // Dealt by size rank, an XCD has of each level (the i-th tiles of all buckets) at most one tile more than another: left so where even then each
  // workgroup has a CU, which costs a small pass 0.7 us less.  (Up to 32 workgroups more whatever there are: 993 tokens, d 2496, 66 blocks of 32, 19 each, skewed 151; spread 142.)
  const int levels = (s.T + FU_ROWS_FEW - 1) / FU_ROWS_FEW, slices = s.Bs / 32;
  a.spread = !a.wide && (!few_rows(s) || (levels > 1 && (max_row_tiles(s, FU_ROWS_FEW) / 8 + levels) * slices > 32));
  a.N = s.N; a.QT = kd_rows(s); a.cap = sc.kd_cap; a.P = P; a.k = s.k;
  a.border = sc.border; a.kd_count = sc.kd_count; a.kd_list = static_cast<KdTile*>(sc.kd_list);
  a.zero_row = reinterpret_cast<uint32_t*>(sc.zero_row);
  a.tok = sc.tok;
  if (sc.rstart) {
    a.R = sp.R; a.nr = sp.nr; a.starts = scatter_starts(sp, sc.rstart);
    a.runs = scatter_runs(sp, sc.rstart); a.nruns = scatter_counts(sp, sc.rstart); a.run_cap = sp.cap; a.run_rows = sp.run_rows;
  }
  a.dw_rows = sc.dw_rows; a.dw_cap = sc.dw_cap; a.dw_pieces = sc.dw_pieces; a.dw_xlist = sc.dw_xlist;
  // One launch, three workgroups side by side (lists; pieces; positions, then run records), where the one that takes all positions is
  // less than a second launch.  us a pass, one launch / two: 6144 pairs in 32 blocks 60.1 / 58.2; 8000 in 16 57 / 55; 16384 in 32 103 / 97; 4096 in 32 34.2 / 36.
  // (The three one after the other in one workgroup, quotients by division, the run starts in memory: the launch 8.6 against 4.8; passes of 512 tokens,
  // d 256, 16 blocks of 64, 4 each 41.3 -> 37.0; 24 tokens, d 4096, 128 of 128, 32 each 79.7 -> 76.6; 100 tokens, d 1024, 128 of 128, 40 each
  // 52.2 -> 45.7; 512 tokens, d 512, 32 of 64, 8 each, forward 39.0 -> 34.2.  Two positions a thread where four are not needed: 0.8 %.)
  const bool all = P <= kAllPairs;
  {
    ScopedKernelTimer tm(kSlotPlan, st);
    if (P <= 2048) plan_kernel<2><<<3, 1024, 0, st>>>(a);
    else if (all) plan_kernel<kAllPairs / 1024><<<3, 1024, 0, st>>>(a);
    else plan_kernel<0><<<2 + (P + 1023) / 1024, 1024, 0, st>>>(a);
  }
  SPT_LAUNCH_CHECK();
  if (sc.rstart && !all) {
    ScopedKernelTimer tm(kSlotPlan, st);
    return run_scatter_ranges(s, sp, sc.rstart, st);
  }
  return hipSuccess;
}

hipError_t run_schedule(const spt_shape_t& s, const int32_t* offsets, const int32_t* perm, const Schedule& sc,
                        hipStream_t st) {
  return run_plan(s, offsets, perm, sc, st);
}

static hipError_t run_combine(const spt_shape_t& s, const uint16_t* part, const int32_t* inv, void* out, int slot,
                              hipStream_t st) {
  const int64_t items = (int64_t)s.T * (s.d / 8);
  ScopedKernelTimer tm(slot, st);
  combine_kernel<<<(unsigned)((items + 255) / 256), 256, 0, st>>>(part, inv, s.T, s.d, s.k, static_cast<uint16_t*>(out));
  SPT_LAUNCH_CHECK();
  return hipSuccess;
}

template <int MODE, int ACT, int KS>
static hipError_t launch_up_t(const spt_shape_t& s, const uint16_t* Wa, const uint16_t* Act,
                              const int32_t* offsets, const Schedule& sc, uint16_t* Hsave, uint16_t* Hact,
                              uint16_t* dHpre, hipStream_t st, const uint16_t* Xe, const uint16_t* We) {
  static const hipError_t attr[2] = {
      hipFuncSetAttribute(reinterpret_cast<const void*>(ffn_up_pair_kernel<MODE, ACT, KS, false>),
                          hipFuncAttributeMaxDynamicSharedMemorySize, UpPair<KS>::SMEM),
      hipFuncSetAttribute(reinterpret_cast<const void*>(ffn_up_pair_kernel<MODE, ACT, KS, true>),
                          hipFuncAttributeMaxDynamicSharedMemorySize, UpPair<KS>::SMEM)};
  const hipError_t e = attr[Xe ? 1 : 0];
  if (e != hipSuccess) return e;
  const int grid = 8 * (sc.kd_cap < 32 ? sc.kd_cap : 32);
  const KdTile* list = static_cast<const KdTile*>(sc.kd_list);
#define SPT_UP_ARGS Wa, Act, offsets, sc.kd_count, list, sc.kd_cap, sc.tok, s.Bs, s.d, Hsave, Hact, dHpre, Xe, We
  if (Xe) ffn_up_pair_kernel<MODE, ACT, KS, true><<<grid, 512, UpPair<KS>::SMEM, st>>>(SPT_UP_ARGS);
  else    ffn_up_pair_kernel<MODE, ACT, KS, false><<<grid, 512, UpPair<KS>::SMEM, st>>>(SPT_UP_ARGS);
  return hipGetLastError();
}

template <int MODE, int ACT>
static hipError_t launch_up_few_rows(const spt_shape_t& s, const uint16_t* Wa, const uint16_t* Act, const int32_t* offsets,
                                     const Schedule& sc, uint16_t* Hsave, uint16_t* Hact, uint16_t* dHpre, hipStream_t st,
                                     const uint16_t* Xe, const uint16_t* We) {
  const int grid = (sc.kd_cap + 7) / 8 * 8 * (s.Bs / 32);   // (an XCD with more tiles than its share takes more rounds)
  const KdTile* list = static_cast<const KdTile*>(sc.kd_list);
  const bool one = (int64_t)s.T * s.k <= (int64_t)24 * s.N;
  if (one) {
    if (Xe) ffn_up_few_rows_kernel<MODE, ACT, 1, true><<<grid, 256, 0, st>>>(SPT_UP_ARGS);
    else    ffn_up_few_rows_kernel<MODE, ACT, 1, false><<<grid, 256, 0, st>>>(SPT_UP_ARGS);
  } else {
    if (Xe) ffn_up_few_rows_kernel<MODE, ACT, 2, true><<<grid, 256, 0, st>>>(SPT_UP_ARGS);
    else    ffn_up_few_rows_kernel<MODE, ACT, 2, false><<<grid, 256, 0, st>>>(SPT_UP_ARGS);
  }
#undef SPT_UP_ARGS
  return hipGetLastError();
}

// K = d GEMM of the narrow-block path.  MODE 0: Hsave (may be null), Hact from Act = X, Wa = W1;
// MODE 1: dHpre, Hact from Act = dY, Wa = W2 and the forward's Hsave.
template <int MODE>
static hipError_t launch_up(const spt_shape_t& s, const uint16_t* Wa, const uint16_t* Act,
                            const int32_t* offsets, const Schedule& sc, uint16_t* Hsave, uint16_t* Hact,
                            uint16_t* dHpre, hipStream_t st, const uint16_t* Xe = nullptr,
                            const uint16_t* We = nullptr) {
  if (few_rows(s))
    return s.act == SPT_ACT_GELU ? launch_up_few_rows<MODE, 0>(s, Wa, Act, offsets, sc, Hsave, Hact, dHpre, st, Xe, We)
                                 : launch_up_few_rows<MODE, 1>(s, Wa, Act, offsets, sc, Hsave, Hact, dHpre, st, Xe, We);
#define SPT_UP(ACT, KS)                                                                                                \
  return launch_up_t<MODE, ACT, KS>(s, Wa, Act, offsets, sc, Hsave, Hact, dHpre, st, Xe, We)
#define SPT_UP_KS(ACT)                    \
  switch (s.Bs / 16) {                    \
    case 2: SPT_UP(ACT, 2);               \
    case 4: SPT_UP(ACT, 4);               \
    case 6: SPT_UP(ACT, 6);               \
    default: SPT_UP(ACT, 8);              \
  }
  if (s.act == SPT_ACT_GELU) { SPT_UP_KS(0) } else { SPT_UP_KS(1) }
#undef SPT_UP_KS
#undef SPT_UP
}

// One instantiation of the weight-gradient GEMM (UT = hidden units per workgroup tile).
template <int UT>
static hipError_t launch_dw_ut(const DwOperands* ops, int nops, const Schedule& sc, int N, int Bs, int d, hipStream_t st) {
  constexpr int dw_smem = dw_smem_bytes<UT>();
  static bool attr_set = false;
  if (!attr_set) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kq_gemm_kernel<UT>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, dw_smem);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  kq_gemm_kernel<UT><<<dim3(dw_grid(sc.dw_cap, d), (Bs + UT - 1) / UT, nops), 256, dw_smem, st>>>(
      ops[0], ops[nops - 1], sc.tok, sc.zero_row, sc.dw_cap, Bs, d, sc.dw_pieces, N);
  return hipGetLastError();
}

// The fixed-order sum of the staged pieces into their blocks (no launch where a routing cannot need any).
static hipError_t launch_dw_sum(const DwOperands* ops, int nops, const Schedule& sc, int N, int Bs, int d, hipStream_t st) {
  if (sc.dw_cap == N) return hipSuccess;
  const size_t groups = (size_t)(sc.dw_cap - N) * Bs * d / 4;   // 16-byte groups of the most blocks that can have pieces
  const unsigned gx = (unsigned)(groups / 256 < 1 ? 1 : groups / 256 > 1024 ? 1024 : groups / 256);
  dw_reduce_kernel<<<dim3(gx, nops), 256, 0, st>>>(ops[0], ops[nops - 1], sc.dw_xlist, Bs, d);
  return hipGetLastError();
}

// dW[b][u][c] = sum_{q in bucket b} Hin[q][u] * Act[tok[q]][c], the narrow-block weight-gradient GEMM over the
// piece table (Schedule::dw_pieces), for one product or two at once, and the sum of its staged pieces.
static hipError_t launch_dw_pieces(const DwOperands* ops, int nops, const Schedule& sc, int N, int Bs, int d, int slot,
                                   hipStream_t st) {
  ScopedKernelTimer tm(slot, st);   // (covers the GEMM and the sum of the staged pieces)
  const hipError_t e = Bs <= 64 ? launch_dw_ut<64>(ops, nops, sc, N, Bs, d, st) : launch_dw_ut<128>(ops, nops, sc, N, Bs, d, st);
  return e != hipSuccess ? e : launch_dw_sum(ops, nops, sc, N, Bs, d, st);
}

static WideArgs wide_args(const spt_shape_t& s, const int32_t* offsets, const Schedule& sc) {
  WideArgs a = {};
  a.offsets = offsets;
  a.kd_count = sc.kd_count;
  a.kd_list = sc.kd_list;
  a.tok = sc.tok;
  a.border = sc.border;
  a.zero_row = sc.zero_row;
  a.N = s.N; a.Bs = s.Bs; a.d = s.d;
  return a;
}

hipError_t run_fwd(const spt_shape_t& s, const void* X, const void* W1, const void* W2,
                   const int32_t* offsets, const int32_t* perm, const int32_t* inv, void* Y,
                   void* Hsave, const FwdWorkspace& w, hipStream_t st, const Schedule* prebuilt) {
  const Schedule& sc = prebuilt ? *prebuilt : w.sched;
  hipError_t e = prebuilt ? hipSuccess : run_plan(s, offsets, perm, sc, st);
  if (e != hipSuccess) return e;
  auto x = static_cast<const uint16_t*>(X);
  auto w1 = static_cast<const uint16_t*>(W1);
  auto w2 = static_cast<const uint16_t*>(W2);
  auto hs = static_cast<uint16_t*>(Hsave);
  if (use_narrow(s)) {
    {
      ScopedKernelTimer tm(kSlotUp, st);
      e = launch_up<0>(s, w1, x, offsets, sc, hs, w.Hact, nullptr, st);
    }
    if (e != hipSuccess) return e;
    ScopedKernelTimer tm(kSlotDown, st);
    return launch_scatter(s, plan_scatter(s), w.Hact, w2, sc.rstart, sc.tok,
                          static_cast<uint16_t*>(Y), nullptr, w.split, st);
  }
  WideArgs a = wide_args(s, offsets, sc);
  a.A = w1; a.B = x; a.Hsave = hs; a.Hact = w.Hact;
  {
    ScopedKernelTimer tm(kSlotUp, st);
    e = launch_wide(kWideUp, s, a, st);
  }
  if (e != hipSuccess) return e;
  a.A = w2; a.B = w.Hact; a.part = w.part;
  {
    ScopedKernelTimer tm(kSlotDown, st);
    e = launch_wide(kWidePart, s, a, st);
  }
  if (e != hipSuccess) return e;
  return run_combine(s, w.part, inv, Y, kSlotCombineY, st);
}

// dX and both weight gradients in one launch.
static bool joined_backward(const spt_shape_t& s, const BwdWorkspace& w, const ScatterPlan& sp) {
  return w.dw_stage2 && scatter_takes_dw(s, sp);
}

hipError_t run_bwd(const spt_shape_t& s, const void* X, const void* W1, const void* W2,
                   const void* dY, const int32_t* offsets, const int32_t* perm,
                   const int32_t* inv, const void* Hsave, void* dX, float* dW1, float* dW2,
                   const BwdWorkspace& w, hipStream_t st, const Schedule* prebuilt) {
  const Schedule& sc = prebuilt ? *prebuilt : w.sched;
  hipError_t e = prebuilt ? hipSuccess : run_plan(s, offsets, perm, sc, st);
  if (e != hipSuccess) return e;
  auto x = static_cast<const uint16_t*>(X);
  auto w1 = static_cast<const uint16_t*>(W1);
  auto w2 = static_cast<const uint16_t*>(W2);
  auto dy = static_cast<const uint16_t*>(dY);
  auto hs = const_cast<uint16_t*>(static_cast<const uint16_t*>(Hsave));
  if (!use_narrow(s)) {
    WideArgs a = wide_args(s, offsets, sc);
    a.A = w2; a.B = dy; a.Hsave = hs; a.Hact = w.Hact; a.dHpre = w.dHpre;
    {
      ScopedKernelTimer tm(kSlotDH, st);
      e = launch_wide(kWideDH, s, a, st);
    }
    if (e != hipSuccess) return e;
    a.A = dy; a.B = w.Hact; a.dW = dW2;
    {
      ScopedKernelTimer tm(kSlotDW2, st);
      e = launch_wide(kWideDW, s, a, st);
    }
    if (e != hipSuccess) return e;
    a.A = x; a.B = w.dHpre; a.dW = dW1;
    {
      ScopedKernelTimer tm(kSlotDW1, st);
      e = launch_wide(kWideDW, s, a, st);
    }
    if (e != hipSuccess) return e;
    a.A = w1; a.B = w.dHpre; a.part = w.part;
    {
      ScopedKernelTimer tm(kSlotDXPart, st);
      e = launch_wide(kWidePart, s, a, st);
    }
    if (e != hipSuccess) return e;
    return run_combine(s, w.part, inv, dX, kSlotCombineDX, st);
  }
  {
    ScopedKernelTimer tm(kSlotDH, st);
    e = launch_up<1>(s, w2, dy, offsets, sc, hs, w.Hact, w.dHpre, st);
  }
  if (e != hipSuccess) return e;
  const DwOperands ops[2] = {{dy, w.Hact, dW2, w.dw_stage}, {x, w.dHpre, dW1, w.dw_stage2}};
  const ScatterPlan sp = plan_scatter(s);
  if (joined_backward(s, w, sp)) {
    ScopedKernelTimer tm(kSlotDXDW, st);
    e = launch_scatter_dw(s, sp, w.dHpre, w1, sc, static_cast<uint16_t*>(dX), ops, st);
    return e != hipSuccess ? e : launch_dw_sum(ops, 2, sc, s.N, s.Bs, s.d, st);
  }
  {
    ScopedKernelTimer tm(kSlotDXPart, st);
    e = launch_scatter(s, sp, w.dHpre, w1, sc.rstart, sc.tok, static_cast<uint16_t*>(dX),
                       nullptr, w.split, st);
  }
  if (e != hipSuccess) return e;
  if (w.dw_stage2) return launch_dw_pieces(ops, 2, sc, s.N, s.Bs, s.d, kSlotDW2, st);   // (both under one slot)
  const DwOperands second = {x, w.dHpre, dW1, w.dw_stage};
  e = launch_dw_pieces(ops, 1, sc, s.N, s.Bs, s.d, kSlotDW2, st);
  return e != hipSuccess ? e : launch_dw_pieces(&second, 1, sc, s.N, s.Bs, s.d, kSlotDW1, st);
}

// ------------------------------------------------------------------------------------------
// Low-rank adapted path (section 2.2 on top of section 4.2).
LoraWorkspace plan_lora(const spt_shape_t& s, void* ws, bool backward) {
  const size_t P = (size_t)s.T * s.k, D = (size_t)s.N * s.Bs, T = s.T, d = s.d;
  char* p = static_cast<char*>(ws);
  size_t o = 0;
  LoraWorkspace w = {};
  auto take = [&](size_t bytes) { void* r = p + o; o += align256(bytes); return r; };
  if (backward) { w.bwd = plan_bwd(s, ws, false); o = w.bwd.bytes; }
  else          { w.fwd = plan_fwd(s, ws); o = w.fwd.bytes; }
  w.A1T = static_cast<uint16_t*>(take(32 * d * 2));
  w.C1T = static_cast<uint16_t*>(take(D * 64 * 2));
  w.C1P = static_cast<uint16_t*>(take(32 * D * 2));
  w.B2T = static_cast<uint16_t*>(take(32 * D * 2));
  w.B2P = static_cast<uint16_t*>(take(D * 64 * 2));
  w.C2P = static_cast<uint16_t*>(take(32 * d * 2));
  w.A1P = static_cast<uint16_t*>(take(d * 32 * 2));
  w.C2T = static_cast<uint16_t*>(take(d * 32 * 2));
  w.Z = use_narrow(s) ? static_cast<uint16_t*>(take(T * d * 2)) : nullptr;
  w.Upad = static_cast<uint16_t*>(take(T * 64 * 2));
  w.Sp = static_cast<float*>(take(P * 32 * 4));
  if (backward) {
    w.Gpad = static_cast<uint16_t*>(take(T * 64 * 2));
    w.Upair = static_cast<uint16_t*>(take(P * 64 * 2));
    w.Gpair = static_cast<uint16_t*>(take(P * 64 * 2));
    w.Rb = static_cast<uint16_t*>(take(T * 32 * 2));
    w.Vb = static_cast<uint16_t*>(take(T * 32 * 2));
    w.Sp2 = static_cast<float*>(take(P * 32 * 4));
    w.piece = grad_piece_rows((int64_t)P, s.N, s.Bs);
    w.max_pieces = (int)(P / w.piece) + s.N;
    w.chunk = grad_piece_rows((int64_t)T, 1, s.d);
    w.nchunks = (int)((T + w.chunk - 1) / w.chunk);
    w.stage[0] = static_cast<float*>(take((size_t)w.max_pieces * s.Bs * 32 * 4));
    w.stage[1] = static_cast<float*>(take((size_t)w.max_pieces * s.Bs * 32 * 4));
    w.stage[2] = static_cast<float*>(take((size_t)w.nchunks * d * 32 * 4));
    w.stage[3] = static_cast<float*>(take((size_t)w.nchunks * d * 32 * 4));
    w.p_first = static_cast<int32_t*>(take((size_t)(s.N + 1) * 4));
    w.p_off = static_cast<int32_t*>(take((size_t)(w.max_pieces + 1) * 4));
  }
  w.bytes = o;
  return w;
}

hipError_t run_lora_fwd(const spt_shape_t& s, int r, const void* X, const void* W1, const void* W2,
                        const void* A1, const void* C1, const void* B2, const void* C2,
                        const int32_t* offsets, const int32_t* perm, const int32_t* inv, void* Y,
                        void* Hsave, const LoraWorkspace& w, hipStream_t st) {
  const int D = s.N * s.Bs, P = s.T * s.k;
  auto x = static_cast<const uint16_t*>(X);
  auto hs = static_cast<uint16_t*>(Hsave);
  hipError_t e = run_plan(s, offsets, perm, w.fwd.sched, st);
  if (e != hipSuccess) return e;
  {
    ScopedKernelTimer tm(kSlotLoraSmall, st);
    const uint16_t *a1 = static_cast<const uint16_t*>(A1), *c1 = static_cast<const uint16_t*>(C1);
    const uint16_t *b2 = static_cast<const uint16_t*>(B2), *c2 = static_cast<const uint16_t*>(C2);
    PadJobs jobs = {};
    jobs.job[0] = PadJob{a1, s.d, r, 1, 0, 1, w.A1T, 32, s.d};   // A1^T      [32][d]
    jobs.job[1] = PadJob{c1, r, D, 1, 1, 0, w.C1T, D, 64};       // C1^T twice [D][64]
    jobs.job[2] = PadJob{b2, D, r, 1, 0, 1, w.B2T, 32, D};       // B2^T      [32][D]
    jobs.job[3] = PadJob{c2, r, s.d, 1, 0, 0, w.C2T, s.d, 32};   // C2^T      [d][32]
    if ((e = lora_setup(jobs, 4, nullptr, st)) != hipSuccess) return e;
    const ProjJob proj = {x, w.A1T, w.Upad, nullptr};             // U = X A1
    if ((e = lora_proj(&proj, 1, inv, s.T, s.d, s.k, st)) != hipSuccess) return e;
  }
  const bool narrow = use_narrow(s);
  if (narrow) {
    ScopedKernelTimer tm(kSlotUp, st);
    e = launch_up<0>(s, static_cast<const uint16_t*>(W1), x, offsets, w.fwd.sched, hs, w.fwd.Hact, nullptr, st,
                     w.Upad, w.C1T);
    if (e != hipSuccess) return e;
  } else {
    WideArgs a = wide_args(s, offsets, w.fwd.sched);
    a.A = W1; a.B = x; a.Hsave = hs; a.Hact = w.fwd.Hact; a.Xe = w.Upad; a.We = w.C1T;
    {
      ScopedKernelTimer tm(kSlotUp, st);
      e = launch_wide(kWideUp, s, a, st);
    }
    if (e != hipSuccess) return e;
    a.A = W2; a.B = w.fwd.Hact; a.part = w.fwd.part; a.Xe = nullptr; a.We = nullptr;
    {
      ScopedKernelTimer tm(kSlotDown, st);
      e = launch_wide(kWidePart, s, a, st);
    }
    if (e != hipSuccess) return e;
  }
  // V[t] = sum_b B2_b^T h_b(t); the write-back adds V C2 per token
  {
    ScopedKernelTimer tm(kSlotLoraSmall, st);
    const PairJob pair = {w.fwd.Hact, w.B2T, w.Sp};
    if ((e = lora_pair_gemm(&pair, 1, narrow, offsets, s.N, s.Bs, P, st)) != hipSuccess) return e;
    if (narrow) e = lora_expand(w.Sp, w.C2T, inv, s.T, s.d, s.k, nullptr, w.Z, nullptr, nullptr, nullptr, st);
    if (e != hipSuccess) return e;
  }
  if (!narrow) {
    ScopedKernelTimer tm(kSlotCombineY, st);
    return lora_expand(w.Sp, w.C2T, inv, s.T, s.d, s.k, w.fwd.part, static_cast<uint16_t*>(Y), nullptr, nullptr, nullptr, st);
  }
  ScopedKernelTimer tm(kSlotDown, st);
  return launch_scatter(s, plan_scatter(s), w.fwd.Hact, static_cast<const uint16_t*>(W2), w.fwd.sched.rstart,
                        w.fwd.sched.tok, static_cast<uint16_t*>(Y), w.Z, w.fwd.split, st);
}

hipError_t run_lora_bwd(const spt_shape_t& s, int r, const void* X, const void* W1, const void* W2,
                        const void* A1, const void* C1, const void* B2, const void* C2, const void* dY,
                        const int32_t* offsets, const int32_t* perm, const int32_t* inv,
                        const void* Hsave, void* dX, float* dA1, float* dC1, float* dB2, float* dC2,
                        const LoraWorkspace& w, hipStream_t st) {
  const int D = s.N * s.Bs, P = s.T * s.k;
  auto x = static_cast<const uint16_t*>(X);
  auto dy = static_cast<const uint16_t*>(dY);
  auto hs = const_cast<uint16_t*>(static_cast<const uint16_t*>(Hsave));
  const Schedule& sc = w.bwd.sched;
  hipError_t e = run_plan(s, offsets, perm, sc, st);
  if (e != hipSuccess) return e;
  {
    ScopedKernelTimer tm(kSlotLoraSmall, st);
    const uint16_t *a1 = static_cast<const uint16_t*>(A1), *c1 = static_cast<const uint16_t*>(C1);
    const uint16_t *b2 = static_cast<const uint16_t*>(B2), *c2 = static_cast<const uint16_t*>(C2);
    PadJobs jobs = {};
    jobs.job[0] = PadJob{a1, s.d, r, 1, 0, 1, w.A1T, 32, s.d};   // A1^T       [32][d]
    jobs.job[1] = PadJob{a1, s.d, r, 0, 0, 0, w.A1P, s.d, 32};   // A1         [d][32]
    jobs.job[2] = PadJob{c1, r, D, 0, 0, 1, w.C1P, 32, D};       // C1         [32][D]
    jobs.job[3] = PadJob{b2, D, r, 1, 0, 1, w.B2T, 32, D};       // B2^T       [32][D]
    jobs.job[4] = PadJob{b2, D, r, 0, 1, 0, w.B2P, D, 64};       // B2 twice   [D][64]
    jobs.job[5] = PadJob{c2, r, s.d, 0, 0, 1, w.C2P, 32, s.d};   // C2         [32][d]
    const PieceTable pieces = {offsets, s.N, w.piece, w.max_pieces, w.p_first, w.p_off};
    if ((e = lora_setup(jobs, 6, &pieces, st)) != hipSuccess) return e;
    const ProjJob proj[2] = {{x, w.A1T, nullptr, w.Upair},        // U = X A1
                             {dy, w.C2P, w.Gpad, w.Gpair}};       // G = dY C2^T
    if ((e = lora_proj(proj, 2, inv, s.T, s.d, s.k, st)) != hipSuccess) return e;
  }
  const bool narrow = use_narrow(s);
  if (narrow) {
    // dH = dY W2_b^T + G B2_b^T; dHpre and Hact go to the workspace
    ScopedKernelTimer tm(kSlotDH, st);
    e = launch_up<1>(s, static_cast<const uint16_t*>(W2), dy, offsets, sc, hs, w.bwd.Hact, w.bwd.dHpre, st,
                     w.Gpad, w.B2P);
    if (e != hipSuccess) return e;
  } else {
    WideArgs a = wide_args(s, offsets, sc);
    a.A = W2; a.B = dy; a.Hsave = hs; a.Hact = w.bwd.Hact; a.dHpre = w.bwd.dHpre; a.Xe = w.Gpad; a.We = w.B2P;
    {
      ScopedKernelTimer tm(kSlotDH, st);
      e = launch_wide(kWideDH, s, a, st);
    }
    if (e != hipSuccess) return e;
    a.A = W1; a.B = w.bwd.dHpre; a.part = w.bwd.part; a.Xe = nullptr; a.We = nullptr;
    {
      ScopedKernelTimer tm(kSlotDXPart, st);
      e = launch_wide(kWidePart, s, a, st);
    }
    if (e != hipSuccess) return e;
  }
  // R[t] = sum_b C1_b dhpre_b(t), V[t] = sum_b B2_b^T h_b(t);  dX = sum_b dhpre_b W1_b + R A1^T
  {
    ScopedKernelTimer tm(kSlotLoraSmall, st);
    const PairJob pair[2] = {{w.bwd.dHpre, w.C1P, w.Sp}, {w.bwd.Hact, w.B2T, w.Sp2}};
    if ((e = lora_pair_gemm(pair, 2, narrow, offsets, s.N, s.Bs, P, st)) != hipSuccess) return e;
    if (narrow) e = lora_expand(w.Sp, w.A1P, inv, s.T, s.d, s.k, nullptr, w.Z, w.Rb, w.Sp2, w.Vb, st);
    if (e != hipSuccess) return e;
  }
  if (narrow) {
    ScopedKernelTimer tm(kSlotDXPart, st);
    e = launch_scatter(s, plan_scatter(s), w.bwd.dHpre, static_cast<const uint16_t*>(W1), sc.rstart, sc.tok,
                       static_cast<uint16_t*>(dX), w.Z, w.bwd.split, st);
  } else {
    ScopedKernelTimer tm(kSlotCombineDX, st);
    e = lora_expand(w.Sp, w.A1P, inv, s.T, s.d, s.k, w.bwd.part, static_cast<uint16_t*>(dX), w.Rb, w.Sp2, w.Vb, st);
  }
  if (e != hipSuccess) return e;
  // dC1[rho][unit] = sum_{q in b} U[tok q][rho] dHpre[q][u],  dB2[unit][rho] = sum_{q in b} Hact[q][u] G[tok q][rho]
  // (U and G as their two bf16 parts, the two products added),  dA1[i][rho] = sum_t X[t][i] R[t][rho],
  // dC2[rho][c] = sum_t V[t][rho] dY[t][c]: per piece of the rows, then the pieces in order
  const int ut = (s.Bs + 127) / 128, dt = (s.d + 127) / 128;
  const GradJobs jobs = {{
      {w.bwd.dHpre, w.Upair, w.stage[0], w.p_off, w.p_first, dC1, s.Bs, 64, 32, w.max_pieces, ut, w.piece, P, s.N, 1},
      {w.bwd.Hact, w.Gpair, w.stage[1], w.p_off, w.p_first, dB2, s.Bs, 64, 32, w.max_pieces, ut, w.piece, P, s.N, 0},
      {x, w.Rb, w.stage[2], nullptr, nullptr, dA1, s.d, 32, 32, w.nchunks, dt, w.chunk, s.T, 1, 0},
      {dy, w.Vb, w.stage[3], nullptr, nullptr, dC2, s.d, 32, 32, w.nchunks, dt, w.chunk, s.T, 1, 1}}};
  ScopedKernelTimer tm(kSlotLoraGrad, st);
  return lora_grads(jobs, narrow, r, sc.zero_row, st);
}

}  // namespace spt

// For tests, not declared in the header: whether a backward pass of the shape has dX and both weight gradients in one launch.
extern "C" int spt_internal_joined_backward(const spt_shape_t* s) {
  using namespace spt;
  return s && use_narrow(*s) && joined_backward(*s, plan_bwd(*s, nullptr, true), plan_scatter(*s));
}
