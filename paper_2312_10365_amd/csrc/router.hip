// Route network + block selection (paper section 4.2, "Dynamic routing").
//
// logit[t][b] = sum_i X[t][i] * W_r[i][b] (+ b_r[b]) accumulated in fp64 and rounded once to
// fp32.  Products of a bf16 and an fp32 value are exact in fp64, so only the order of the
// additions can move the fp64 sum, by parts in 1e-16 -- far below the fp32 rounding step.
// The k largest keys win; equal keys go to the lower block id; ids are emitted ascending.
//
// Many tokens without the caller's logits: the ids come from bf16 products and fp32 sums, from fp64 ones where those
// leave a doubt (router_near_kernel, topk_near_kernel).  Otherwise:
// Kernel 1 (logits): fp64 matrix cores, v_mfma_f64_16x16x4_f64.  A workgroup owns 16 MT tokens x 16 NT
// blocks and its KS wavefronts split d; their sums are added through LDS in wavefront order.
// Operands go straight from global memory to registers: a lane reads 8
// consecutive bf16 of one token row and the matching 8 rows of one W_r column, widens them to
// fp64, and feeds 8 MFMAs; which real k sits in which MFMA k-slot is the same for both
// operands, which is all a contraction needs.
// Kernel 2 (top-k): one wavefront per token; the k-th largest key is found by a 32-step radix
// search on the order-preserving integer image of the fp32 keys, the keys above it are selected,
// ties at it go to the lowest block ids: block b is selected iff fewer than k blocks b' have
// key[b'] > key[b] or (key[b'] == key[b] and b' < b).  With at most 32 blocks one workgroup holds all
// logits of its tokens and selects in the same launch.
#include "ffn_common.hpp"
#include "spt_host.hpp"
#include "profile.hpp"

namespace spt {

typedef double f64x4 __attribute__((ext_vector_type(4)));

// Top-k of one token by one wavefront, NPL keys per lane (block b = lane + 64 n, logit[n]; lanes past N
// ignored).  The k-th largest key is found by a radix search on the order-preserving integer image of
// the fp32 keys (32 steps of compare + ballot + popcount: the largest T with at least k keys >= T);
// every key above it is selected, and of the keys equal to it the lowest block ids, as many as are
// still missing.  Ids are emitted ascending.
__device__ __forceinline__ uint32_t key_image(float logit, int flags) {   // larger key <=> larger image, never 0
  const float key = ((flags & 1) ? fabsf(logit) : logit) + 0.0f;           // -0 -> +0: equal keys, equal images
  const uint32_t bits = __float_as_uint(key);
  const uint32_t u = (bits & 0x80000000u) ? ~bits : (bits | 0x80000000u);
  return u ? u : 1u;                       // (only a NaN with all mantissa bits set maps to 0)
}
// The k-th largest of the images u (block lane + 64 n; 0, below every real one, past the last block).
template <int NPL>
__device__ __forceinline__ uint32_t kth_image(const uint32_t (&u)[NPL], int k) {
  uint32_t thr = 0u;
#pragma unroll 1
  for (int bit = 31; bit >= 0; --bit) {
    const uint32_t cand = thr | (1u << bit);
    int c = 0;
#pragma unroll
    for (int n = 0; n < NPL; ++n) c += __popcll(__ballot(u[n] >= cand));
    if (c >= k) thr = cand;                // uniform
  }
  return thr;
}
template <int NPL>
__device__ __forceinline__ void emit_topk(const uint32_t (&u)[NPL], uint32_t thr, int lane, int k,
                                          int32_t* __restrict__ out) {
  int above = 0;
#pragma unroll
  for (int n = 0; n < NPL; ++n) above += __popcll(__ballot(u[n] > thr));
  int need = k - above;                    // keys equal to the threshold still to take, lowest ids first
  int base = 0;
#pragma unroll
  for (int n = 0; n < NPL; ++n) {
    const unsigned long long below = (1ull << lane) - 1ull;
    const unsigned long long eq = __ballot(u[n] == thr);
    const bool sel = (u[n] > thr) || (u[n] == thr && __popcll(eq & below) < need);
    need -= min(need, (int)__popcll(eq));
    const unsigned long long m = __ballot(sel);
    const int pos = base + __popcll(m & below);
    if (sel) out[pos] = lane + 64 * n;
    base += __popcll(m);
  }
}

// One wavefront holds 16 MT tokens x 16 NT blocks of fp64 accumulators; the wavefronts share
// the 32-wide chunks of d evenly, with those of other workgroups (gridDim.z) when `partial` is given: then
// the fp64 sums go there and the top-k kernel adds them.  Operands are loaded DEPTH - 1 chunks ahead of the
// MFMAs that consume them.  `TOPK`: the workgroup's tile covers all blocks (N <= 16 NT) and the block
// ids are selected here too.
template <int MT, int NT, int KS, int DEPTH, bool TOPK>
__global__ __launch_bounds__(64 * KS) void router_logits_kernel(
    const uint16_t* __restrict__ X, const float* __restrict__ Wr, const float* __restrict__ br, int T, int d, int N,
    float* __restrict__ logits, double* __restrict__ partial, int k, int flags, int32_t* __restrict__ idx) {
  constexpr int TOK = 16 * MT, BLK = 16 * NT;
  __shared__ double red[KS > 1 ? KS / 2 : 1][MT * NT * 4][64];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, slot = lane >> 4;
  const int tok0 = blockIdx.x * TOK, blk0 = blockIdx.y * BLK;

  const uint16_t* xrow[MT];
  const float* wcol[NT];
#pragma unroll
  for (int m = 0; m < MT; ++m)
    xrow[m] = X + (size_t)min(tok0 + 16 * m + r16, T - 1) * d + 8 * slot;  // clamped rows are computed but never stored
#pragma unroll
  for (int n = 0; n < NT; ++n)
    wcol[n] = Wr + (size_t)(8 * slot) * N + min(blk0 + 16 * n + r16, N - 1);  // ... columns likewise
  f64x4 acc[MT][NT];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int n = 0; n < NT; ++n) acc[m][n] = f64x4{0.0, 0.0, 0.0, 0.0};

  uint4 xq[DEPTH][MT];
  float wq[DEPTH][NT][8];
  auto fetch = [&](int st, int c) {
    const int k0 = c * 32;
#pragma unroll
    for (int m = 0; m < MT; ++m) xq[st][m] = *reinterpret_cast<const uint4*>(xrow[m] + k0);
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
      for (int e = 0; e < 8; ++e) wq[st][n][e] = wcol[n][(size_t)(k0 + e) * N];
  };
  auto consume = [&](int st) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      double a[MT], b[NT];
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        const uint32_t w32 = reinterpret_cast<const uint32_t*>(&xq[st][m])[e >> 1];
        a[m] = (double)((e & 1) ? hi_bf16(w32) : lo_bf16(w32));
      }
#pragma unroll
      for (int n = 0; n < NT; ++n) b[n] = (double)wq[st][n][e];
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int n = 0; n < NT; ++n)
          acc[m][n] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[m], b[n], acc[m][n], 0, 0, 0);
    }
  };
  const int chunks = d / 32, parts = KS * gridDim.z, pw = blockIdx.z * KS + wave;
  const int cbeg = pw * chunks / parts, cend = (pw + 1) * chunks / parts;
  if (cbeg < cend) {
    const int clast = cend - 1;  // (requests past the last chunk repeat it: no branch around a load)
#pragma unroll
    for (int s = 0; s < DEPTH - 1; ++s) fetch(s, min(cbeg + s, clast));
    int c = cbeg;
    for (; c + DEPTH <= cend; c += DEPTH) {  // DEPTH chunks per trip keep the ring slots static
#pragma unroll
      for (int s = 0; s < DEPTH; ++s) {
        fetch((s + DEPTH - 1) % DEPTH, min(c + s + DEPTH - 1, clast));
        consume(s);
      }
    }
#pragma unroll
    for (int s = 0; s < DEPTH - 1; ++s)
      if (c + s < cend) consume(s);
  }

  // The upper half of the wavefronts hands its sums to the lower half, and so on: a fixed order.
#pragma unroll
  for (int half = KS / 2; half >= 1; half >>= 1) {
    if (wave >= half && wave < 2 * half) {
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int n = 0; n < NT; ++n)
#pragma unroll
          for (int v = 0; v < 4; ++v) red[wave - half][(m * NT + n) * 4 + v][lane] = acc[m][n][v];
    }
    __syncthreads();
    if (wave < half) {
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int n = 0; n < NT; ++n)
#pragma unroll
          for (int v = 0; v < 4; ++v) acc[m][n][v] += red[wave][(m * NT + n) * 4 + v][lane];
    }
    __syncthreads();
  }

  // D layout of the 16x16 fp64 tile: lane holds column (lane & 15), rows 4*v + (lane >> 4).
  uint32_t* keys = reinterpret_cast<uint32_t*>(&red[0][0][0]);  // [TOK][BLK] key images
  if (wave == 0) {
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int n = 0; n < NT; ++n) {
        const int b = blk0 + 16 * n + r16;
        const double bias = (br && b < N) ? (double)br[b] : 0.0;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int row = 16 * m + 4 * v + slot;
          const double sum = acc[m][n][v] + bias;
          if (TOPK) keys[row * BLK + 16 * n + r16] = b < N ? key_image((float)sum, flags) : 0u;
          if (b < N && tok0 + row < T) {
            const size_t at = (size_t)(tok0 + row) * N + b;
            if (partial) partial[(size_t)blockIdx.z * T * N + at] = acc[m][n][v];
            else if (logits) logits[at] = (float)sum;
          }
        }
      }
  }
  if (TOPK) {
    // A block's rank = blocks with a larger key, or an equal one and a lower id.  BLK lanes per token,
    // 64 / BLK tokens per wavefront at a time.
    __syncthreads();
    const int b = lane % BLK;
    for (int row0 = wave * (64 / BLK); row0 < TOK; row0 += KS * (64 / BLK)) {
      const int row = row0 + lane / BLK, t = tok0 + row;
      const uint32_t mine = keys[row * BLK + b];
      int rank = 0;
#pragma unroll
      for (int o = 0; o < BLK; o += 4) {
        const uint4 q = *reinterpret_cast<const uint4*>(keys + row * BLK + o);
        rank += (q.x > mine) || (q.x == mine && o < b);
        rank += (q.y > mine) || (q.y == mine && o + 1 < b);
        rank += (q.z > mine) || (q.z == mine && o + 2 < b);
        rank += (q.w > mine) || (q.w == mine && o + 3 < b);
      }
      const bool sel = rank < k;
      const unsigned long long m = __ballot(sel);
      const uint32_t group = (uint32_t)(m >> (lane - b)) & (BLK == 32 ? 0xFFFFFFFFu : (1u << (BLK & 31)) - 1u);
      if (sel && t < T) idx[(size_t)t * k + __popc(group & ((1u << b) - 1u))] = b;
    }
  }
}

// (Rank-by-counting, the first version, compared every key with every other: 1400 instructions per token
// at N = 128 against about 250.)
template <int NPL>
__global__ __launch_bounds__(256) void topk_kernel(const float* __restrict__ logits,
                                                   const double* __restrict__ partial, const float* __restrict__ br,
                                                   int splits, int T, int N, int k, int flags,
                                                   int32_t* __restrict__ idx) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int t = blockIdx.x * 4 + wave;
  if (t >= T) return;                      // whole wavefront; the kernel has no barrier
  float l[NPL];
#pragma unroll
  for (int n = 0; n < NPL; ++n) {
    const int b = lane + 64 * n;
    l[n] = 0.f;
    if (b < N) {
      if (partial) {   // the parts of d, in order
        double sum = 0.0;
        for (int z0 = 0; z0 < splits; z0 += 8) {   // eight loads in flight
          double p[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) p[u] = z0 + u < splits ? partial[((size_t)(z0 + u) * T + t) * N + b] : 0.0;
#pragma unroll
          for (int u = 0; u < 8; ++u) sum += p[u];
        }
        l[n] = (float)(sum + (br ? (double)br[b] : 0.0));
      } else {
        l[n] = logits[(size_t)t * N + b];
      }
    }
  }
  uint32_t u[NPL];
#pragma unroll
  for (int n = 0; n < NPL; ++n) u[n] = lane + 64 * n < N ? key_image(l[n], flags) : 0u;
  emit_topk<NPL>(u, kth_image<NPL>(u, k), lane, k, idx + (size_t)t * k);
}

// Many tokens, 33 to 128 blocks, only the ids wanted: the order of a token's logits rarely hangs on their last bits.  Sums
// good to a few parts in 10^6 of |x| |w_b| settle it for 97 to 99 % of the tokens; for the rest the blocks around
// the k-th are summed again, in fp64 as above (topk_near_kernel).  The ids are those of the fp64 logits.
//
// router_near_kernel: bf16 matrix cores at 29 times the fp64 rate.  X is bf16, W_r is split into three bf16 whose sum it is, so
// the products are exact and the sums are fp32: over one stage of the d axis in the MFMA chain, the stages added outside
// of it.  A workgroup has 128 tokens, all blocks and a part of d (gridDim = tiles x parts); its wavefronts are CTW column tiles of
// 32 blocks x KP interleaved shares of the K-steps, so each value of W_r is loaded and split once per workgroup.  Stages
// of 128 columns of X go through LDS, requested a stage ahead, as is W_r.
// What a sum can be off by: every MFMA by two units in the last place of the magnitudes so far (a bound on its inner
// additions, in whatever order), every fp32 addition by half a unit; sum |x w| <= |x| |w| over the part (x and w with
// the squares that underflow added: `tiny`); exactly 0 where the tokens or the weights are zeros.  `reach` holds it per token
// and part, with the largest |w| of the blocks.  Measured over d 64 to 8192: at most 0.014 of it, 0.0025 at d = 4096.
//
// us, both launches, fp64 -> this: T 8192, d 4096, N 128 151 -> 54; T 3001 65 -> 38; T 16384, d 1024, N 64 50 -> 34.  The fp64
// units were busy 70 % of the time; here no unit is (T 3001: MFMA 23 %, vector units 39 % of the cycles): a workgroup's first
// loads, its last sums and three to eight stages one after the other.  Registers (235) hold it at one workgroup per CU: the
// next step's split among the MFMAs spilled and took 50 us where 38 is, a fixed stage without branches 45.
constexpr int kNearTokens = 128, kNearWaves = 8, kNearStage = 8;   // tokens; wavefronts; K-steps of 16 of a stage
template <int CTW>
__global__ __launch_bounds__(64 * kNearWaves, 2) void router_near_kernel(
    const uint16_t* __restrict__ X, const float* __restrict__ Wr, int T, int d, int N, int splits, float tie,
    float* __restrict__ near, float* __restrict__ reach, float* __restrict__ Wt) {
  constexpr int MT = kNearTokens / 32, KP = kNearWaves / CTW, JS = kNearStage / KP, NTH = 64 * kNearWaves;
  __shared__ uint4 smem[2 * kNearTokens * 16];             // two stages: rows of 128 columns, 16-byte pieces permuted by row
  const int tid = threadIdx.x, lane = tid & 63, i = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), ct = wave % CTW, kp = wave / CTW;
  const int z = blockIdx.x % splits, tile = blockIdx.x / splits, tiles = gridDim.x / splits, tok0 = tile * kNearTokens;
  const int units = (d + 63) / 64;                         // (parts begin at whole cache lines of a token)
  const int sbeg = 4 * (int)((int64_t)z * units / splits), send = min(4 * (int)((int64_t)(z + 1) * units / splits), d / 16);
  const bool active = ct * 32 < N;
  const int share = min(tiles, send - sbeg);

  // pieces of a stage: row tid / 16 + 32 u, piece tid % 16
  const int prow = tid >> 4, pcol = tid & 15;
  const uint16_t* xbase = X + (size_t)tok0 * d;            // (one base for the workgroup, 32-bit offsets)
  uint32_t xrow[MT];
#pragma unroll
  for (int u = 0; u < MT; ++u) xrow[u] = (uint32_t)min(prow + 32 * u, T - 1 - tok0) * (uint32_t)d;
  u32x4 xn[MT];
  float x2[MT] = {};
  uint32_t xany[MT] = {};
  auto request_x = [&](int s) {
    const int c = min((sbeg + s * kNearStage) * 16 + pcol * 8, d - 8);   // (past the end: a piece nobody multiplies)
#pragma unroll
    for (int u = 0; u < MT; ++u) xn[u] = *reinterpret_cast<const u32x4*>(xbase + (xrow[u] + c));
  };
  auto store_x = [&](int buf) {
#pragma unroll
    for (int u = 0; u < MT; ++u) {
      const int r = prow + 32 * u;
      *reinterpret_cast<u32x4*>(smem + buf * (kNearTokens * 16) + r * 16 + (pcol ^ (r & 15))) = xn[u];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bf16x2 v = __builtin_bit_cast(bf16x2, (uint32_t)xn[u][e]);
        x2[u] = __builtin_amdgcn_fdot2_f32_bf16(v, v, x2[u], false);
        xany[u] |= xn[u][e];
      }
    }
  };
  const uint32_t wcol = 8 * h * N + min(ct * 32 + i, N - 1);
  float wq[JS][8], w2 = 0.f;
  uint32_t wany = 0u;
  auto request_w = [&](int j, int step) {
    const float* p = Wr + (size_t)min(step, send - 1) * 16 * N;
#pragma unroll
    for (int e = 0; e < 8; ++e) wq[j][e] = (p + (size_t)e * N)[wcol];
  };

  f32x16 sum[MT];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int v = 0; v < 16; ++v) sum[m][v] = 0.f;
  request_x(0);
#pragma unroll
  for (int j = 0; j < JS; ++j) request_w(j, sbeg + kp + KP * j);
  store_x(0);
  __syncthreads();
  const int stages = (send - sbeg + kNearStage - 1) / kNearStage;
  for (int s = 0; s < stages; ++s) {
    const bool more = s + 1 < stages;                      // uniform
    if (more) request_x(s + 1);
    const int s0 = sbeg + s * kNearStage + kp;
    if (active && s0 < send) {                             // uniform over the wavefront
      const uint4* rows = smem + (s & 1) * (kNearTokens * 16);
      f32x16 acc[MT];
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[m][v] = 0.f;
#pragma unroll
      for (int j = 0; j < JS; ++j) {
        const int step = s0 + KP * j;
        if (step >= send) break;                           // uniform
        bf16x8 part[3], xf[MT];
        u32x4 wa, wb;
#pragma unroll
        for (int e = 0; e < 4; ++e) { wa[e] = __float_as_uint(wq[j][e]); wb[e] = __float_as_uint(wq[j][e + 4]); }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          w2 = fmaf(wq[j][e], wq[j][e], w2);
          wany |= __float_as_uint(wq[j][e]);
        }
        // (the copy of W_r with the blocks as rows, by each tile of tokens a share of it)
        if ((step - sbeg) % share == tile && ct * 32 + i < N) {
          u32x4* to = reinterpret_cast<u32x4*>(Wt + (size_t)(ct * 32 + i) * d + step * 16 + 8 * h);
          to[0] = wa;
          to[1] = wb;
        }
        split_bf16x3(wa, wb, part[0], part[1], part[2]);
        request_w(j, step + kNearStage);
#pragma unroll
        for (int m = 0; m < MT; ++m) {
          const int r = 32 * m + i;
          xf[m] = __builtin_bit_cast(bf16x8, rows[r * 16 + ((2 * (kp + KP * j) + h) ^ (r & 15))]);
        }
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
          for (int m = 0; m < MT; ++m)
            acc[m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xf[m], part[c], acc[m], 0, 0, 0);
      }
#pragma unroll
      for (int m = 0; m < MT; ++m) sum[m] += acc[m];
    }
    if (more) store_x((s + 1) & 1);
    __syncthreads();
  }

  // How far a token's sums over this part of d can be off (see above).
  float* xnorm = reinterpret_cast<float*>(smem);           // [128] of the tokens
  float* wnorm = xnorm + kNearTokens;                      // [KP][32 CTW] of the blocks
  uint32_t* wmax = reinterpret_cast<uint32_t*>(wnorm + KP * 32 * CTW);
  const float tiny = (float)d * 0x1p-100f;
#pragma unroll
  for (int u = 0; u < MT; ++u) {
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) {
      x2[u] += __shfl_xor(x2[u], o);
      xany[u] |= (uint32_t)__shfl_xor((int)xany[u], o);
    }
    if (pcol == 0) xnorm[prow + 32 * u] = xany[u] & 0x7FFF7FFFu ? x2[u] + tiny : 0.f;
  }
  w2 += __shfl_xor(w2, 32);
  wany |= (uint32_t)__shfl_xor((int)wany, 32);
  if (h == 0) wnorm[kp * (32 * CTW) + ct * 32 + i] = wany << 1 ? w2 + tiny : 0.f;
  __syncthreads();
  if (tid < 32 * CTW) {
    float v = 0.f;
#pragma unroll
    for (int q = 0; q < KP; ++q) v += wnorm[q * (32 * CTW) + tid];
    int bits = __float_as_int(v) & 0x7FFFFFFF;             // (as whole numbers: a NaN is the largest)
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) bits = max(bits, __shfl_xor(bits, o));
    if (lane == 0) wmax[wave] = (uint32_t)bits;
  }
  __syncthreads();
  if (tid < kNearTokens && tok0 + tid < T) {
    uint32_t bits = wmax[0];
    if (CTW > 2) bits = max(bits, wmax[1]);
    reach[(size_t)z * T + tok0 + tid] = tie * sqrtf(xnorm[tid]) * sqrtf(__uint_as_float(bits));
  }

  // The wavefronts of a column tile add their sums up in pairs, each keeping half of the token tiles: a fixed order.
  f32x4* red = reinterpret_cast<f32x4*>(smem);             // [wavefront][8][64], then [4]
  int mine = 0;                                            // the first token tile kept
#pragma unroll
  for (int half = KP / 2, cnt = MT / 2; half >= 1; half >>= 1, cnt >>= 1) {
    if (kp & half) {                                       // uniform: what is kept comes first
      mine += cnt;
#pragma unroll
      for (int m = 0; m < cnt; ++m) {
        const f32x16 x = sum[m];
        sum[m] = sum[m + cnt];
        sum[m + cnt] = x;
      }
    }
    __syncthreads();
#pragma unroll
    for (int m = 0; m < cnt; ++m)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        red[(wave * 8 + m * 4 + v) * 64 + lane] =
            f32x4{sum[m + cnt][4 * v], sum[m + cnt][4 * v + 1], sum[m + cnt][4 * v + 2], sum[m + cnt][4 * v + 3]};
    __syncthreads();
    const f32x4* from = red + (size_t)((kp ^ half) * CTW + ct) * (8 * 64) + lane;
#pragma unroll
    for (int m = 0; m < cnt; ++m)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const f32x4 x = from[(m * 4 + v) * 64];
#pragma unroll
        for (int e = 0; e < 4; ++e) sum[m][4 * v + e] += x[e];
      }
  }
  // (accumulator: column = block, rows v % 4 + 8 (v / 4) + 4 h = tokens)
  const int b = ct * 32 + i;
  if (b < N) {
    float* out = near + ((size_t)z * T + tok0) * N + b;
#pragma unroll
    for (int m = 0; m < MT / KP; ++m)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int t = 32 * (mine + m) + (v & 3) + 8 * (v >> 2) + 4 * h;
        if (tok0 + t < T) out[t * N] = sum[m][v];
      }
  }
}

// Selection from those sums, a wavefront per token.  kth - after, the distance between the k-th key and the one after, beyond
// what both can be off by (twice `reach` and the rounding to fp32): the k largest are the right ones.  Otherwise every key
// more than that above `after` is in, every key more than that below kth is out, and those between are summed in fp64 (x times a
// row of the copy of W_r that the kernel above leaves: its columns are a cache line per value) and compete for the places
// left.  Sums that are not finite leave all blocks open.
// How many are open hangs on the data (weights with a large part common to all blocks, blocks alike, tokens that are
// not finite: all of them), so the 16 tokens of a workgroup share that work.  Up to kNearTurns turns of two blocks are dealt to the
// wavefronts whatever token they are of; beyond that the fp64 matrix cores sum all blocks of the 16 tokens, which costs the
// same for any data.  The line lies where the two meet: T 8192, d 4096, N 128 with a common part of 300 times what tells the
// blocks apart (14 open a token) 136 us dealt, 222 summed; with half the turns it would go to the second.
// us, both launches, a wavefront per token with all its open blocks -> this: T 8192, d 4096, N 128: ordinary weights 57 -> 58,
// common part x 30 67 -> 65, x 1000 345 -> 222, all alike 850 -> 222 (fp64 throughout: 150), one token of NaN 204 -> 75; T 3001
// 37 -> 38, 290 -> 121 (65); T 16384, d 1024, N 64 32 -> 34, 210 -> 74 (50); T 40000, d 256, N 128 67 -> 70, 750 -> 137 (100).
// Workgroups of 16 wavefronts wait for 16 places, which is what ordinary weights pay: at most 64 registers, so that a CU has two
// (with 72 and one: 63, 40 and 92 us).
constexpr int kOpenTokens = 16, kNearTurns = 8 * kOpenTokens;
template <int NPL>
__global__ __launch_bounds__(64 * kOpenTokens, 8) void topk_near_kernel(
    const float* __restrict__ near, const float* __restrict__ reach, const float* __restrict__ Wt,
    const uint16_t* __restrict__ X, const float* __restrict__ br, int splits, int T, int d, int N, int k, int flags,
    int32_t* __restrict__ idx) {
  constexpr int CT = 4 * NPL, KP = kOpenTokens / CT;       // column tiles of 16 blocks, shares of d (matrix cores)
  __shared__ uint8_t list[kOpenTokens][64 * NPL];          // the open blocks of a token
  __shared__ int turns[kOpenTokens];
  __shared__ uint32_t keys[kOpenTokens][64 * NPL];         // images of their fp64 logits
  __shared__ double red[KP - 1][CT][4][64];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tok0 = blockIdx.x * kOpenTokens, t = tok0 + wave;
  const bool live = t < T;                 // (a wavefront without a token still shares the work)
  uint32_t u[NPL], thr = 0u;
  unsigned long long open[NPL] = {};
  if (live) {
    double sum[NPL] = {};
    float off = 0.f;
    for (int z0 = 0; z0 < splits; z0 += 8) {   // eight parts in flight
      float p[8][NPL], r[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const size_t row = (size_t)min(z0 + q, splits - 1) * T + t;
        r[q] = z0 + q < splits ? reach[row] : 0.f;
#pragma unroll
        for (int n = 0; n < NPL; ++n) p[q][n] = z0 + q < splits && lane + 64 * n < N ? near[row * N + lane + 64 * n] : 0.f;
      }
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        off += r[q];
#pragma unroll
        for (int n = 0; n < NPL; ++n) sum[n] += (double)p[q][n];
      }
    }
    float key[NPL];
    bool finite = true;
#pragma unroll
    for (int n = 0; n < NPL; ++n) {
      const int b = lane + 64 * n;
      const float l = b < N ? (float)(sum[n] + (br ? (double)br[b] : 0.0)) : 0.f;
      key[n] = (flags & 1) ? fabsf(l) : l;
      u[n] = b < N ? key_image(l, flags) : 0u;
      finite = finite && fabsf(l) < INFINITY;
    }
    thr = kth_image<NPL>(u, k);
    off = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(off)));
    if (off != 0.f) {                      // (no error: the sums are zeros; NaN != 0)
      auto value = [](uint32_t image) { return __uint_as_float((image & 0x80000000u) ? image & 0x7FFFFFFFu : ~image); };
      int at_least = 0;
      uint32_t next = 0u;                  // the largest image not selected
#pragma unroll
      for (int n = 0; n < NPL; ++n) {
        at_least += (int)__popcll(__ballot(u[n] >= thr));
        next = max(next, u[n] < thr ? u[n] : 0u);
      }
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) next = max(next, (uint32_t)__shfl_xor((int)next, o));
      if (at_least > k) next = thr;
      const float kth = value(thr), after = value(next);
      float margin = 2.f * off + 0x1p-22f * fmaxf(fabsf(kth), fabsf(after));
      if (!__all(finite)) margin = INFINITY;
      if (next != 0u && !(kth - after > margin)) {
#pragma unroll
        for (int n = 0; n < NPL; ++n) {
          const int b = lane + 64 * n;
          const bool in = key[n] - margin > after, out = key[n] + margin < kth;
          open[n] = __ballot(b < N && !in && !out);
          u[n] = b < N && in ? 0xFFFFFFFFu : 0u;
        }
      }
    }
  }
  int count = 0;
#pragma unroll
  for (int n = 0; n < NPL; ++n) {
    if (open[n] >> lane & 1) list[wave][count + __popcll(open[n] & ((1ull << lane) - 1ull))] = (uint8_t)(lane + 64 * n);
    count += (int)__popcll(open[n]);
  }
  if (lane == 0) turns[wave] = (count + 1) >> 1 | count << 16;
  __syncthreads();
  // Lane i: the turns of token i and of those before it.
  const int mine = lane < kOpenTokens ? turns[lane] : 0;
  int upto = mine & 0xFFFF;
#pragma unroll
  for (int o = 1; o < kOpenTokens; o <<= 1) {
    const int below = __shfl_up(upto, o);
    if (lane >= o) upto += below;
  }
  const int total = __builtin_amdgcn_readlane(upto, kOpenTokens - 1);
  if (total > kNearTurns) {
    // All blocks of the 16 tokens, as router_logits_kernel has it: a wavefront takes a column tile and a share of d's chunks of 32.
    const int r16 = lane & 15, slot = lane >> 4, ct = wave % CT, kp = wave / CT, b = 16 * ct + r16;
    f64x4 acc = {0.0, 0.0, 0.0, 0.0};
    if (16 * ct < N) {                     // uniform
      const uint16_t* x = X + (size_t)min(tok0 + r16, T - 1) * d + 8 * slot;
      const float* w = Wt + (size_t)min(b, N - 1) * d + 8 * slot;
      const int last = d / 32 - 1;
      u32x4 xn;
      f32x4 wn[2];
      auto request = [&](int c) {          // (past the last chunk: repeated, not used)
        xn = *reinterpret_cast<const u32x4*>(x + 32 * min(c, last));
        wn[0] = *reinterpret_cast<const f32x4*>(w + 32 * min(c, last));
        wn[1] = *reinterpret_cast<const f32x4*>(w + 32 * min(c, last) + 4);
      };
      request(kp);
      for (int c = kp; c <= last; c += KP) {
        const u32x4 xv = xn;
        const f32x4 wv[2] = {wn[0], wn[1]};
        request(c + KP);
#pragma unroll
        for (int e = 0; e < 8; ++e)
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)(e & 1 ? hi_bf16(xv[e / 2]) : lo_bf16(xv[e / 2])),
                                                     (double)wv[e / 4][e % 4], acc, 0, 0, 0);
      }
      if (kp > 0) {
#pragma unroll
        for (int v = 0; v < 4; ++v) red[kp - 1][ct][v][lane] = acc[v];
      }
    }
    __syncthreads();
    if (kp == 0 && b < N) {                // (the shares in order; rows 4 v + slot are the tokens)
      const double bias = br ? (double)br[b] : 0.0;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
#pragma unroll
        for (int q = 0; q < KP - 1; ++q) acc[v] += red[q][ct][v][lane];
        keys[4 * v + slot][b] = key_image((float)(acc[v] + bias), flags);
      }
    }
  } else {
    for (int turn = wave; turn < total; turn += kOpenTokens) {   // two blocks of a token
      const int i = (int)__popcll(__ballot(lane < kOpenTokens && upto <= turn));
      const int first = 2 * (turn - (i ? __builtin_amdgcn_readlane(upto, i - 1) : 0));
      const int second = min(first + 1, (__builtin_amdgcn_readlane(mine, i) >> 16) - 1);
      const int b0 = __builtin_amdgcn_readfirstlane(list[i][first]), b1 = __builtin_amdgcn_readfirstlane(list[i][second]);
      const uint16_t* x = X + (size_t)(tok0 + i) * d;
      const float *w0 = Wt + (size_t)b0 * d, *w1 = Wt + (size_t)b1 * d;
      double s0 = 0.0, s1 = 0.0;
      for (int k0 = 8 * lane; k0 < d; k0 += 512 * 2) {
        u32x4 xv[2];
        f32x4 wv[2][4];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const int c = min(k0 + 512 * q, d - 8);
          xv[q] = *reinterpret_cast<const u32x4*>(x + c);
          wv[q][0] = *reinterpret_cast<const f32x4*>(w0 + c);
          wv[q][1] = *reinterpret_cast<const f32x4*>(w0 + c + 4);
          wv[q][2] = *reinterpret_cast<const f32x4*>(w1 + c);
          wv[q][3] = *reinterpret_cast<const f32x4*>(w1 + c + 4);
        }
        // (all of them requested before the first is used)
        asm volatile("" : "+v"(xv[0]), "+v"(xv[1]), "+v"(wv[0][0]), "+v"(wv[0][1]), "+v"(wv[0][2]), "+v"(wv[0][3]),
                     "+v"(wv[1][0]), "+v"(wv[1][1]), "+v"(wv[1][2]), "+v"(wv[1][3]));
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          if (k0 + 512 * q >= d) break;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const double xe = (double)(e & 1 ? hi_bf16(xv[q][e / 2]) : lo_bf16(xv[q][e / 2]));
            s0 = fma(xe, (double)wv[q][e / 4][e % 4], s0);
            s1 = fma(xe, (double)wv[q][2 + e / 4][e % 4], s1);
          }
        }
      }
      // (lanes below 32 go on with the first sum, the others with the second)
      double both = (lane < 32 ? s0 : s1) + __shfl_xor(lane < 32 ? s1 : s0, 32);
#pragma unroll
      for (int o = 16; o >= 1; o >>= 1) both += __shfl_xor(both, o);
      const int b = lane < 32 ? b0 : b1;
      if ((lane & 31) == 0) keys[i][b] = key_image((float)(both + (br ? (double)br[b] : 0.0)), flags);
    }
  }
  if (total > 0) __syncthreads();          // uniform
  if (!live) return;
  if (count > 0) {                         // uniform
#pragma unroll
    for (int n = 0; n < NPL; ++n)
      if (open[n] >> lane & 1) u[n] = keys[wave][lane + 64 * n];
    thr = kth_image<NPL>(u, k);
  }
  emit_topk<NPL>(u, thr, lane, k, idx + (size_t)t * k);
}

// Parts of d for that path, 0 for none: it costs 13 to 40 us, the more the longer a row, however few the tokens, against fp64
// units that take 30 x 10^6 products a us.  us, fp64 / this: d 4096, N 128 T 1024 28 / 33, 2048 46 / 37; d 2048, N 64 T 2048
// 16 / 20, 4096 27 / 23; d 1024, N 64 T 4096 18 / 19, 8192 29 / 24; d 512, N 64 T 8192 20 / 21, 16384 34 / 30; d 256, N 128
// T 8192 25 / 26, 16384 45 / 37; d 8192, N 128 T 1024 46 / 41.  (Up to 32 blocks the fp64 kernel selects as well.)
static int near_splits(const spt_shape_t& s) {
  if (s.N <= 32 || s.N > 128 || (int64_t)s.T * s.N * s.d < (1ll << 28) + (1ll << 17) * s.d) return 0;
  const int tiles = (s.T + kNearTokens - 1) / kNearTokens, units = (s.d + 63) / 64;
  // the fewest rounds of workgroups times units of 64 columns, and about three units' time before and after them
  int best = 1;
  int64_t least = INT64_MAX;
  for (int p = 1; p <= 16 && (p == 1 || units / p >= 4); ++p) {
    const int64_t rounds = ((int64_t)tiles * p + 255) / 256, cost = rounds * ((units + p - 1) / p + 3);
    if (cost < least) { least = cost; best = p; }
  }
  return best;
}
// What a sum can be off by, as a multiple of |x| |w|: three MFMAs for each of a stage's K-steps of a wavefront, each by two units
// in the last place of the magnitudes so far, a half for each addition of a stage, of the wavefronts and of the parts.
static float near_tie(const spt_shape_t& s, int splits) {
  const int steps = 4 * ((((s.d + 63) / 64) + splits - 1) / splits);
  return (float)(48 + (steps + kNearStage - 1) / kNearStage + kNearWaves + splits) * 0x1p-24f;
}
// Workspace: W_r with the blocks as rows, the sums of the parts, what they can be off by.
static size_t near_copy_floats(const spt_shape_t& s) { return (size_t)s.N * s.d; }
static void launch_near(const spt_shape_t& s, const uint16_t* X, const float* Wr, float* ws, int splits, hipStream_t st) {
  const int grid = (s.T + kNearTokens - 1) / kNearTokens * splits;
  float *near = ws + near_copy_floats(s), *reach = near + (size_t)splits * s.T * s.N;
  const float tie = near_tie(s, splits);
  if (s.N <= 64) router_near_kernel<2><<<grid, 64 * kNearWaves, 0, st>>>(X, Wr, s.T, s.d, s.N, splits, tie, near, reach, ws);
  else router_near_kernel<4><<<grid, 64 * kNearWaves, 0, st>>>(X, Wr, s.T, s.d, s.N, splits, tie, near, reach, ws);
}
template <int NPL>
static void launch_topk_near(const spt_shape_t& s, const uint16_t* X, const float* br, const float* ws, int splits,
                             int32_t* idx, hipStream_t st) {
  const float *near = ws + near_copy_floats(s), *reach = near + (size_t)splits * s.T * s.N;
  topk_near_kernel<NPL><<<(s.T + kOpenTokens - 1) / kOpenTokens, 64 * kOpenTokens, 0, st>>>(
      near, reach, ws, X, br, splits, s.T, s.d, s.N, s.k, s.flags, idx);
}

template <int NPL>
static void launch_topk(const spt_shape_t& s, const float* logits, const double* partial, const float* br, int splits,
                        int32_t* idx, hipStream_t st) {
  topk_kernel<NPL><<<(s.T + 3) / 4, 256, 0, st>>>(logits, partial, br, splits, s.T, s.N, s.k, s.flags, idx);
}

// Parts d is split into over workgroups: a tile of 16 tokens x 16 blocks keeps one CU's fp64 units busy
// for 4 d cycles (8 us at d = 4096), so a batch with few tiles hands every tile to several CUs.
static int router_splits(const spt_shape_t& s) {
  const int64_t tiles = (int64_t)((s.T + 15) / 16) * ((s.N + 15) / 16);
  if (tiles > 64 || s.d < 1024) return 1;
  const int fill = (int)(256 / tiles), most = s.d / 256;
  const int p = fill < most ? fill : most;
  return p < 16 ? p : 16;
}

size_t router_ws_bytes(const spt_shape_t& s) {
  const size_t n = (size_t)s.T * s.N;
  if (const int near = near_splits(s)) return align256((near_copy_floats(s) + (n + s.T) * near) * sizeof(float));
  const int splits = router_splits(s);
  return align256(splits > 1 ? n * splits * sizeof(double) : n * sizeof(float));
}

template <int MT, int NT, int KS, int DEPTH, bool TOPK>
static void launch_logits(const spt_shape_t& s, const uint16_t* X, const float* Wr, const float* br, int32_t* idx,
                          float* logits, double* partial, int splits, hipStream_t st) {
  const dim3 grid((s.T + 16 * MT - 1) / (16 * MT), (s.N + 16 * NT - 1) / (16 * NT), splits);
  router_logits_kernel<MT, NT, KS, DEPTH, TOPK><<<grid, 64 * KS, 0, st>>>(X, Wr, br, s.T, s.d, s.N, logits, partial,
                                                                         s.k, s.flags, idx);
}

hipError_t run_router_topk(const spt_shape_t& s, const void* X, const float* Wr, const float* br,
                           int32_t* idx, float* logits, float* ws, hipStream_t st) {
  const uint16_t* x = static_cast<const uint16_t*>(X);
  if (const int near = logits ? 0 : near_splits(s)) {
    {
      ScopedKernelTimer tm(kSlotRouter, st);
      launch_near(s, x, Wr, ws, near, st);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    ScopedKernelTimer tm(kSlotTopk, st);
    if (s.N <= 64) launch_topk_near<1>(s, x, br, ws, near, idx, st);
    else launch_topk_near<2>(s, x, br, ws, near, idx, st);
    return hipGetLastError();
  }
  // (the caller's logits leave no workspace to split over)
  const int splits = logits ? 1 : router_splits(s);
  const bool fused = s.N <= 32 && splits == 1;
  double* partial = splits > 1 ? reinterpret_cast<double*>(ws) : nullptr;
  float* l = logits ? logits : (fused || partial) ? nullptr : ws;
  {
    ScopedKernelTimer tm(kSlotRouter, st);
    auto tiles = [&](int mt, int nt) {
      return (int64_t)((s.T + 16 * mt - 1) / (16 * mt)) * ((s.N + 16 * nt - 1) / (16 * nt));
    };
    // The largest tile of which there are two for every CU (a wider one shares the conversions of a
    // token's values between its blocks; measured at N = 128, d = 4096, with logits, us: T 8192 164 with 32 x 32 against
    // 186 with 16 x 16, T 3001 87 against 75 with 16 x 32, T 24 46 against 21 with 16 x 16).
    if (fused && s.N <= 16) launch_logits<1, 1, 8, 3, true>(s, x, Wr, br, idx, l, partial, splits, st);
    else if (fused) launch_logits<1, 2, 8, 3, true>(s, x, Wr, br, idx, l, partial, splits, st);
    else if (tiles(2, 2) >= 512) launch_logits<2, 2, 8, 3, false>(s, x, Wr, br, idx, l, partial, splits, st);
    else if (tiles(1, 2) >= 512) launch_logits<1, 2, 8, 3, false>(s, x, Wr, br, idx, l, partial, splits, st);
    else launch_logits<1, 1, 8, 3, false>(s, x, Wr, br, idx, l, partial, splits, st);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || fused) return e;
  {
    ScopedKernelTimer tm(kSlotTopk, st);
    const int npl = (s.N + 63) / 64;
    if (npl <= 1) launch_topk<1>(s, l, partial, br, splits, idx, st);
    else if (npl <= 2) launch_topk<2>(s, l, partial, br, splits, idx, st);
    else if (npl <= 4) launch_topk<4>(s, l, partial, br, splits, idx, st);
    else if (npl <= 8) launch_topk<8>(s, l, partial, br, splits, idx, st);
    else launch_topk<16>(s, l, partial, br, splits, idx, st);
  }
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// Load-balancing loss of the route network (section 4.2 names such a loss; the formula is this
// build's choice, the usual one for top-k routers):
//   f_b = share of the (token, slot) pairs routed to block b (from the bucket offsets, held constant),
//   p_t = softmax of the token's logits, pbar_b = mean_t p_t[b],  loss = N sum_b f_b pbar_b,
//   dlogit[t][c] = (N / T) p_t[c] (f_c - sum_b f_b p_t[b]),  dW_r = X^T dlogit,  db_r = sum_t dlogit[t].
// Kernel 1: one wavefront per token (8 tokens per wavefront), softmax in fp32; writes
// dlogit as bf16 rows padded to a multiple of 32 blocks (the operand of the dW_r contraction) and, per
// workgroup, the sums of p and dlogit over its 32 tokens (added up in kernel 3 in group order).  A token is a
// chain of a load and eighteen cross-lane steps, so four of them go through it side by side where the registers allow.
// (32 tokens one after the other: 39 us for 8192 tokens, 64 blocks.)
// Kernel 2: the contraction of X with dlogit over chunks of the tokens (row_contraction).
constexpr int kBalTokPerWave = 8;

template <int NPL>
__global__ __launch_bounds__(256) void balance_kernel(const float* __restrict__ logits,
                                                      const int32_t* __restrict__ offsets, int T, int N,
                                                      int k, int npad, uint16_t* __restrict__ dl,
                                                      float* __restrict__ part,
                                                      uint32_t* __restrict__ zero_row) {
  __shared__ float red[3][2][NPL * 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (blockIdx.x == 0 && threadIdx.x < 64) zero_row[threadIdx.x] = 0u;
  float f[NPL], sp[NPL], sd[NPL];
  const float inv_pairs = 1.0f / ((float)T * (float)k);
#pragma unroll
  for (int n = 0; n < NPL; ++n) {
    const int b = lane + 64 * n;
    f[n] = (b < N) ? (float)(offsets[b + 1] - offsets[b]) * inv_pairs : 0.f;
    sp[n] = 0.f;
    sd[n] = 0.f;
  }
  const float scale = (float)N / (float)T;
  const int t0 = (blockIdx.x * 4 + wave) * kBalTokPerWave;
  constexpr int TB = NPL <= 4 ? 4 : 1;   // tokens side by side
  for (int i = 0; i < kBalTokPerWave; i += TB) {
    if (t0 + i >= T) break;  // wave-uniform
    float x[TB][NPL], m[TB], ssum[TB], c[TB];
#pragma unroll
    for (int a = 0; a < TB; ++a) {
      const int t = min(t0 + i + a, T - 1);
      m[a] = -INFINITY;
#pragma unroll
      for (int n = 0; n < NPL; ++n) {
        const int b = lane + 64 * n;
        x[a][n] = (b < N) ? logits[(size_t)t * N + b] : -INFINITY;
      }
    }
#pragma unroll
    for (int a = 0; a < TB; ++a)
#pragma unroll
      for (int n = 0; n < NPL; ++n) m[a] = fmaxf(m[a], x[a][n]);
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1)
#pragma unroll
      for (int a = 0; a < TB; ++a) m[a] = fmaxf(m[a], __shfl_xor(m[a], o));
#pragma unroll
    for (int a = 0; a < TB; ++a) {
      ssum[a] = 0.f;
#pragma unroll
      for (int n = 0; n < NPL; ++n) {
        x[a][n] = (lane + 64 * n < N) ? __expf(x[a][n] - m[a]) : 0.f;
        ssum[a] += x[a][n];
      }
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1)
#pragma unroll
      for (int a = 0; a < TB; ++a) ssum[a] += __shfl_xor(ssum[a], o);
#pragma unroll
    for (int a = 0; a < TB; ++a) {
      const float inv = 1.0f / ssum[a];
      c[a] = 0.f;
#pragma unroll
      for (int n = 0; n < NPL; ++n) {
        x[a][n] *= inv;  // p_t[b]
        c[a] += f[n] * x[a][n];
      }
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1)
#pragma unroll
      for (int a = 0; a < TB; ++a) c[a] += __shfl_xor(c[a], o);
#pragma unroll
    for (int a = 0; a < TB; ++a) {
      const int t = t0 + i + a;
      if (t >= T) break;  // wave-uniform
#pragma unroll
      for (int n = 0; n < NPL; ++n) {
        const int b = lane + 64 * n;
        const float g = scale * x[a][n] * (f[n] - c[a]);
        sp[n] += x[a][n];
        sd[n] += g;
        if (b < npad) dl[(size_t)t * npad + b] = (uint16_t)f32_to_bf16_bits(b < N ? g : 0.f);
      }
    }
  }
  if (wave > 0) {
#pragma unroll
    for (int n = 0; n < NPL; ++n) {
      red[wave - 1][0][lane + 64 * n] = sp[n];
      red[wave - 1][1][lane + 64 * n] = sd[n];
    }
  }
  __syncthreads();
  if (wave == 0) {
#pragma unroll
    for (int n = 0; n < NPL; ++n) {
      const int b = lane + 64 * n;
      if (b >= N) continue;
      const float p3 = ((sp[n] + red[0][0][b]) + red[1][0][b]) + red[2][0][b];
      const float d3 = ((sd[n] + red[0][1][b]) + red[1][1][b]) + red[2][1][b];
      part[((size_t)blockIdx.x * 2 + 0) * N + b] = p3;
      part[((size_t)blockIdx.x * 2 + 1) * N + b] = d3;
    }
  }
}

// Kernel 3.  dWr[i][b] = sum over the chunks, in order, of the staged contraction of X with dlogit; the last
// workgroup adds the partial sums of kernel 1 in fixed order instead: pbar, db_r, the block shares and the loss.  (That
// sum by a workgroup in a launch of its own, one value in flight per thread, took 18 us for 64 groups.)
__global__ __launch_bounds__(1024) void balance_finish_kernel(const float* __restrict__ stage, int nchunks, int npad,
                                                              int d, float* __restrict__ dWr,
                                                              const float* __restrict__ part,
                                                              const int32_t* __restrict__ offsets, int groups, int T,
                                                              int N, int k, float* __restrict__ loss,
                                                              float* __restrict__ frac, float* __restrict__ dbr) {
  if (blockIdx.x + 1 < gridDim.x) {
    const int64_t id = (int64_t)blockIdx.x * 1024 + threadIdx.x;
    const int64_t i = id / npad;
    const int b = (int)(id % npad);
    if (i >= d || b >= N) return;
    const size_t stride = (size_t)d * npad;
    float s = 0.f;
#pragma unroll 8
    for (int c = 0; c < nchunks; ++c) s += stage[(size_t)c * stride + id];
    dWr[(size_t)i * N + b] = s;
    return;
  }
  // Columns (p of block 0 .. N-1, then dlogit of them) on the fast axis; where there are fewer than 1024 of them,
  // seg threads share one, each with every seg-th group, and their sums are added in order.
  __shared__ float sums[2048];
  const int cols = 2 * N, seg = cols < 1024 ? 1024 / cols : 1;
  for (int c0 = 0; c0 < cols; c0 += 1024) {
    const int c = c0 + (int)threadIdx.x % cols, sg = seg > 1 ? (int)threadIdx.x / cols : 0;
    float s = 0.f;
    if (c < cols && sg < seg) {
      const float* col = part + c;
      int g = sg;
      for (; g + 7 * seg < groups; g += 8 * seg) {
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = col[(size_t)(g + e * seg) * cols];
#pragma unroll
        for (int e = 0; e < 8; ++e) s += v[e];
      }
      for (; g < groups; g += seg) s += col[(size_t)g * cols];
    }
    sums[c0 + threadIdx.x] = s;
  }
  __syncthreads();
  const int b = threadIdx.x;
  float sp = 0.f, sd = 0.f, fb = 0.f;
  if (b < N) {
    for (int g = 0; g < seg; ++g) {
      sp += sums[g * cols + b];
      sd += sums[g * cols + N + b];
    }
    fb = (float)(offsets[b + 1] - offsets[b]) / ((float)T * (float)k);
    if (frac) frac[b] = fb;
    if (dbr) dbr[b] = sd;
  }
  __syncthreads();
  sums[b] = (b < N) ? fb * (sp / (float)T) : 0.f;
  for (int o = 512; o >= 1; o >>= 1) {
    __syncthreads();
    if (b < o) sums[b] += sums[b + o];
  }
  if (b == 0) *loss = (float)N * sums[0];
}

template <int NPL>
static void launch_balance(const float* logits, const int32_t* offsets, const spt_shape_t& s,
                           const BalanceWorkspace& w, hipStream_t st) {
  balance_kernel<NPL><<<w.groups, 256, 0, st>>>(logits, offsets, s.T, s.N, s.k, w.npad, w.dl, w.part,
                                                reinterpret_cast<uint32_t*>(w.zero_row));
}

BalanceWorkspace plan_balance(const spt_shape_t& s, void* ws) {
  char* p = static_cast<char*>(ws);
  size_t o = 0;
  BalanceWorkspace w = {};
  auto take = [&](size_t bytes) { void* r = p + o; o += align256(bytes); return r; };
  w.npad = (s.N + 31) / 32 * 32;
  w.groups = (s.T + 4 * kBalTokPerWave - 1) / (4 * kBalTokPerWave);
  w.chunk = grad_piece_rows(s.T, 1, s.d * ((w.npad + 63) / 64));
  w.nchunks = (s.T + w.chunk - 1) / w.chunk;
  w.dl = static_cast<uint16_t*>(take((size_t)s.T * w.npad * 2));
  w.part = static_cast<float*>(take((size_t)w.groups * 2 * s.N * 4));
  w.gchunks = static_cast<float*>(take((size_t)w.nchunks * w.npad * s.d * 4));
  w.zero_row = static_cast<uint16_t*>(take(256));
  w.bytes = o;
  return w;
}

hipError_t run_router_balance(const spt_shape_t& s, const void* X, const float* logits,
                              const int32_t* offsets, float* loss, float* frac, float* dWr, float* dbr,
                              const BalanceWorkspace& w, hipStream_t st) {
  hipError_t e;
  ScopedKernelTimer tm(kSlotBalance, st);
  const int npl = (s.N + 63) / 64;
  if (npl <= 1) launch_balance<1>(logits, offsets, s, w, st);
  else if (npl <= 2) launch_balance<2>(logits, offsets, s, w, st);
  else if (npl <= 4) launch_balance<4>(logits, offsets, s, w, st);
  else if (npl <= 8) launch_balance<8>(logits, offsets, s, w, st);
  else launch_balance<16>(logits, offsets, s, w, st);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  // dW_r[i][b] = sum_t X[t][i] dlogit[t][b], per chunk of the tokens
  GradJob jb = {};
  jb.H = static_cast<const uint16_t*>(X); jb.R = w.dl; jb.out = w.gchunks;
  jb.units = s.d; jb.ldr = w.npad; jb.ldo = w.npad;
  jb.npieces = w.nchunks; jb.tiles = (s.d + 127) / 128; jb.piece = w.chunk; jb.rows = s.T; jb.nblocks = 1;
  if ((e = row_contraction(jb, w.zero_row, st)) != hipSuccess) return e;
  const int64_t items = (int64_t)s.d * w.npad;
  balance_finish_kernel<<<(unsigned)((items + 1023) / 1024) + 1, 1024, 0, st>>>(
      w.gchunks, w.nchunks, w.npad, s.d, dWr, w.part, offsets, w.groups, s.T, s.N, s.k, loss, frac, dbr);
  return hipGetLastError();
}

}  // namespace spt
