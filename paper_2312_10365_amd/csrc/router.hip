// Route network + block selection (paper section 4.2, "Dynamic routing").
//
// logit[t][b] = sum_i X[t][i] * W_r[i][b] (+ b_r[b]) accumulated in fp64 and rounded once to
// fp32.  Products of a bf16 and an fp32 value are exact in fp64, so only the order of the
// additions can move the fp64 sum, by parts in 1e-16 -- far below the fp32 rounding step.
// The k largest keys win; equal keys go to the lower block id; ids are emitted ascending.
//
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
#include "spt_device.hpp"
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
template <int NPL>
__device__ __forceinline__ void select_topk(const float (&logit)[NPL], int lane, int N, int k, int flags,
                                            int32_t* __restrict__ out) {
  uint32_t u[NPL];                         // 0 for lanes past N: below every real key
#pragma unroll
  for (int n = 0; n < NPL; ++n)
    u[n] = lane + 64 * n < N ? key_image(logit[n], flags) : 0u;
  uint32_t thr = 0u;
#pragma unroll 1
  for (int bit = 31; bit >= 0; --bit) {
    const uint32_t cand = thr | (1u << bit);
    int c = 0;
#pragma unroll
    for (int n = 0; n < NPL; ++n) c += __popcll(__ballot(u[n] >= cand));
    if (c >= k) thr = cand;                // uniform
  }
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
    need -= min(need, __popcll(eq));
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
  select_topk<NPL>(l, lane, N, k, flags, idx + (size_t)t * k);
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
    // token's values between its blocks; measured at N = 128, d = 4096, us: T 8192 164 with 32 x 32 against
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
