// Token batching by activated block: Algorithm 4's per-block token selection, done once
// for all blocks as a stable counting sort of the (token, slot) pairs by block id.
//
// Small integer kernels, exact and deterministic.  Per chunk of 128 tokens a (block x token) membership
// bitmask in LDS gives the chunk's histogram; then each chunk rebuilds its bitmask, adds up the
// histograms of the chunks before it, and the rank of a pair inside its bucket is that base plus the
// number of lower tokens of the chunk in the same bucket (popcount).  Few pairs are sorted whole by one
// workgroup in one launch; very many blocks times chunks get their bases from a launch of their own.
// A token lists each block at most once, so one bit per (block, token) is enough, and the
// order inside a bucket is by token id, i.e. stable.
#include "spt_device.hpp"
#include "spt_host.hpp"
#include "profile.hpp"

namespace spt {

constexpr int kWordsPerChunk = kBucketChunkTokens / 32;

// A thread's pairs of a chunk of `count`: the first eight, tid, tid + threads, .., are held in registers (requested together, and once
// for all passes over them), what is beyond -- more than eight times the threads -- is loaded in every pass.
struct ChunkPairs {
  const int32_t* idx;
  int count, held[8];
  __device__ __forceinline__ ChunkPairs(const int32_t* from, int n) : idx(from), count(n) {
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int e = threadIdx.x + u * blockDim.x;
      held[u] = e < count ? idx[e] : -1;
    }
  }
  // f(pair, its block), for blocks below N
  template <class F>
  __device__ __forceinline__ void each(int N, F f) const {
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (held[u] >= 0 && held[u] < N) f((int)(threadIdx.x + u * blockDim.x), held[u]);
    for (int e = threadIdx.x + 8 * blockDim.x; e < count; e += blockDim.x) {
      const int b = idx[e];
      if (b >= 0 && b < N) f(e, b);
    }
  }
};

__device__ __forceinline__ void build_chunk_mask(const ChunkPairs& pairs, int N, int k, uint32_t* mask) {
  for (int e = threadIdx.x; e < N * kWordsPerChunk; e += blockDim.x) mask[e] = 0u;
  __syncthreads();
  pairs.each(N, [&](int e, int b) {
    const int tl = e / k;
    atomicOr(&mask[b * kWordsPerChunk + (tl >> 5)], 1u << (tl & 31));
  });
  __syncthreads();
}

__global__ __launch_bounds__(1024) void bucket_hist_kernel(const int32_t* __restrict__ idx, int T,
                                                          int N, int k,
                                                          int32_t* __restrict__ chunk_hist) {
  extern __shared__ uint32_t mask[];
  const int t0 = blockIdx.x * kBucketChunkTokens;
  const ChunkPairs pairs(idx + (int64_t)t0 * k, min(kBucketChunkTokens, T - t0) * k);
  build_chunk_mask(pairs, N, k, mask);
  for (int b = threadIdx.x; b < N; b += blockDim.x) {
    int c = 0;
#pragma unroll
    for (int w = 0; w < kWordsPerChunk; ++w) c += __popc(mask[b * kWordsPerChunk + w]);
    chunk_hist[(size_t)blockIdx.x * N + b] = c;
  }
}

// One workgroup of 1024 threads; thread b owns bucket b.
__global__ __launch_bounds__(1024) void bucket_scan_kernel(int32_t* __restrict__ chunk_hist,
                                                           int nchunks, int N,
                                                           int32_t* __restrict__ offsets) {
  __shared__ int32_t scan[16];
  const int b = threadIdx.x;
  int total = 0;
  if (b < N) {
    for (int c0 = 0; c0 < nchunks; c0 += 16) {   // sixteen loads in flight, then the running sums
      int v[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) v[u] = (c0 + u < nchunks) ? chunk_hist[(size_t)(c0 + u) * N + b] : 0;
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        if (c0 + u < nchunks) chunk_hist[(size_t)(c0 + u) * N + b] = total;  // pairs of this bucket in earlier chunks
        total += v[u];
      }
    }
  }
  // exclusive scan of the bucket totals: wavefront prefix by shuffles, wavefront sums through LDS
  const int lane = b & 63, wave = b >> 6;
  int incl = total;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int up = __shfl_up(incl, o);
    if (lane >= o) incl += up;
  }
  if (lane == 63) scan[wave] = incl;
  __syncthreads();
  int before = incl - total;
  for (int wv = 0; wv < wave; ++wv) before += scan[wv];
  if (b < N) offsets[b] = before;
  if (b == N - 1) offsets[N] = before + total;
}

// kScan: chunk_hist holds the chunks' histograms as they are and this kernel adds up those before its own
// chunk (and all of them, for the offsets, which workgroup 0 writes); otherwise it holds the bases and
// `offsets` is complete.
template <bool kScan>
__global__ __launch_bounds__(1024) void bucket_scatter_kernel(
    const int32_t* __restrict__ idx, int T, int N, int k, const int32_t* __restrict__ chunk_hist, int nchunks,
    int32_t* __restrict__ offsets, int32_t* __restrict__ perm, int32_t* __restrict__ inv) {
  extern __shared__ uint32_t mask[];                       // [N][4] bits, then [N] first position per bucket
  int32_t* first = reinterpret_cast<int32_t*>(mask + N * kWordsPerChunk);
  __shared__ int32_t wtot[16];
  const int chunk = blockIdx.x, t0 = chunk * kBucketChunkTokens;
  const int64_t p0 = (int64_t)t0 * k;
  const ChunkPairs pairs(idx + p0, min(kBucketChunkTokens, T - t0) * k);
  if (kScan) {
    // thread = bucket and a share of the chunks (sixteen or more, if the threads are not enough), sixteen loads in flight
    __shared__ int2 share[1024];
    const int blog = N > 1 ? 32 - __clz(N - 1) : 0, shares = min((int)blockDim.x >> blog, (nchunks + 15) / 16);
    const int b = threadIdx.x, sb = b & ((1 << blog) - 1), sh = b >> blog;
    const int per = (nchunks + shares - 1) / shares, cend = sh < shares ? min(nchunks, (sh + 1) * per) : 0;
    int before = 0, all = 0;
    if (sb < N) {
      for (int c0 = sh * per; c0 < cend; c0 += 16) {
        int v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) v[u] = (c0 + u < cend) ? chunk_hist[(size_t)(c0 + u) * N + sb] : 0;
#pragma unroll
        for (int u = 0; u < 16; ++u) {
          before += c0 + u < chunk ? v[u] : 0;
          all += v[u];
        }
      }
    }
    share[b] = make_int2(before, all);
    __syncthreads();
    before = all = 0;
    if (b < N) {
      for (int x = 0; x < shares; ++x) {
        const int2 y = share[(x << blog) + b];
        before += y.x;
        all += y.y;
      }
    }
    int total;
    const int off = block_inclusive_sum(all, wtot, total) - all;
    if (b < N) first[b] = off + before;
    if (chunk == 0) {
      if (b < N) offsets[b] = off;
      if (b == 0) offsets[N] = total;
    }
  } else {
    for (int b = threadIdx.x; b < N; b += blockDim.x) first[b] = offsets[b] + chunk_hist[(size_t)chunk * N + b];
  }
  build_chunk_mask(pairs, N, k, mask);
  pairs.each(N, [&](int e, int b) {
    const int tl = e / k;
    const uint32_t* m = mask + b * kWordsPerChunk;
    int r = __popc(m[tl >> 5] & ((1u << (tl & 31)) - 1u));
    for (int w = 0; w < (tl >> 5); ++w) r += __popc(m[w]);
    const int q = first[b] + r;
    perm[q] = (int32_t)(p0 + e);
    inv[p0 + e] = q;
  });
}

// All pairs by one workgroup: the (block x token) bitmask of the whole batch, bits before each of its words, and
// the block totals' prefix all sit in LDS.  A thread has Q pairs, loaded before the masks are cleared; P k < 2^31, so that a pair's token is
// exact as a product.  (Loaded twice, divisions, eight of them whatever P: us a pass of 512 tokens in 32 blocks, 8 each 34.2, now 33.5; of 24 tokens in 128, 32
// each 76.7, 76.1.)
template <int Q>
__global__ __launch_bounds__(1024) void bucket_small_kernel(const int32_t* __restrict__ idx, int T, int N, int k,
                                                            int32_t* __restrict__ offsets, int32_t* __restrict__ perm,
                                                            int32_t* __restrict__ inv) {
  extern __shared__ uint32_t mask[];                       // [N][nwp] bits, [N][nwp] set bits in earlier words, [N] totals
  __shared__ int32_t wtot[16];
  const int nw = (T + 31) >> 5, nwp = nw | 1, P = T * k;   // odd row stride: rows start on different banks
  uint16_t* pre = reinterpret_cast<uint16_t*>(mask + N * nwp);
  int32_t* tot = reinterpret_cast<int32_t*>(pre + ((N * nwp + 1) & ~1));
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint32_t k_inv = (0x80000000u + k - 1) / k;
  int held[Q], tok[Q];
#pragma unroll
  for (int u = 0; u < Q; ++u) held[u] = tid + u * 1024 < P ? idx[tid + u * 1024] : -1;
  for (int e = tid; e < N * nwp; e += 1024) mask[e] = 0u;
  __syncthreads();
#pragma unroll
  for (int u = 0; u < Q; ++u) {
    tok[u] = (int)((uint64_t)(uint32_t)(tid + u * 1024) * k_inv >> 31);
    if (held[u] >= 0 && held[u] < N) atomicOr(&mask[held[u] * nwp + (tok[u] >> 5)], 1u << (tok[u] & 31));
  }
  __syncthreads();
  // 2^seg lanes over the words of a block (all 64 from 33 words on), as many blocks side by side as a wavefront then holds: few
  // tokens are few steps, and one turn for 64 blocks where it was one each (24 tokens, 128 blocks: 7.4 -> 4.0 us).
  const int seg = nw > 32 ? 6 : (nw > 1 ? 32 - __clz(nw - 1) : 0), width = 1 << seg, lw = lane & (width - 1);
  for (int b0 = wave << (6 - seg); b0 < N; b0 += 16 << (6 - seg)) {
    const int b = b0 + (lane >> seg);
    int sum = 0;
    for (int w0 = 0; w0 < nw; w0 += 64) {
      const int w = w0 + lw;
      const int c = b < N && w < nw ? __popc(mask[b * nwp + w]) : 0;
      int incl = c;
      for (int o = 1; o < width; o <<= 1) {
        const int up = __shfl_up(incl, o);
        if (lw >= o) incl += up;
      }
      if (b < N && w < nw) pre[b * nwp + w] = (uint16_t)(sum + incl - c);
      sum += __shfl(incl, lane | (width - 1));
    }
    if (b < N && lw == 0) tot[b] = sum;
  }
  __syncthreads();
  const int mine = tid < N ? tot[tid] : 0;
  int total;
  const int off = block_inclusive_sum(mine, wtot, total) - mine;
  if (tid < N) { tot[tid] = off; offsets[tid] = off; }
  if (tid == 0) offsets[N] = total;
  __syncthreads();
#pragma unroll
  for (int u = 0; u < Q; ++u) {
    const int b = held[u], t = tok[u];
    if (b < 0 || b >= N) continue;
    const int w = b * nwp + (t >> 5);
    const int q = tot[b] + pre[w] + __popc(mask[w] & ((1u << (t & 31)) - 1u));
    perm[q] = tid + u * 1024;
    inv[tid + u * 1024] = q;
  }
}

// Fixed scratch of the allocation-free entry point (spt_bucket_tokens_noalloc): the per-chunk
// histogram table of the three kernels above.  The array's name is only a host-side handle;
// its device address is looked up once per device and used everywhere the memory is meant.
static __device__ __align__(256) int32_t scratch[kStaticBucketScratchInts];

hipError_t bucket_static_scratch(int32_t** out) {
  constexpr int kMaxDevices = 64;
  static int32_t* ptr_of_device[kMaxDevices] = {};
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  if (!ptr_of_device[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));   // the current device's copy of the array
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    ptr_of_device[dev] = static_cast<int32_t*>(p);
  }
  *out = ptr_of_device[dev];
  return hipSuccess;
}

hipError_t run_bucket(const spt_shape_t& s, const int32_t* idx, int32_t* offsets, int32_t* perm,
                      int32_t* inv, int32_t* chunk_hist, hipStream_t st) {
  // One workgroup up to where it takes as long as the two launches and what the second one costs a pass that is waited for, 5 to 7 us.
  // us in a graph, one workgroup / two launches: 2048 pairs 4.8 / 7.0, 4096 5.8 / 7.1, 6144 7.0 / 7.2, 8192 8.0 / 7.4, 12288 10.9 / 7.3,
  // 16384 13.0 / 7.5 (16 blocks, 4 each); 4096 6.5 / 9.8, 8192 9.5 / 9.9, 12288 13.8 / 10.2 (128, 32); 8192 11.0 / 7.6, 12288 17.0 / 7.8 (128, 8).
  const size_t nwp = ((s.T + 31) / 32) | 1;
  const size_t small = (size_t)s.N * nwp * 4 + ((size_t)s.N * nwp + 1) / 2 * 4 + (size_t)s.N * 4;
  const int64_t P = (int64_t)s.T * s.k;
  if (P <= 8192 && small <= 60 * 1024) {
    ScopedKernelTimer tm(kSlotBucketScatter, st);
    if (P <= 2048) bucket_small_kernel<2><<<1, 1024, small, st>>>(idx, s.T, s.N, s.k, offsets, perm, inv);
    else if (P <= 4096) bucket_small_kernel<4><<<1, 1024, small, st>>>(idx, s.T, s.N, s.k, offsets, perm, inv);
    else bucket_small_kernel<8><<<1, 1024, small, st>>>(idx, s.T, s.N, s.k, offsets, perm, inv);
    return hipGetLastError();
  }
  const int nchunks = (s.T + kBucketChunkTokens - 1) / kBucketChunkTokens;
  const size_t smem = (size_t)s.N * kWordsPerChunk * sizeof(uint32_t);
  // Two pairs of a chunk per thread up to 16 of a token's blocks, k / 8 beyond (1024 threads at most; the first eight held in registers), a thread
  // per bucket and 256 at least.  A chunk's work is a chain of loads, LDS atomics and
  // stores whose length is the number of pairs a thread has, behind that of the histograms it adds up.  us, 256 threads with
  // the pairs loaded anew for every pass and all histograms per thread -> this: 8192 tokens, 128 blocks, 32 each 13.8 -> 9.4;
  // 16384, 64, 16 11.3 -> 7.3; 3001, 128, 32 11.8 -> 8.2.  512 threads there: 10.9, 7.6, 9.8; 1024 threads for 2 of 4 blocks, 8192
  // tokens, 8.5 where 256 take 6.0.
  int threads = 256;
  while (threads < 1024 && (threads < s.N || threads < kBucketChunkTokens / 2 * s.k)) threads *= 2;
  {
    ScopedKernelTimer tm(kSlotBucketHist, st);
    bucket_hist_kernel<<<nchunks, threads, smem, st>>>(idx, s.T, s.N, s.k, chunk_hist);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // Every chunk's workgroup reads the whole histogram table (N x chunks counts) unless that is more than
  // 64 KiB of them: then one workgroup turns it into bases first.
  const bool scan = (int64_t)nchunks * s.N > 16384;
  if (scan) {
    ScopedKernelTimer tm(kSlotBucketScan, st);
    bucket_scan_kernel<<<1, 1024, 0, st>>>(chunk_hist, nchunks, s.N, offsets);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  ScopedKernelTimer tm(kSlotBucketScatter, st);
  const size_t sm = smem + (size_t)s.N * sizeof(int32_t);
  if (scan)
    bucket_scatter_kernel<false><<<nchunks, threads, sm, st>>>(idx, s.T, s.N, s.k, chunk_hist, nchunks, offsets, perm, inv);
  else
    bucket_scatter_kernel<true><<<nchunks, threads, sm, st>>>(idx, s.T, s.N, s.k, chunk_hist, nchunks, offsets, perm, inv);
  return hipGetLastError();
}

}  // namespace spt
