// Host-side declarations shared by the translation units of libspt.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/spt.h"

namespace spt {

constexpr int kBucketChunkTokens = 128;  // tokens per workgroup in the bucketing pass

inline size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

// logits may be null: then ws (router_ws_bytes) holds them, or the parts of their sums, between the two
// kernels (or nothing does, with few blocks).
size_t router_ws_bytes(const spt_shape_t& s);
hipError_t run_router_topk(const spt_shape_t& s, const void* X, const float* Wr, const float* br,
                           int32_t* idx, float* logits, float* ws, hipStream_t st);
hipError_t run_bucket(const spt_shape_t& s, const int32_t* idx, int32_t* offsets, int32_t* perm,
                      int32_t* inv, int32_t* chunk_hist, hipStream_t st);
// Device address, on the current device, of the library's fixed bucketing scratch
// (kStaticBucketScratchInts int32: 1 MiB per GPU, held until the process ends).
constexpr size_t kStaticBucketScratchInts = 262144;
hipError_t bucket_static_scratch(int32_t** out);

// Device-built schedule tables shared by the forward and backward launches.
// One work item of the narrow-block weight-gradient GEMMs: the rows [lo, hi) of one bucket and
// where the product goes (dst < N: block dst of the gradient itself; dst >= N: staging slot
// dst - N, added to the block afterwards in slot order; dst < 0: unused table entry).
struct DwPiece { int32_t lo, hi, dst, pad; };
struct Schedule {
  int32_t* border;       // [N] buckets by size, largest first
  int32_t* kd_count;     // [8] row tiles of the K = d GEMMs per XCD; wide blocks: [0] all, [1] those in front of the tails
  void* kd_list;         // [8][kd_cap] (bucket, rows, first row) in per-XCD run order; wide blocks: one list
  int32_t* tok;          // [P] token id of every sorted position
  uint16_t* zero_row;    // 256 bytes of zeros (padding rows of the dW GEMMs' K dimension)
  int32_t* rstart;       // narrow blocks: per token range, the non-empty runs of bucket rows (ffn_scatter.hip)
  int kd_cap;
  // narrow blocks, backward: buckets cut into pieces of at most dw_rows rows (largest bucket first)
  DwPiece* dw_pieces;    // [dw_cap]
  int32_t* dw_xlist;     // [0] = number of buckets with staged pieces, then (bucket, first slot, end slot) triples
  int dw_cap, dw_rows;
};
struct FwdWorkspace {
  Schedule sched;
  uint16_t* Hact;        // bf16 activated hidden values per pair (narrow blocks: fragment order)
  uint16_t* part;        // [P,d] bf16 per-pair partial output rows (wide blocks only)
  float* split;          // ScatterPlan::split_bytes (narrow blocks)
  size_t bytes;
};
struct BwdWorkspace {
  Schedule sched;
  uint16_t* Hact;   // act(Hsave) per pair  (narrow blocks: fragment order, ffn_common.hpp;
  uint16_t* dHpre;  // dHpre per pair        wide blocks: row-major [P,Bs])
  uint16_t* part;   // [P,d] per-pair partial dX rows (wide blocks only)
  float* split;     // ScatterPlan::split_bytes (narrow blocks)
  float* dw_stage;  // [dw_cap - N][Bs][d] products of the pieces after a bucket's first (narrow blocks)
  float* dw_stage2; // ... of the second gradient, when both are formed in one launch; else null
  size_t bytes;
};
FwdWorkspace plan_fwd(const spt_shape_t& s, void* ws);
// weight_grads = false: no tables or staging for the weight-gradient GEMMs (low-rank variant)
BwdWorkspace plan_bwd(const spt_shape_t& s, void* ws, bool weight_grads = true);

// Token-range-stationary K = Bs contraction of narrow blocks (down-projection, dX) with the
// per-token write-back folded in: R tokens x 64 columns per workgroup, nr ranges, nslab slabs.
struct ScatterPlan {
  int R, nr, nslab, smem;
  int cap;               // run records per range
  int run_rows;          // rows of a record at most
  int nt;                // ... in tiles of 16
  int inner;             // column slabs that run side by side on an XCD
  int splits;            // parts of the block list given to workgroups of their own (few tokens; else 1)
  size_t split_bytes;    // [splits][T][d] fp32 sums of the parts, added afterwards
  size_t runs_bytes;     // bytes of the [nr][cap] run records
  size_t counts_bytes;   // bytes of the per-range record counts
  size_t table_bytes;    // run records + counts + the dense [nr+1][N] table of run starts
};
ScatterPlan plan_scatter(const spt_shape_t& s);
// The dense table starts[r][b] (written by the schedule kernel) inside the run-table buffer.
int32_t* scatter_starts(const ScatterPlan& p, int32_t* table);
struct RunRec;   // the ranges' run records [nr][cap] and their counts [nr] in the same buffer
RunRec* scatter_runs(const ScatterPlan& p, int32_t* table);
int32_t* scatter_counts(const ScatterPlan& p, int32_t* table);
// Turns the dense table into the per-range lists of non-empty runs.
hipError_t run_scatter_ranges(const spt_shape_t& s, const ScatterPlan& p, int32_t* table, hipStream_t st);
// out[t][:] = sum_{b in S(t), ascending} Hin[pos(t,b)][:] W[b]  (+ Z[t][:] when Z is given)
hipError_t launch_scatter(const spt_shape_t& s, const ScatterPlan& p, const uint16_t* Hin, const uint16_t* W,
                          const int32_t* rstart, const int32_t* tok, uint16_t* out, const uint16_t* Z,
                          float* split, hipStream_t st);
// One product of the narrow-block weight-gradient GEMM: its operands, the gradient, and the staging slots of pieces.
struct DwOperands {
  const uint16_t *Act, *Hin;
  float *dW, *stage;
};
// The same contraction and both weight-gradient GEMMs in one launch (their pieces still to be summed): short token ranges only.
bool scatter_takes_dw(const spt_shape_t& s, const ScatterPlan& p);
hipError_t launch_scatter_dw(const spt_shape_t& s, const ScatterPlan& p, const uint16_t* Hin, const uint16_t* W, const Schedule& sc,
                             uint16_t* out, const DwOperands* ops, hipStream_t st);

// Arguments of the wide-block GEMM kernels (blocks of more than 128 hidden units).
struct WideArgs {
  const void* A;             // A-side operand (MFMA rows): W block, or the gathered activations
  const void* B;             // B-side operand: gathered activation rows, or H / dHpre
  const int32_t* offsets;
  const int32_t* kd_count;   // number of row tiles, and of those in front of the tails (wide_tails)
  const void* kd_list;       // row tiles, bucket-major, the tails behind them
  const int32_t* tok;
  const int32_t* border;
  const uint16_t* zero_row;
  int N, Bs, d;
  uint16_t* Hsave;           // written by the up-projection (may be null), read by dH
  uint16_t* Hact;
  uint16_t* dHpre;
  uint16_t* part;            // [P,d] row-major partial rows
  float* dW;
  const uint16_t* Xe;        // low-rank extension of the K = d GEMMs: [T][64] per token, or null
  const uint16_t* We;        //                                        [N*Bs][64] per hidden unit
};
enum WideOp { kWideUp = 0, kWideDH = 1, kWidePart = 2, kWideDW = 3 };
// Buckets so small that their last rows are listed apart (wide_rows_kernel).
inline bool wide_tails(const spt_shape_t& s) { return (int64_t)s.T * s.k <= 64 * (int64_t)s.N; }
hipError_t launch_wide(int op, const spt_shape_t& s, const WideArgs& a, hipStream_t st);

// The schedule in a buffer of its own (the layout plan_bwd carves, weight-gradient tables included),
// filled once per bucketing by run_schedule; run_fwd / run_bwd given it as `prebuilt` skip building
// their own.
size_t schedule_bytes(const spt_shape_t& s);
Schedule plan_schedule(const spt_shape_t& s, void* buf);
hipError_t run_schedule(const spt_shape_t& s, const int32_t* offsets, const int32_t* perm, const Schedule& sc,
                        hipStream_t st);

hipError_t run_fwd(const spt_shape_t& s, const void* X, const void* W1, const void* W2,
                   const int32_t* offsets, const int32_t* perm, const int32_t* inv, void* Y,
                   void* Hsave, const FwdWorkspace& w, hipStream_t st, const Schedule* prebuilt = nullptr);
hipError_t run_bwd(const spt_shape_t& s, const void* X, const void* W1, const void* W2,
                   const void* dY, const int32_t* offsets, const int32_t* perm,
                   const int32_t* inv, const void* Hsave, void* dX, float* dW1, float* dW2,
                   const BwdWorkspace& w, hipStream_t st, const Schedule* prebuilt = nullptr);

// Load-balancing loss of the route network and its gradient.
struct BalanceWorkspace {
  uint16_t* dl;        // [T][Npad] bf16 d loss / d logit
  float* part;         // [groups][2][N] partial sums of p and of dlogit
  float* gchunks;      // [chunks][d][Npad] gradient staging
  uint16_t* zero_row;
  int npad, groups, chunk, nchunks;
  size_t bytes;
};
BalanceWorkspace plan_balance(const spt_shape_t& s, void* ws);
hipError_t run_router_balance(const spt_shape_t& s, const void* X, const float* logits,
                              const int32_t* offsets, float* loss, float* frac, float* dWr, float* dbr,
                              const BalanceWorkspace& w, hipStream_t st);

// Low-rank adapted variant.  Workspace = the forward / backward
// workspace followed by zero-padded 32-wide adapter panels and the small intermediates.
struct LoraWorkspace {
  FwdWorkspace fwd;
  BwdWorkspace bwd;
  uint16_t *A1T, *C1T, *C1P, *B2T, *B2P, *C2P;  // [32][d] [D][64] [32][D] [32][D] [D][64] [32][d]
  uint16_t *A1P, *C2T;                          // [d][32] [d][32]: K-contiguous forms for lora_expand
  uint16_t* Z;                                  // [T][d] bf16, narrow blocks: the low-rank term of an outer projection
  uint16_t *Upad, *Gpad;                        // [T][64] bf16 value | remainder: X A1, dY C2^T
  uint16_t *Upair, *Gpair;                      // [P][64] the same rows in sorted order (backward)
  uint16_t *Rb, *Vb;                            // [T][32] bf16 rounded token sums (backward)
  float *Sp, *Sp2;                              // [P][32] per pair
  float* stage[4];                              // gradient staging: [pieces][Bs][32] twice, [chunks][d][32] twice
  int32_t *p_first, *p_off;                     // buckets cut into pieces (PieceTable)
  int piece, chunk, nchunks;                    // rows of a piece / of a chunk of the tokens
  int max_pieces;
  size_t bytes;
};
LoraWorkspace plan_lora(const spt_shape_t& s, void* ws, bool backward);
hipError_t run_lora_fwd(const spt_shape_t& s, int r, const void* X, const void* W1, const void* W2,
                        const void* A1, const void* C1, const void* B2, const void* C2,
                        const int32_t* offsets, const int32_t* perm, const int32_t* inv, void* Y,
                        void* Hsave, const LoraWorkspace& w, hipStream_t st);
hipError_t run_lora_bwd(const spt_shape_t& s, int r, const void* X, const void* W1, const void* W2,
                        const void* A1, const void* C1, const void* B2, const void* C2, const void* dY,
                        const int32_t* offsets, const int32_t* perm, const int32_t* inv,
                        const void* Hsave, void* dX, float* dA1, float* dC1, float* dB2, float* dC2,
                        const LoraWorkspace& w, hipStream_t st);
// One zero-padded bf16 panel: dst[a][b] (drows x dcols) = transpose ? src[b'][a] : src[a][b'],
// b' = dup ? b % 32 : b, zero outside src (srows x scols).
struct PadJob {
  const uint16_t* src;
  int srows, scols, transpose, dup, frag;   // frag: in operand order, see lora_setup_kernel
  uint16_t* dst;
  int drows, dcols;
};
constexpr int kMaxPadJobs = 6;
struct PadJobs { PadJob job[kMaxPadJobs]; };
// Buckets cut into pieces of at most `piece` rows (see lora_setup_kernel).
struct PieceTable {
  const int32_t* offsets;
  int N, piece, max_pieces;
  int32_t *first, *off;
};
struct ProjJob {              // X A or dY C^T: [T][d] x panel [32][d]
  const uint16_t *act, *panel;
  uint16_t *by_token, *by_pair;   // [T][64], [P][64]; either may be null
};
struct PairJob {              // per pair: Hin [P][Bs] x panel [32][N*Bs]
  const uint16_t *hin, *panel;
  float* out;                 // [P][32]
};
// out[piece][u][rho] = sum over the piece's rows q of H[q][u] R[q][rho].
struct GradJob {
  const uint16_t *H, *R;      // [rows][units], [rows][ldr]
  float* out;                 // staging [npieces][units][ldo]
  const int32_t* off;         // piece boundaries; null: `piece` rows each, up to `rows`
  const int32_t* first;       // first piece of each block; null: all pieces belong to the one block
  float* result;
  int units, ldr, ldo, npieces, tiles, piece, rows, nblocks, transpose;   // tiles: ceil(units / 128)
};
struct GradJobs { GradJob job[4]; };
hipError_t lora_setup(const PadJobs& jobs, int njobs, const PieceTable* pieces, hipStream_t st);
hipError_t lora_proj(const ProjJob* jobs, int njobs, const int32_t* inv, int T, int d, int k, hipStream_t st);
hipError_t lora_pair_gemm(const PairJob* jobs, int njobs, bool narrow, const int32_t* offsets, int N, int Bs, int P,
                          hipStream_t st);
hipError_t lora_expand(const float* Sp, const uint16_t* panel, const int32_t* inv, int T, int d, int k,
                       const uint16_t* part, uint16_t* out, uint16_t* Sb, const float* Sp2, uint16_t* Sb2, hipStream_t st);
hipError_t lora_grads(const GradJobs& jobs, bool frag, int r, const uint16_t* zero_row, hipStream_t st);
hipError_t row_contraction(const GradJob& jb, const uint16_t* zero_row, hipStream_t st);
int grad_piece_rows(int64_t rows, int blocks, int units);

}  // namespace spt
