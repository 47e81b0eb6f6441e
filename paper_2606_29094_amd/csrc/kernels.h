// Launch functions of the denoising-step kernels (internal to libdlm.so).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dlm {

constexpr int kMaxReq = 64;
constexpr int kMaxBlock = 64;
constexpr int kNStats = 8;      // confidence statistics per request
constexpr int kQTile = 64;      // rows per RoPE tile

// Per-request plan of one step, passed by value as a kernel argument.
struct ReqPlan {
  int row0;      // first packed recompute row
  int nrows;     // recompute rows
  int pos0;      // position of the first recompute row
  int seq_len;   // keys attended (all positions of the slot)
  int prompt_len;
  int slot;
  int tok_off;   // offset of position 0 in tokens/mask
  int blk_s;     // active block [blk_s, blk_s + blk_len)
  int blk_len;
  int tile0;     // first tile of this request (kQTile rows; the attention launches number their own)
  int blk0;      // offset of this request's block rows in the packed block-row order
  float gamma;   // threshold
};
struct StepPlan {
  int n_req;
  int n_rows;    // total recompute rows N
  int n_tiles;   // total tiles
  int n_blk;     // total block rows
  ReqPlan r[kMaxReq];
};

// Request of a packed row or of a tile (tiles numbered request by request,
// ReqPlan::tile0). Every lane of the wave must be active. Lane l looks at request l
// and a ballot counts those that start at or before the row (a walk over 64 requests
// of 64 rows is 64 dependent loads at the start of each block: RoPE and key/value
// write 34 us against 20, attention 123 against 117). One request needs no look-up:
// the load and the ballot cost its launches 0.3-0.5 us (512 rows of 32 heads, RoPE
// 11.6 / 11.3, attention 15.5 / 14.9); a scalar walk for up to 3, 4 or 8 requests was
// no faster than the ballot (RoPE of 3 x 64 rows 7.6 / 7.3, of 8 x 64 13.3 / 11.8).
static_assert(kMaxReq <= 64, "one lane per request");
__device__ __forceinline__ int plan_req_at(const StepPlan& p, int ReqPlan::*start, int at) {
  if (p.n_req == 1) return 0;
  const int lane = threadIdx.x & 63;
  return __popcll(__ballot(lane < p.n_req && p.r[lane].*start <= at)) - 1;
}
__device__ __forceinline__ int plan_req_of_row(const StepPlan& p, int row) {
  return plan_req_at(p, &ReqPlan::row0, row);
}
__device__ __forceinline__ int plan_req_of_tile(const StepPlan& p, int tile) {
  return plan_req_at(p, &ReqPlan::tile0, tile);
}
// The same plan with its tiles numbered for another tile height, tiles(nrows) of each
// request. (Filled on the host: a prefix sum over the lanes in every block took 0.3-0.6
// us more, e.g. 64 rows over 1024 keys of 28/4 heads 9.4 / 8.8 us.)
template <class F>
inline StepPlan plan_with_tiles(const StepPlan& p, F tiles) {
  StepPlan t = p;
  t.n_tiles = 0;
  for (int r = 0; r < t.n_req; ++r) {
    t.r[r].tile0 = t.n_tiles;
    t.n_tiles += tiles(t.r[r].nrows);
  }
  return t;
}

// ---- GEMM family (gemm.hip, gemm_dl.hip) ----
// cfg >= 0: a direct-load tile configuration (bf16); cfg < 0: register-staged
// kernel (kSmallF32: the small-tile fp32 kernel). splits: number of K slices (fp32 partial slices, summed by the consumer).
// group_m: tile order (0 = plain); sub, n_tail: the last n_tail tiles of the
// order are each run as `sub` (2 or 4) sub-tiles (0: none); active_cus > 0
// (LM head over several row tiles only): one launch of blocks on that many
// CUs that walk the tiles of the rows needing a prediction (see
// gemm_dl_head_launch) instead of one block per tile
struct GemmPlan { int cfg; int splits; int group_m; int sub = 0; int n_tail = 0; int active_cus = 0; };
// allow_mf32: configurations with 32x32x16 MFMA tiles may be chosen (their
// epilogues exist for the plain, residual-add and SwiGLU stores; SwiGLU needs
// d_ffn % 32 == 0)
// direct-load bf16 kernel: one launch of configuration cfg; its output tile,
// MFMA shape and the sub-tile splits it allows (bit 1: halves, bit 2: quarters)
template <class Epi>
hipError_t gemm_dl_launch(int cfg, const bf16* A, int lda, const bf16* B, int ldb, int M, int N,
                          int K, int splits, int group_m, int sub, int n_tail, const Epi& epi,
                          hipStream_t st);
struct EpiLMHead;
// LM head whose row count is known only on the device (epi.m_count): as many
// blocks as fit on num_cu CUs, each XCD's blocks walking the tiles of its
// contiguous range of column tiles whose rows lie below the count
hipError_t gemm_dl_head_launch(int cfg, const bf16* A, int lda, const bf16* B, int ldb, int M,
                               int N, int K, int num_cu, const EpiLMHead& epi, hipStream_t st);
int gemm_dl_tile(int cfg, int* bm, int* bn, int* threads);
int gemm_dl_mfma(int cfg);
int gemm_dl_subs(int cfg);
int gemm_dl_odd(int cfg);
int gemm_dl_stages(int cfg);
// one launch of configuration cfg with epilogue 0 (fp32 store of `splits` K
// slices), 1 (SwiGLU to bf16, N = 2 F) or 2 (fp32 add), A [M, K], B [N, K],
// C row-major (test hook)
hipError_t gemm_debug_launch(int cfg, int epilogue, int sub, int n_tail, int group_m,
                             int splits, const bf16* A, const bf16* B, void* C, int M, int N,
                             int K, hipStream_t st);
// allow_tail: the last round may be split into sub-tiles (epilogues that allow it)
// allow_odd: configurations whose wave tiles hold an odd number of column
// fragments may be chosen (every epilogue but SwiGLU)
// few_rows: launches of up to that many rows are planned by the few-row model
constexpr int kFewRows = 1024;
// allow_small: fp32 launches whose 128-wide tiles would not fill the CUs may use
// the 16x32-tile kernel (plan cfg kSmallF32; every epilogue that needs only its
// own wave)
constexpr int kSmallF32 = -2;
GemmPlan gemm_plan(int elem_bytes, int M, int N, int K, bool splittable, int num_cu,
                   bool allow_mf32 = true, bool allow_tail = true, bool allow_odd = true,
                   int few_rows = kFewRows, bool allow_small = true);
// plan of the LM-head GEMM (M rows x V vocab entries)
GemmPlan lm_head_plan(int elem_bytes, int M, int V, int K, int num_cu);
template <typename T>
hipError_t gemm_store_f32(const GemmPlan& p, const T* A, int lda, const T* B, int ldb, int M,
                          int N, int K, float* C, int ldc, hipStream_t st);
template <typename T>
hipError_t gemm_add_f32(const GemmPlan& p, const T* A, int lda, const T* B, int ldb, int M, int N,
                        int K, float* C, int ldc, hipStream_t st);
template <typename T>
hipError_t gemm_scaled_f32(const GemmPlan& p, const T* A, int lda, const T* B, int ldb, int M,
                           int N, int K, float scale, float* C, int ldc, hipStream_t st);
template <typename T>
hipError_t gemm_swiglu(const GemmPlan& p, const T* A, int lda, const T* W, int ldw, int M, int F,
                       int K, T* out, int ldo, hipStream_t st);
int lm_head_tiles(const GemmPlan& p, int V);
template <typename T>
hipError_t gemm_lm_head(const GemmPlan& p, const T* U, int ldu, const T* W, int M, int V, int K,
                        float inv_tau, float* pm, float* ps, int* pi, int ld,
                        const int* m_count, hipStream_t st);

// ---- per-row kernels (rowwise.hip) ----
// the step's first kernel: h = embedding rows, out = rmsnorm(h) * g, cs = rotary table
template <typename T>
hipError_t embed_norm_rows(const StepPlan& p, const T* E, int d, int vocab, int mask_id,
                           const int32_t* tokens, const uint8_t* mask, const float* g, float eps,
                           int head_dim, float theta, float* h, T* out, float2* cs,
                           hipStream_t st);
template <typename T>
hipError_t rmsnorm_rows(const float* h, const float* g, int n, int d, float eps, T* out,
                        hipStream_t st);
// h[n] += sum of split-K slices (part may be null), then out = rmsnorm(h) (out may be null)
template <typename T>
hipError_t add_rmsnorm_rows(float* h, const float* part, int splits, long stride, const float* g,
                            int n, int d, float eps, T* out, hipStream_t st);
template <typename T>
hipError_t qkv_rope_scatter(const StepPlan& p, const float* qkv, int splits, long split_stride,
                            const float2* cs, int hq, int hkv, int dh, T* q_out,
                            T* kcache, T* vcache, int s_max, hipStream_t st);
hipError_t lm_select_rows(const StepPlan& p, const uint8_t* mask, int all_rows, int* lm_rows,
                          int* lm_count, int* req_lm_off, int* req_lm_cnt, hipStream_t st);
template <typename T>
hipError_t final_norm_gather(const float* h, const float* g, const int* lm_rows,
                             const int* lm_count, int m_max, int d, float eps, T* u,
                             hipStream_t st);
// lm_count: device-side number of rows (nullptr: m_max)
hipError_t lm_combine(const float* pm, const float* ps, const int* pi, int tiles, int ld,
                      const int* lm_count, int m_max, float* conf, int* tok, hipStream_t st);
hipError_t unmask_select(const StepPlan& p, const float* conf, const int* tok,
                         const int* req_lm_off, int32_t* tokens, uint8_t* mask,
                         int32_t* n_unmasked, int32_t* out_pos, int32_t* out_tok,
                         float* out_conf, float* blk_conf, int32_t* blk_tok, float* tok_conf,
                         float* stats, hipStream_t st);

// ---- attention (attention.hip) ----
// Kernels of a bf16 launch: shared tiles in blocks of eight or four waves; one query
// head per block with 32 rows and four key groups, 64 and two, 32 and two (the
// four-wave blocks for head_dim 64 only). splits > 1 (kAttnShared): every block takes
// one of that many key ranges and leaves its partial in scratch; attention_merge
// then writes out. attention_plan keeps the partials of the step within
// scratch_bytes (16-byte aligned; splits 1: scratch is not used). fp32: one kernel.
enum AttnKernel { kAttnShared, kAttnShared4, kAttnHead32x4, kAttnHead64x2, kAttnHead32x2 };
struct AttnPlan { AttnKernel kernel = kAttnShared; int splits = 1; };
AttnPlan attention_plan(const StepPlan& p, int hq, int hkv, int dh, size_t elem,
                        size_t scratch_bytes, int num_cu);
template <typename T>
hipError_t attention(const StepPlan& p, const T* q, const T* kcache, const T* vcache,
                     int s_max, int hq, int hkv, int dh, T* out, AttnPlan plan, float* scratch,
                     hipStream_t st);
hipError_t attention_merge(const StepPlan& p, int hq, int dh, int splits, const float* scratch,
                           bf16* out, hipStream_t st);

}  // namespace dlm
