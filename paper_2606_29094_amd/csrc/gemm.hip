// NT GEMM on the gfx950 matrix cores: C[m][n] = sum_k A[m][k] * B[n][k],
// A [M, K] and B [N, K] both K-contiguous (activations x weights^T), fp32
// accumulation, with the work after the contraction fused into a tile
// epilogue:
//   * store fp32 (split-K partial slices),
//   * add into an fp32 residual stream,
//   * SwiGLU: gate and up columns computed in the same tile, silu(g) * u stored,
//   * fused LM head: per row, the online (max, sum of exp, lowest argmax) of the
//     scaled logits over the tile's vocabulary columns; logits are never stored,
//   * scaled fp32 store (test hook).
//
// Tiling: 256 threads (4 waves), block tile BM x BN, k-tile of 128 bytes per
// row (64 bf16 or 32 fp32), double-buffered in LDS with 16-byte row padding so
// that 16 lanes reading 16 rows hit distinct banks; global loads are 16-byte
// vectors, prefetched into registers one k-tile ahead. bf16 uses
// v_mfma_f32_16x16x32_bf16, fp32 uses v_mfma_f32_16x16x4_f32 (four per 16-byte
// fragment, the k order is the same permutation for A and B).
#include <algorithm>
#include <cmath>

#include "common.h"
#include "gemm_common.h"
#include "kernels.h"

namespace dlm {

// ---------------------------------------------------------------- kernel --
template <typename T, int BM, int BN, int WAVES_M, int WAVES_N, class Epi>
__global__ __launch_bounds__(256) void gemm_nt_kernel(
    const T* __restrict__ A, int lda, const T* __restrict__ B, int ldb,
    int M, int N, int K, int k_per_split, Epi epi) {
  static_assert(WAVES_M * WAVES_N == 4, "4 waves");
  constexpr int TM = BM / WAVES_M, TN = BN / WAVES_N;
  constexpr int FM = TM / 16, FN = TN / 16;
  constexpr int kVec = MfmaTraits<T>::kVec;
  constexpr int BK = kRowBytes / sizeof(T);
  constexpr int CHUNKS = (BM + BN) * (kRowBytes / 16);
  static_assert(CHUNKS % 256 == 0, "chunk split");
  constexpr int PER = CHUNKS / 256;
  constexpr int STAGE = (BM + BN) * kLdsRow;
  __shared__ __attribute__((aligned(16))) char smem[2 * STAGE];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WAVES_N, wn = wave % WAVES_N;
  const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
  if (epi.skip_tile(m0)) return;   // uniform over the block
  const int kbeg = blockIdx.z * k_per_split;
  const int kend = min(K, kbeg + k_per_split);
  const int nkt = kend > kbeg ? ceil_div(kend - kbeg, BK) : 0;

  // per-thread global source rows (fixed over k)
  const T* src[PER];
  bool row_ok[PER];
  int coff[PER];
#pragma unroll
  for (int p = 0; p < PER; ++p) {
    int c = tid + p * 256;
    int r = c >> 3;
    coff[p] = (c & 7) * kVec;
    if (r < BM) {
      int m = m0 + r;
      row_ok[p] = m < M;
      src[p] = A + (long)(row_ok[p] ? m : 0) * lda;
    } else {
      int n = n0 + r - BM;
      row_ok[p] = n < N;
      src[p] = B + (long)(row_ok[p] ? epi.b_row(n) : 0) * ldb;
    }
  }

  u32x4 reg[PER];
  auto gload = [&](int kt) {
    int kb = kbeg + kt * BK;
#pragma unroll
    for (int p = 0; p < PER; ++p) {
      int k = kb + coff[p];
      if (row_ok[p] && k < kend)
        reg[p] = *reinterpret_cast<const u32x4*>(src[p] + k);
      else
        reg[p] = u32x4{0u, 0u, 0u, 0u};
    }
  };
  auto sstore = [&](int buf) {
    char* s = smem + buf * STAGE;
#pragma unroll
    for (int p = 0; p < PER; ++p) {
      int c = tid + p * 256;
      *reinterpret_cast<u32x4*>(s + (c >> 3) * kLdsRow + (c & 7) * 16) = reg[p];
    }
  };

  f32x4 acc[FM][FN];
#pragma unroll
  for (int a = 0; a < FM; ++a)
#pragma unroll
    for (int b = 0; b < FN; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int arow = (wm * TM + (lane & 15)) * kLdsRow;
  const int brow = (BM + wn * TN + (lane & 15)) * kLdsRow;
  const int kq = (lane >> 4) * 16;

  if (nkt > 0) {
    gload(0);
    sstore(0);
  }
  __syncthreads();
  for (int kt = 0; kt < nkt; ++kt) {
    const int cur = kt & 1;
    if (kt + 1 < nkt) gload(kt + 1);
    const char* s = smem + cur * STAGE;
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      u32x4 af[FM], bfr[FN];
#pragma unroll
      for (int fm = 0; fm < FM; ++fm)
        af[fm] = *reinterpret_cast<const u32x4*>(s + arow + fm * 16 * kLdsRow + g * 64 + kq);
#pragma unroll
      for (int fn = 0; fn < FN; ++fn)
        bfr[fn] = *reinterpret_cast<const u32x4*>(s + brow + fn * 16 * kLdsRow + g * 64 + kq);
#pragma unroll
      for (int fm = 0; fm < FM; ++fm)
#pragma unroll
        for (int fn = 0; fn < FN; ++fn)
          acc[fm][fn] = MfmaTraits<T>::mma(af[fm], bfr[fn], acc[fm][fn]);
    }
    if (kt + 1 < nkt) sstore(cur ^ 1);
    __syncthreads();
  }
  epi(acc, m0 + wm * TM, n0 + wn * TN, lane, wn, smem, WAVES_N, BM, m0, (int)blockIdx.x,
      (int)blockIdx.z);
}

// fp32 launches of few tiles: a block of kSmallWaves waves computes a 16 x 32
// output tile, wave w multiplying the 16-wide k groups w, w + kSmallWaves, ...
// straight from global memory (both operands are cache-resident at these sizes
// and a block reads each fragment once, so LDS staging would only add barriers),
// and wave 0 sums the waves' partials in wave order before the epilogue. What
// bounds these launches is the serial walk over K, not bandwidth: with 128 rows
// the 128x128 tiles of the kernel above are 2 blocks for a 256-wide output (49
// us at K = 688) and 11 for the gate/up GEMM (24 us); these are 64 and 344
// blocks (6 and 7 us).
constexpr int kSmallWaves = 8;
template <class Epi>
__global__ __launch_bounds__(kSmallWaves * 64) void gemm_f32_small_kernel(
    const float* __restrict__ A, int lda, const float* __restrict__ B, int ldb, int M, int N,
    int K, Epi epi) {
  constexpr int FN = 2, UNR = 3;           // column fragments; k groups in flight per wave
  __shared__ f32x4 part[kSmallWaves][FN][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int n0 = blockIdx.x * 16 * FN, m0 = blockIdx.y * 16;
  // element e of a lane's fragment of k group c is k = 16 c + 4 (lane / 16) + e, for A and B alike
  const float* a = A + (long)min(m0 + (lane & 15), M - 1) * lda + 4 * (lane >> 4);
  const float* b[FN];
#pragma unroll
  for (int fn = 0; fn < FN; ++fn)
    b[fn] = B + (long)epi.b_row(min(n0 + 16 * fn + (lane & 15), N - 1)) * ldb + 4 * (lane >> 4);
  f32x4 acc[1][FN];
#pragma unroll
  for (int fn = 0; fn < FN; ++fn) acc[0][fn] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int nc = K / 16;
  for (int c0 = wave; c0 < nc; c0 += kSmallWaves * UNR) {
    f32x4 av[UNR], bv[UNR][FN];
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      const int c = min(c0 + u * kSmallWaves, nc - 1);   // past the end: loaded, not used
      av[u] = *reinterpret_cast<const f32x4*>(a + 16 * c);
#pragma unroll
      for (int fn = 0; fn < FN; ++fn) bv[u][fn] = *reinterpret_cast<const f32x4*>(b[fn] + 16 * c);
    }
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      if (c0 + u * kSmallWaves >= nc) break;
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int fn = 0; fn < FN; ++fn) acc[0][fn] = mfma16_f32(av[u][e], bv[u][fn][e], acc[0][fn]);
    }
  }
#pragma unroll
  for (int fn = 0; fn < FN; ++fn) part[wave][fn][lane] = acc[0][fn];
  __syncthreads();
  if (wave != 0) return;
#pragma unroll
  for (int fn = 0; fn < FN; ++fn)
#pragma unroll
    for (int w = 1; w < kSmallWaves; ++w) acc[0][fn] += part[w][fn][lane];
  epi(acc, m0, n0, lane, 0, nullptr, 1, 16, m0, (int)blockIdx.x, 0);
}

// --------------------------------------------------------------- launch --

// Register-staged kernel: any K that is a multiple of 16 bytes, fp32 or bf16.
template <typename T, class Epi>
static hipError_t launch_rs(const T* A, int lda, const T* B, int ldb, int M, int N, int K,
                            int splits, const Epi& epi, hipStream_t st) {
  if (M <= 0 || N <= 0) return hipSuccess;
  constexpr int BK = kRowBytes / sizeof(T);
  // split-K slices must tile K exactly: the consumers sum every slice
  if (splits < 1 || (splits > 1 && K % (splits * BK) != 0)) return hipErrorInvalidValue;
  const int kps = splits == 1 ? ceil_div(K, BK) * BK : K / splits;
  if (M <= 32) {
    dim3 g(ceil_div(N, 128), ceil_div(M, 32), splits);
    DLM_LAUNCH((gemm_nt_kernel<T, 32, 128, 1, 4, Epi>), g, dim3(256), 0, st,
                       A, lda, B, ldb, M, N, K, kps, epi);
  } else if (M <= 64) {
    dim3 g(ceil_div(N, 128), ceil_div(M, 64), splits);
    DLM_LAUNCH((gemm_nt_kernel<T, 64, 128, 2, 2, Epi>), g, dim3(256), 0, st,
                       A, lda, B, ldb, M, N, K, kps, epi);
  } else {
    dim3 g(ceil_div(N, 128), ceil_div(M, 128), splits);
    DLM_LAUNCH((gemm_nt_kernel<T, 128, 128, 2, 2, Epi>), g, dim3(256), 0, st,
                       A, lda, B, ldb, M, N, K, kps, epi);
  }
  return hipGetLastError();
}

template <typename T, class Epi>
static hipError_t launch(const GemmPlan& p, const T* A, int lda, const T* B, int ldb, int M,
                         int N, int K, const Epi& epi, hipStream_t st) {
  if constexpr (sizeof(T) == 2) {
    if (p.cfg >= 0)
      return gemm_dl_launch<Epi>(p.cfg, A, lda, B, ldb, M, N, K, p.splits, p.group_m,
                                 Epi::kTailSplit ? p.sub : 0, p.n_tail, epi, st);
  } else if constexpr (Epi::kWaveLocal) {
    if (p.cfg == kSmallF32 && M > 0 && N > 0) {
      if (K % 16 != 0 || p.splits != 1) return hipErrorInvalidValue;
      DLM_LAUNCH((gemm_f32_small_kernel<Epi>), dim3(ceil_div(N, 32), ceil_div(M, 16)),
                 dim3(kSmallWaves * 64), 0, st, A, lda, B, ldb, M, N, K, epi);
      return hipGetLastError();
    }
  }
  return launch_rs<T, Epi>(A, lda, B, ldb, M, N, K, p.splits, epi, st);
}

// Tile/split choice. bf16 with K a multiple of 64 uses the direct-load kernel.
// A configuration keeps `occ` blocks per CU resident. Its time is rounds x
// (time of one round at the block's k-tile count), the per-round times being
// medians of 757 launches measured on MI355X (the projection shapes of both
// model shapes at M = 256 .. 8192, every split, weights streamed from HBM),
// interpolated linearly in k-tiles (proportionally outside the measured range);
// a last, partly filled round of a multi-block configuration costs
// max(0.7, fill) of a full one. A last round that fills at most a quarter
// (half) of the CUs of a one-block-per-CU configuration may run its tiles as
// quarter (half) tiles, where the configuration has them: it then costs
// 0.55 (0.75) of a full round. These two factors minimise the summed measured
// time of the chosen plans over 56 projection shapes (both model shapes,
// 256 .. 7936 rows, every configuration with and without the split; 1.6 %
// below the plans without sub-tiles, within 0.1 % of the best measured plan
// of every shape; e.g. GQA QKV at 4096 rows 143 -> 130 us, gate/up 921 -> 894
// us, output projection at 5056 rows 165 -> 146 us). When K is split, the extra fp32 slices add
// the consumer's reads of them (their writes are inside the measured round
// times; charging both picked worse plans, e.g. 62 vs 52 us for the 512-row
// MHA QKV projection). The cheapest
// (configuration, split) wins. 128x192 with two blocks per CU (cfg 22) runs
// without K splits only (its table holds unsplit launches). Up to 1024 rows
// the model of kFewRowTiles applies instead. The eight-wave configurations run the split-phase tile
// form with a three-stage weight ring (6, 21, 70) or three stages of both
// operands (29); their tables are the ones measured for their two-ring form,
// each entry scaled by the time ratios of the forms measured at that k-tile
// count (full rounds: 0.94-0.98 from the split-phase loop, about 0.98-0.99
// more from the third weight stage; the 256x192 tile 0.93, measured at 256 to
// 6400 rows with the weights streamed from HBM); the three-stage 256x128 tile
// (29) takes the mean of the estimates from the tables of the two-ring
// 256x128 tiles it replaces (3- and 4-stage weight rings, scaled by
// 0.87-0.94 and 0.90-0.97).
namespace {
struct RoundTable {
  int cfg, occ;
  bool unsplit_only;
  int n;
  float kt[15], us[15];
  int min_kt = 0;          // used only for at least this many k-tiles per block
  int max_m = 1 << 30;     // and for at most this many rows
};
const RoundTable kRoundTables[] = {
    {6, 1, false, 15,
     {8, 14, 16, 24, 28, 32, 37, 48, 56, 64, 74, 96, 148, 192, 296},
     {23.9f, 28.5f, 33.9f, 48.5f, 45.5f, 55.0f, 70.8f, 81.0f, 84.3f, 100.1f, 122.4f, 141.7f, 213.1f, 263.3f, 398.9f}},
    {21, 1, false, 15,
     {8, 14, 16, 24, 28, 32, 37, 48, 56, 64, 74, 96, 148, 192, 296},
     {18.2f, 23.6f, 26.3f, 38.7f, 37.9f, 43.6f, 56.3f, 64.7f, 67.5f, 80.5f, 95.1f, 118.5f, 175.2f, 223.3f, 343.0f}},
    {22, 2, true, 4, {56, 64, 192, 296}, {81.9f, 93.1f, 282.1f, 435.5f}},
    {29, 1, false, 15,
     {8, 14, 16, 24, 28, 32, 37, 48, 56, 64, 74, 96, 148, 192, 296},
     {15.2f, 17.6f, 21.0f, 28.5f, 27.5f, 33.1f, 42.6f, 49.1f, 51.6f, 63.0f, 74.3f, 89.6f, 131.7f, 168.7f, 249.4f}},
    {42, 1, false, 15,
     {8, 14, 16, 24, 28, 32, 37, 48, 56, 64, 74, 96, 148, 192, 296},
     {14.6f, 18.1f, 20.7f, 29.2f, 27.6f, 32.4f, 41.1f, 47.7f, 47.8f, 56.8f, 70.6f, 80.0f, 124.7f, 154.4f, 232.9f}},
    // (LM head only: the projections of up to 1024 rows use the model below)
    {1, 2, false, 15,
     {8, 14, 16, 24, 28, 32, 37, 48, 56, 64, 74, 96, 148, 192, 296},
     {17.1f, 22.4f, 25.6f, 37.3f, 33.5f, 40.8f, 51.1f, 65.7f, 65.8f, 71.1f, 90.8f, 119.1f, 171.0f, 214.9f, 335.1f},
     0, 128},
    // 32x32x16 MFMA tiles: 256x128 with four 128x64-wave tiles, and 384x256
    // with eight 96x128-wave tiles (two waves per SIMD). Their round times
    // were measured against configurations 29 and 6 in the same runs (full
    // rounds, weights streamed from HBM) and scaled by those configurations'
    // tables above, so all tables share one measurement basis.
    {62, 1, false, 15,
     {8, 14, 16, 24, 28, 32, 37, 48, 56, 64, 74, 96, 148, 192, 296},
     {17.3f, 20.0f, 24.6f, 35.1f, 33.5f, 40.8f, 50.3f, 61.1f, 61.9f, 79.5f, 87.3f, 110.3f, 158.0f, 211.6f, 330.7f}},
    {65, 1, false, 15,
     {8, 14, 16, 24, 28, 32, 37, 48, 56, 64, 74, 96, 148, 192, 296},
     {37.4f, 46.5f, 57.2f, 79.0f, 73.6f, 88.7f, 118.5f, 131.5f, 126.5f, 156.3f, 204.0f, 238.4f, 360.9f, 430.0f, 679.5f},
     148},   // measured ahead only with long K walks (the GQA down projection); the
             // table overrates it at 56 k-tiles (4096-row output projection 145 vs 112 us)
    // 256x224: measured against configuration 6 in the same runs (one and two
    // full rounds per k-tile count) and scaled by that configuration's table;
    // a round takes 0.82-0.94 (mean 0.89) of a 256x256 round for 0.875 of its work
    {70, 1, false, 15,
     {8, 14, 16, 24, 28, 32, 37, 48, 56, 64, 74, 96, 148, 192, 296},
     {22.5f, 25.7f, 31.3f, 45.6f, 42.3f, 51.5f, 64.1f, 71.1f, 70.6f, 94.1f, 111.6f, 126.1f, 192.8f, 234.0f, 374.4f}},
};

// Launches of up to kFewRows (kernels.h) rows, mostly one round of blocks. Modelled
// time of a launch of `units` blocks that walk kt k-tiles each:
//   4.3 + sqrt(walk^2 + stream^2) + output bytes / 6.46 TB/s       (us), with
//   walk   = kt x rounds x us_kt, 27 % less where a tile holds no rows and 9 % less
//            where no blocks run (in proportion),
//   stream = the weights at 7.11 TB/s,
// both 5 % longer where the row tiles walk weight rows a power of two apart from
// the same k-tile (every block in step then reads the same HBM channels; the
// four-stage tiles with one row tile start each column tile elsewhere), and the
// consumer's reads of the extra K slices, 0.08 us + 0.25 a slice + 7.65 TB/s, with
// 0.03 us a MB for slices beyond the 32 MB of the L2s; within 1 % the fewer slices,
// which need less workspace.
// rounds: whole ones, also a last partly filled one, which in quarter (half) tiles
// counts 0.55 (0.75); 6 % more for five or more row tiles over two rounds or more
// (28672 x 4096 at 800 to 960 rows: 192 x 192 tiles 195-203 us, 256 x 256 175-186).
// Of configurations that fit twice on a CU (64 or 80 KB of LDS) a round of two blocks
// takes 1.6 times that of one, a last partly filled one at least 0.75 of it.
// The constants are fitted to the choice, not to the times: they minimise what the
// chosen plans took over 2300 shapes and row counts (18000 launches inside steps,
// MI355X, weights streamed from HBM; eight model shapes of 2048 to 8192 wide, 4 to
// 1024 rows, every projection with its consumer). Over those samples the chosen plans
// take 0.4 % longer than the best measured for the repository's two bf16 models and
// 0.8 to 2 % for the others; single launches are up to 10 % off. Tables of
// times by k-tile count, measured for the two models alone, chose as well for
// them and up to 28 % worse elsewhere (2048 x 2048 at 512 to 1024 rows, 15.9 / 19.6
// to 20.6 / 26.3 us).
struct FewRowTile {
  int cfg;
  float us_kt;
  int occ = 1;             // blocks that fit on a CU
};
const FewRowTile kFewRowTiles[] = {
    {80, 0.279f, 2}, {81, 0.357f, 2}, {82, 0.614f}, {83, 0.569f}, {84, 0.403f}, {85, 0.455f},
    {86, 0.640f}, {87, 0.520f}, {88, 0.617f}, {89, 0.652f}, {90, 0.778f}, {92, 0.678f},
    {93, 0.873f}, {22, 0.839f, 2}, {29, 0.807f}, {21, 1.163f}, {70, 1.266f}, {6, 1.378f},
};

// The parts that need no tile: fixed, output and slices (with the 1 %), in us.
double few_rows_base_us(int M, int N, int s, bool gate_up) {
  const double mb = (double)M * N * 4e-6;   // of a slice; gate/up stores half the columns in bf16
  const double us = 4.29 + (gate_up ? 0.25 : (double)s) * mb / 6.46;
  if (s == 1) return us;
  return 1.01 * (us + mb * (s - 1) / 7.65 + 0.079 + 0.251 * (s - 1) +
                 0.03 * std::max(0.0, mb * s - 32.0));
}

// A tile of kFewRowTiles with its dimensions.
struct FewRowDims {
  int cfg, bm, bn, stages, subs, occ;
  bool odd;
  double us_kt;
};
constexpr int kFewRowCount = sizeof(kFewRowTiles) / sizeof(kFewRowTiles[0]);
const FewRowDims* few_row_dims() {
  struct Dims {
    FewRowDims d[kFewRowCount];
    Dims() {
      for (int i = 0; i < kFewRowCount; ++i) {
        const FewRowTile& t = kFewRowTiles[i];
        FewRowDims& x = d[i];
        int th;
        gemm_dl_tile(t.cfg, &x.bm, &x.bn, &th);
        x.cfg = t.cfg, x.us_kt = t.us_kt, x.occ = t.occ;
        x.stages = gemm_dl_stages(t.cfg), x.odd = gemm_dl_odd(t.cfg) != 0;
        x.subs = t.occ == 1 ? gemm_dl_subs(t.cfg) : 0;
      }
    }
  };
  static const Dims dims;
  return dims.d;
}

double round_us(const RoundTable& t, double kt) {
  if (kt <= t.kt[0]) return t.us[0] * kt / t.kt[0];
  for (int i = 1; i < t.n; ++i)
    if (kt <= t.kt[i]) {
      const double w = (kt - t.kt[i - 1]) / (t.kt[i] - t.kt[i - 1]);
      return t.us[i - 1] + w * (t.us[i] - t.us[i - 1]);
    }
  return t.us[t.n - 1] * kt / t.kt[t.n - 1];
}

// Sub-tiles (0, 2 or 4 per tile) of a last round of rem tiles: quarters where they
// fill a quarter of the CUs at most, halves at a half, as the configuration allows.
int last_round_subs(int subs, long rem, long slots) {
  if (rem <= 0) return 0;
  if ((subs & 4) && 4 * rem <= slots) return 4;
  return (subs & 2) && 2 * rem <= slots ? 2 : 0;
}
}  // namespace

GemmPlan gemm_plan(int es, int M, int N, int K, bool splittable, int num_cu, bool allow_mf32,
                   bool allow_tail, bool allow_odd, int few_rows, bool allow_small) {
  GemmPlan best{-1, 1, 0};
  if (M <= 0 || N <= 0) return best;
  if (es != 2 || K % 64 != 0) {
    const int bm = M <= 32 ? 32 : (M <= 64 ? 64 : 128);
    const long tiles = (long)ceil_div(N, 128) * ceil_div(M, bm);
    // Small tiles where the staged kernel's leave half of the CUs idle. 1376 x 256 at
    // 1280, 1536 and 2048 rows (110, 132 and 176 staged tiles): staged 24.9, 25.4 and
    // 26.2 us, small 22.0, 25.7 and 31.7; 768 x 256 at 3072 and 3840 rows (144 and 180)
    // 26.5 and 27.3 against 26.7 and 33.2; 256 x 256 at 5120 (80) 33.2 against 21.1.
    // (16 MB: the weights it was measured with, 0.26-1.4 MB, and others that stay in
    // cache; larger ones stream, which the staged kernel's K split does)
    if (es == 4 && K % 16 == 0 && allow_small && 2 * tiles <= num_cu &&
        (long)N * K * es <= 16L << 20) {
      best.cfg = kSmallF32;
      return best;
    }
    if (splittable) {
      int s = 1;
      while (tiles * s < 2L * num_cu && K % (s * 2 * 64) == 0 && K / (s * 2) >= 512 && s < 8)
        s *= 2;
      best.splits = s;
    }
    return best;
  }
  double best_t = 1e30;
  if (M <= few_rows) {
    double base[9];
    for (int sp = 1; sp <= 8; sp *= 2) base[sp] = few_rows_base_us(M, N, sp, !splittable);
    const bool pow2 = (K & (K - 1)) == 0 && K >= 2048;
    const double stream0 = (double)N * K * 2e-6 / 7.11, inv_cu = 1.0 / num_cu;
    const FewRowDims* const tiles = few_row_dims();
    for (int i = 0; i < kFewRowCount; ++i) {
      const FewRowDims& c = tiles[i];
      if (!allow_odd && c.odd) continue;
      const int n_m = ceil_div(M, c.bm);
      if (c.bm < 192 && n_m > 5) continue;   // (the weights once per row tile)
      const double f = pow2 && !(n_m == 1 && c.stages == 4) ? 1.0 + 0.054 / n_m : 1.0;
      const double stream = stream0 * f;
      const double us_kt = c.us_kt * f * (1.0 - 0.27 * (1.0 - (double)M / ((double)n_m * c.bm)));
      const long n_tiles = (long)n_m * ceil_div(N, c.bn);
      for (int s = 1; s <= 8; s *= 2) {
        if (s > 1 && (!splittable || c.cfg == 22 || (K / 64) % s != 0 || K / s < 512)) continue;
        const double scale = s > 1 ? 1.01 : 1.0;
        if (base[s] + stream * scale >= best_t) break;   // (more slices only add to the base)
        const long units = n_tiles * s, full = units / num_cu, rem = units - full * num_cu;
        const int sub = allow_tail ? last_round_subs(c.subs, rem, num_cu) : 0;
        double rounds = (double)full;
        if (c.occ == 2) {
          const long pairs = full / 2, last = units - pairs * 2 * num_cu;
          rounds = pairs + (last == 0 ? 0.0 : pairs ? std::max(0.75, 0.5 * last * inv_cu) : 1.0);
          rounds = units <= num_cu ? 1.0 : 1.6 * rounds;
        } else {
          rounds += sub == 4 ? 0.55 : sub == 2 ? 0.75 : rem ? 1.0 : 0.0;
          if (n_m >= 5 && full >= 2) rounds *= 1.06;
        }
        const double walk = (K / 64 / s) * rounds * us_kt *
                            (1.0 - 0.093 * (1.0 - std::min(1.0, units * inv_cu)));
        if (base[s] + walk * scale >= best_t) continue;
        const double t = base[s] + std::sqrt(walk * walk + stream * stream) * scale;
        if (t < best_t * 0.999) {
          best_t = t;
          best = GemmPlan{c.cfg, s, 0, sub, sub ? (int)rem : 0};
        }
      }
    }
  }
  for (const RoundTable& c : kRoundTables) {
    if (M <= few_rows) break;
    if (M > c.max_m) continue;
    if (!allow_mf32 && gemm_dl_mfma(c.cfg) == 32) continue;
    if (!allow_odd && gemm_dl_odd(c.cfg)) continue;
    int bm, bn, th;
    gemm_dl_tile(c.cfg, &bm, &bn, &th);
    for (int s = 1; s <= 8; s *= 2) {
      if (s > 1 && (c.unsplit_only || !splittable || (K / 64) % s != 0 || K / s < 512)) continue;
      if (K / 64 / s < c.min_kt) continue;
      const long units = (long)ceil_div(M, bm) * ceil_div(N, bn) * s;
      const long slots = (long)num_cu * c.occ;
      const long full = units / slots;
      const long rem = units - full * slots;
      const double fill = (double)rem / slots;
      const int sub = allow_tail && c.occ == 1 ? last_round_subs(gemm_dl_subs(c.cfg), rem, slots) : 0;
      double rounds = (double)full;
      if (sub)
        rounds += sub == 4 ? 0.55 : 0.75;
      else if (rem > 0)
        rounds += c.occ > 1 ? std::max(0.7, fill) : 1.0;
      double t = rounds * round_us(c, (double)(K / s) / 64.0);
      if (s > 1) t += (double)M * N * 4.0 * (s - 1) / 5.0e12 * 1e6;   // the consumer's reads
      if (t < best_t * 0.999) {
        best_t = t;
        best = GemmPlan{c.cfg, s, 0, sub, sub ? (int)rem : 0};
      }
    }
  }
  // weights larger than the last-level cache (256 MB Infinity Cache) stream
  // from HBM once per row tile in plain order: use the grouped XCD order
  int bm, bn, th;
  if (best.cfg >= 0 && gemm_dl_tile(best.cfg, &bm, &bn, &th) && ceil_div(M, bm) > 1 &&
      (double)N * K * es > 256e6)
    best.group_m = 8;
  return best;
}

// The LM head at <= 64 rows streams the vocab matrix once and is bound by HBM,
// not by the round-time tables: measured with the rotated K walk, a weight row
// pitch that is a multiple of 8 KB (the 4096-wide MHA head) runs best with the
// 3-stage 64x128 tiles (two weight tiles in flight per block, 5.9 TB/s), other
// pitches (the 3584-wide GQA head) with the 2-stage ones (three blocks per CU,
// 5.8 TB/s).
GemmPlan lm_head_plan(int es, int M, int V, int K, int num_cu) {
  // the head's epilogue is 16x16 and keeps whole tiles (its partial results are per column tile)
  // It also runs many rounds at any row count, so the few-row model (one
  // round) does not describe it.
  GemmPlan p = gemm_plan(es, M, V, K, false, num_cu, false, false, false, 0, false);
  if (p.cfg >= 0 && M <= 64) p = GemmPlan{((long)K * es) % 8192 == 0 ? 11 : 10, 1, 0};
  // The head is planned for its largest row count and skips, on the device,
  // the row tiles beyond the rows that need a prediction. The grouped order
  // must then span every row tile in one group: with several groups, the
  // XCDs that receive the later groups' ranges would only hold skipped tiles
  // (half the XCDs idle with two groups).
  int bm, bn, th;
  if (p.group_m > 0 && gemm_dl_tile(p.cfg, &bm, &bn, &th)) p.group_m = ceil_div(M, bm);
  // over several row tiles, walk only the tiles of the rows that need a prediction
  if (p.cfg >= 0 && gemm_dl_tile(p.cfg, &bm, &bn, &th) && ceil_div(M, bm) > 1)
    p.active_cus = num_cu;
  return p;
}

template <typename T>
hipError_t gemm_store_f32(const GemmPlan& p, const T* A, int lda, const T* B, int ldb, int M,
                          int N, int K, float* C, int ldc, hipStream_t st) {
  EpiStore e{C, ldc, (long)M * ldc, M, N};
  return launch<T>(p, A, lda, B, ldb, M, N, K, e, st);
}

template <typename T>
hipError_t gemm_add_f32(const GemmPlan& p, const T* A, int lda, const T* B, int ldb, int M, int N,
                        int K, float* C, int ldc, hipStream_t st) {
  if (p.splits != 1) return hipErrorInvalidValue;
  EpiAdd e{C, ldc, M, N};
  return launch<T>(p, A, lda, B, ldb, M, N, K, e, st);
}

template <typename T>
hipError_t gemm_scaled_f32(const GemmPlan& p, const T* A, int lda, const T* B, int ldb, int M,
                           int N, int K, float scale, float* C, int ldc, hipStream_t st) {
  if (p.splits != 1) return hipErrorInvalidValue;
  EpiScaledStore e{C, ldc, M, N, scale};
  return launch<T>(p, A, lda, B, ldb, M, N, K, e, st);
}

template <typename T>
hipError_t gemm_swiglu(const GemmPlan& p, const T* A, int lda, const T* W, int ldw, int M, int F,
                       int K, T* out, int ldo, hipStream_t st) {
  if (p.splits != 1) return hipErrorInvalidValue;
  // 32x32 tiles interleave gate and up columns in groups of 32
  if (p.cfg >= 0 && gemm_dl_mfma(p.cfg) == 32 && F % 32 != 0) return hipErrorInvalidValue;
  EpiSwiGLU<T> e{out, ldo, M, F};
  return launch<T>(p, A, lda, W, ldw, M, 2 * F, K, e, st);
}

hipError_t gemm_debug_launch(int cfg, int epilogue, int sub, int n_tail, int group_m,
                             int splits, const bf16* A, const bf16* B, void* C, int M, int N,
                             int K, hipStream_t st) {
  if (epilogue == 0) {
    EpiStore e{reinterpret_cast<float*>(C), N, (long)M * N, M, N};
    return gemm_dl_launch<EpiStore>(cfg, A, K, B, K, M, N, K, splits, group_m, sub, n_tail, e,
                                    st);
  }
  if (splits != 1) return hipErrorInvalidValue;
  if (epilogue == 1) {
    EpiSwiGLU<bf16> e{reinterpret_cast<bf16*>(C), N / 2, M, N / 2};
    return gemm_dl_launch<EpiSwiGLU<bf16>>(cfg, A, K, B, K, M, N, K, 1, group_m, sub, n_tail, e,
                                           st);
  }
  if (epilogue == 2) {
    EpiAdd e{reinterpret_cast<float*>(C), N, M, N};
    return gemm_dl_launch<EpiAdd>(cfg, A, K, B, K, M, N, K, 1, group_m, sub, n_tail, e, st);
  }
  return hipErrorInvalidValue;
}

int lm_head_tiles(const GemmPlan& p, int V) {
  int bm = 128, bn = 128, th = 256;
  if (p.cfg >= 0) gemm_dl_tile(p.cfg, &bm, &bn, &th);
  return ceil_div(V, bn);
}

template <typename T>
hipError_t gemm_lm_head(const GemmPlan& p, const T* U, int ldu, const T* W, int M, int V, int K,
                        float inv_tau, float* pm, float* ps, int* pi, int ld,
                        const int* m_count, hipStream_t st) {
  if (p.splits != 1) return hipErrorInvalidValue;
  EpiLMHead e{pm, ps, pi, M, V, inv_tau, ld, m_count};
  if constexpr (sizeof(T) == 2) {
    if (p.cfg >= 0 && p.active_cus > 0)
      return gemm_dl_head_launch(p.cfg, U, ldu, W, K, M, V, K, p.active_cus, e, st);
  }
  return launch<T>(p, U, ldu, W, K, M, V, K, e, st);
}

#define INST(T)                                                                                \
  template hipError_t gemm_store_f32<T>(const GemmPlan&, const T*, int, const T*, int, int, int, \
                                        int, float*, int, hipStream_t);                         \
  template hipError_t gemm_add_f32<T>(const GemmPlan&, const T*, int, const T*, int, int, int,   \
                                      int, float*, int, hipStream_t);                           \
  template hipError_t gemm_scaled_f32<T>(const GemmPlan&, const T*, int, const T*, int, int,     \
                                         int, int, float, float*, int, hipStream_t);            \
  template hipError_t gemm_swiglu<T>(const GemmPlan&, const T*, int, const T*, int, int, int,    \
                                     int, T*, int, hipStream_t);                                \
  template hipError_t gemm_lm_head<T>(const GemmPlan&, const T*, int, const T*, int, int, int,   \
                                      float, float*, float*, int*, int, const int*, hipStream_t);
INST(bf16)
INST(float)

}  // namespace dlm
