// Bidirectional (non-causal) attention of the recomputed query rows over every
// cached key/value position of their request's slot: O = softmax(Q K^T /
// sqrt(dh)) V per query head; query head h reads key/value head h / (Hq/Hkv).
//
// bf16 path (matrix cores), two kernels:
//  * attn_gqa_kernel (shared tiles): one block = eight (16 query rows, query
//    head) groups that read one key/value head of one request; 64-key tiles
//    loaded directly into a two-stage LDS ring. For few blocks over long
//    sequences the keys are split over blocks, whose partials attn_merge_kernel
//    adds.
//  * attn_bf16_kernel (per head): one block = 32 or 64 query rows of one request
//    x one query head; waves split the rows in groups of 16 and the keys in
//    four or two groups, tiles staged through registers. Used for launches with
//    few blocks that a key split does not pay for.
//  attention_plan chooses.
// Key tiles are staged in LDS keys row-major and values transposed, which is
// how the cache stores them.
// Each wave computes S^T = K Q^T with v_mfma_f32_16x16x32_bf16 (keys as the A
// operand, its 16 query rows as B, held in registers), so that every lane
// ends up owning one query and 16 keys: the online softmax needs only two
// cross-lane steps, and the probabilities feed O^T = V^T P^T directly as the B
// operand (the key order inside the 32-wide k step is permuted identically in
// A and B, which leaves the sum unchanged). fp32 softmax, exp2 with the scale
// folded in; P enters the PV product as the sum of two bf16 terms (about 16
// significant bits), the output is rounded to bf16.
//
// fp32 path: attn_f32_kernel, on v_mfma_f32_16x16x4_f32; it serves the small
// fp32 model.
#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace dlm {

// P split into hi + lo bf16 terms (p = hi + lo to about 16 significant bits)
// for the eight probabilities a lane feeds one PV MFMA: lo = bf16(p - hi),
// converted two at a time (one packed conversion per pair for each term)
__device__ __forceinline__ void split_p8(const f32x4& a, const f32x4& b, bf16x8& ph, bf16x8& pl) {
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  typedef float f32x2_t __attribute__((ext_vector_type(2)));
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const f32x2_t v = e < 2 ? f32x2_t{a[2 * e], a[2 * e + 1]} : f32x2_t{b[2 * e - 4], b[2 * e - 3]};
    const bf16x2_t h = __builtin_convertvector(v, bf16x2_t);
    const bf16x2_t l = __builtin_convertvector(v - __builtin_convertvector(h, f32x2_t), bf16x2_t);
    ph[2 * e] = h[0];
    ph[2 * e + 1] = h[1];
    pl[2 * e] = l[0];
    pl[2 * e + 1] = l[1];
  }
}


// Wave layout: QG query groups of 16 rows x KG key groups. A block stages
// key tiles of 64 * KG positions; key group kg works on keys [64 kg, 64 kg +
// 64) of each tile. Each wave keeps its own online-softmax state; the key
// groups are merged in LDS at the end (rescaling by the group maxima), so the
// result is the same softmax over all keys.
//
// Softmax bookkeeping per query: m is a reference maximum of the raw scores,
// l and O^T are kept relative to 2^((s - m) c) with c = log2(e) / sqrt(dh).
// m is only moved (and l, O^T rescaled) when a tile's maximum exceeds it by
// more than 8 / c, so the weights stay below 2^8 and most tiles skip the
// rescale; the normalised result is the same.
// P is fed to the PV product as two bf16 terms (P = P_hi + P_lo, about
// 16 significant bits, two MFMAs per block) instead of one.
template <int DH, int QG, int KG>
__global__ __launch_bounds__(QG* KG * 64) void attn_bf16_kernel(StepPlan p, const bf16* __restrict__ q,
                                                               const bf16* __restrict__ kc,
                                                               const bf16* __restrict__ vc,
                                                               int s_max, int hq, int hkv,
                                                               bf16* __restrict__ out,
                                                               float scale_log2) {
  constexpr int NT = QG * KG * 64;
  constexpr int QT = 16 * QG;             // query rows per block
  constexpr int SK = 64 * KG;             // keys per staged tile
  constexpr int KS = DH + 8;              // K tile row stride (elements)
  constexpr int VS = SK + 8;              // V^T tile row stride (elements)
  constexpr int NDB = DH / 16;            // output dh blocks
  constexpr int NKS = DH / 32;            // k steps of S
  __shared__ __attribute__((aligned(16))) bf16 ks[SK * KS];
  __shared__ __attribute__((aligned(16))) bf16 vs[DH * VS];

  // head-major grid: consecutive blocks (spread over the XCDs round-robin) are
  // different heads, so the query tiles of one head share one XCD's L2
  const int h = blockIdx.x, tile = blockIdx.y;
  const ReqPlan& rq = p.r[plan_req_of_tile(p, tile)];
  const int lrow0 = (tile - rq.tile0) * QT;
  const int nvalid = min(QT, rq.nrows - lrow0);
  const int L = rq.seq_len;
  const int kvh = h / (hq / hkv);
  const bf16* kb = kc + ((long)(rq.slot * hkv + kvh) * s_max) * DH;
  const bf16* vb = vc + ((long)(rq.slot * hkv + kvh) * DH) * s_max;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int qg = wave % QG, kg = wave / QG;
  const int qr = qg * 16 + (lane & 15);           // query row of this lane in the tile
  const bool q_ok = qr < nvalid;
  const long qrow = rq.row0 + lrow0 + qr;
  const int g = lane >> 4;

  // Q fragments (B operand): col = query lane&15, k = dh 32*s + 8*g .. +7
  u32x4 qf[NKS];
#pragma unroll
  for (int s = 0; s < NKS; ++s) {
    if (q_ok)
      qf[s] = *reinterpret_cast<const u32x4*>(q + qrow * hq * DH + h * DH + s * 32 + g * 8);
    else
      qf[s] = u32x4{0u, 0u, 0u, 0u};
  }

  f32x4 o[NDB];
#pragma unroll
  for (int i = 0; i < NDB; ++i) o[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_ref = -INFINITY, l_run = 0.f;

  // K/V^T tiles go through registers: the next tile's global loads are issued
  // before the current tile's MFMAs and written to LDS after them.
  constexpr int KCH = SK * (DH / 8) / NT;   // 16-byte K chunks per thread
  constexpr int VCH = DH * (SK / 8) / NT;   // 16-byte V^T chunks per thread
  static_assert(KCH * NT == SK * (DH / 8) && VCH * NT == DH * (SK / 8), "tile split");
  u32x4 kreg[KCH], vreg[VCH];
  auto load_tile = [&](int key0) {
    if (key0 + SK <= L) {                       // whole tile inside the sequence
#pragma unroll
      for (int i = 0; i < KCH; ++i) {
        const int c = tid + i * NT;
        kreg[i] = *reinterpret_cast<const u32x4*>(kb + (long)(key0 + c / (DH / 8)) * DH +
                                                  (c % (DH / 8)) * 8);
      }
#pragma unroll
      for (int i = 0; i < VCH; ++i) {
        const int c = tid + i * NT;
        vreg[i] = *reinterpret_cast<const u32x4*>(vb + (long)(c / (SK / 8)) * s_max + key0 +
                                                  (c % (SK / 8)) * 8);
      }
    } else {
      // last tile: keys >= L read as zero. A V^T chunk starting below L lies
      // inside the slot (L <= s_max, both chunk start and s_max multiples of
      // 8); its values at keys >= L are cleared.
#pragma unroll
      for (int i = 0; i < KCH; ++i) {
        const int c = tid + i * NT;
        const int kk = key0 + c / (DH / 8);
        kreg[i] = kk < L ? *reinterpret_cast<const u32x4*>(kb + (long)kk * DH + (c % (DH / 8)) * 8)
                         : u32x4{0u, 0u, 0u, 0u};
      }
#pragma unroll
      for (int i = 0; i < VCH; ++i) {
        const int c = tid + i * NT;
        const int kk0 = key0 + (c % (SK / 8)) * 8;
        u32x4 v = u32x4{0u, 0u, 0u, 0u};
        if (kk0 < L) {
          v = *reinterpret_cast<const u32x4*>(vb + (long)(c / (SK / 8)) * s_max + kk0);
          const int n = L - kk0;                // valid keys in this chunk (> 0)
#pragma unroll
          for (int w = 0; w < 4; ++w) {
            const uint32_t keep = (2 * w < n ? 0x0000ffffu : 0u) | (2 * w + 1 < n ? 0xffff0000u : 0u);
            v[w] &= keep;
          }
        }
        vreg[i] = v;
      }
    }
  };
  // K rows are stored in the permuted key order of the shared-tile kernel:
  // inside each group of 32 keys, key 8 g + 4 h + i goes to row 16 h + 4 g + i
  // (h < 2, g < 4, i < 4), so the S^T values lane group g owns are the keys
  // 8 g .. 8 g + 7 of each 32-key group and V^T is read as one 16-byte chunk
  // per lane
  auto store_tile = [&]() {
#pragma unroll
    for (int i = 0; i < KCH; ++i) {
      const int c = tid + i * NT;
      const int k = c / (DH / 8);
      const int row = (k & ~31) | (((k >> 2) & 1) << 4) | (((k >> 3) & 3) << 2) | (k & 3);
      *reinterpret_cast<u32x4*>(ks + row * KS + (c % (DH / 8)) * 8) = kreg[i];
    }
#pragma unroll
    for (int i = 0; i < VCH; ++i) {
      const int c = tid + i * NT;
      *reinterpret_cast<u32x4*>(vs + (c / (SK / 8)) * VS + (c % (SK / 8)) * 8) = vreg[i];
    }
  };

  const int ntiles = ceil_div(L, SK);
  load_tile(0);
  store_tile();
  __syncthreads();
  for (int t = 0; t < ntiles; ++t) {
    const int key0 = t * SK + kg * 64;          // this wave's 64 keys
    if (t + 1 < ntiles) load_tile((t + 1) * SK);
    const bf16* ksg = ks + kg * 64 * KS;

    // S^T blocks: sblk[kb][i] = raw score(key = key0 + 32 (kb / 2) + 8 g + 4 (kb % 2) + i,
    // query = lane&15)
    f32x4 sblk[4];
#pragma unroll
    for (int kbk = 0; kbk < 4; ++kbk) {
      f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < NKS; ++s) {
        const u32x4 a = *reinterpret_cast<const u32x4*>(ksg + (kbk * 16 + (lane & 15)) * KS + s * 32 + g * 8);
        acc = mfma16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, qf[s]), acc);
      }
      sblk[kbk] = acc;
    }
    if (t == ntiles - 1) {                      // keys beyond L only in the last tile
#pragma unroll
      for (int kbk = 0; kbk < 4; ++kbk)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (key0 + 32 * (kbk >> 1) + 8 * g + 4 * (kbk & 1) + i >= L) sblk[kbk][i] = -INFINITY;
    }
    float mt = -INFINITY;
#pragma unroll
    for (int kbk = 0; kbk < 4; ++kbk)
#pragma unroll
      for (int i = 0; i < 4; ++i) mt = fmaxf(mt, sblk[kbk][i]);
    mt = fmaxf(mt, __shfl_xor(mt, 16, 64));
    mt = fmaxf(mt, __shfl_xor(mt, 32, 64));
    // move the reference maximum only on a large increase (false while both
    // are -inf: a key group that has seen no key below L yet)
    const bool grow = (mt - m_ref) * scale_log2 > 8.0f;
    if (__builtin_amdgcn_ballot_w64(grow)) {
      const float alpha = grow ? __builtin_amdgcn_exp2f((m_ref - mt) * scale_log2) : 1.0f;
      if (grow) m_ref = mt;
      l_run *= alpha;
#pragma unroll
      for (int i = 0; i < NDB; ++i) o[i] *= alpha;
    }
    const float nm = m_ref == -INFINITY ? 0.0f : -m_ref * scale_log2;
    float lsum = 0.f;
#pragma unroll
    for (int kbk = 0; kbk < 4; ++kbk)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float e = __builtin_amdgcn_exp2f(fmaf(sblk[kbk][i], scale_log2, nm));
        sblk[kbk][i] = e;
        lsum += e;
      }
    l_run += lsum;

    // O^T += V^T P^T over two 32-key steps; B operand slot 8g+e <-> key
    // 32*j + 8g + e (sblk[2j] holds keys 8g..8g+3, sblk[2j+1] keys 8g+4..8g+7)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      bf16x8 ph, pl;
      split_p8(sblk[2 * j], sblk[2 * j + 1], ph, pl);
#pragma unroll
      for (int db = 0; db < NDB; ++db) {
        const bf16* vrow = vs + (db * 16 + (lane & 15)) * VS + kg * 64 + 32 * j + 8 * g;
        const bf16x8 a = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(vrow));
        o[db] = mfma16_bf16(a, ph, o[db]);
        o[db] = mfma16_bf16(a, pl, o[db]);
      }
    }
    if (t + 1 < ntiles) {
      __syncthreads();   // every wave is done with tile t
      store_tile();
      __syncthreads();
    }
  }

  // merge the key groups: groups kg > 0 publish (m, partial l, O^T) in LDS,
  // group 0 of the same query group rescales and adds them
  if constexpr (KG > 1) {
    __syncthreads();                              // K/V tiles no longer needed
    float* xm = reinterpret_cast<float*>(ks);     // [KG-1][QG][64]
    float* xl = xm + (KG - 1) * QG * 64;          // [KG-1][QG][64]
    float* xo = reinterpret_cast<float*>(vs);     // [KG-1][QG][NDB*4][64]
    static_assert((KG - 1) * QG * 64 * 2 * 4 <= SK * KS * 2, "merge scratch (m, l)");
    static_assert((KG - 1) * QG * NDB * 4 * 64 * 4 <= DH * VS * 2, "merge scratch (O)");
    if (kg > 0) {
      const int slot = (kg - 1) * QG + qg;
      xm[slot * 64 + lane] = m_ref;
      xl[slot * 64 + lane] = l_run;
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int i = 0; i < 4; ++i) xo[(slot * NDB * 4 + db * 4 + i) * 64 + lane] = o[db][i];
    }
    __syncthreads();
    if (kg > 0) return;
#pragma unroll
    for (int k = 1; k < KG; ++k) {
      const int slot = (k - 1) * QG + qg;
      const float m2 = xm[slot * 64 + lane];
      const float l2 = xl[slot * 64 + lane];
      const float mm = fmaxf(m_ref, m2);
      const float a1 = m_ref == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f((m_ref - mm) * scale_log2);
      const float a2 = m2 == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f((m2 - mm) * scale_log2);
      l_run = l_run * a1 + l2 * a2;
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          o[db][i] = o[db][i] * a1 + xo[(slot * NDB * 4 + db * 4 + i) * 64 + lane] * a2;
      m_ref = mm;
    }
  }

  // finish: l over the 4 lanes sharing the query, normalise, store
  l_run += __shfl_xor(l_run, 16, 64);
  l_run += __shfl_xor(l_run, 32, 64);
  const float inv = 1.0f / l_run;
  if (q_ok) {
    bf16* dst = out + qrow * hq * DH + h * DH;
#pragma unroll
    for (int db = 0; db < NDB; ++db) {
      bf16x4 v;
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = (bf16)(o[db][i] * inv);
      *reinterpret_cast<bf16x4*>(dst + db * 16 + 4 * g) = v;
    }
  }
}

// Shared-tile kernel (gh query heads per key/value head; 1 for MHA): one block =
// eight consecutive groups of (16 query rows, query head) that read one
// key/value head of one request, one wave per group, heads fastest, so every
// staged K/V tile serves 128 query rows whatever gh is (a launch of 7-head blocks
// of seven waves left one SIMD in four with a wave less: 16 x 1024 rows of 28/4
// heads 442 -> 375 us; MHA blocks of 64 rows moved each tile twice as often:
// 8 x 1280 rows of 32 heads 443 -> 325 us). Waves whose group does not exist load
// and meet the barriers only. Tiles of 64 keys are fetched with
// direct global->LDS loads into a two-stage ring: the next tile's loads run
// during the current tile's MFMAs and no registers hold tiles in flight,
// which keeps the register count low enough for two blocks per CU.
//
// LDS layout of a stage:
//   K: 64 rows of DH. Row rho holds key pi(rho) of the tile, where inside each
//      group of 32 keys pi(16 h + 4 g + i) = 8 g + 4 h + i (h < 2, g < 4,
//      i < 4). With this order the S^T values a lane of lane group g owns
//      are the keys 8 g .. 8 g + 7 of each 32-key group, which is the k slice
//      that lane group supplies to the PV MFMA, so V^T is read as one
//      16-byte chunk per lane and no shuffle is needed.
//   V^T: DH rows of 64 keys (128 bytes).
//   The 16-byte chunk c of row r is stored at chunk slot c ^ (r & 7): the
//   eight lanes of one LDS read phase (one chunk of eight consecutive rows)
//   hit distinct banks. Each lane of a load instruction fetches the global
//   chunk that belongs at its slot.
// Keys at or beyond L inside the last tile are read from the slot (a slot
// holds s_max positions, a multiple of 64) and then masked: their scores are
// set to -inf and their V^T entries cleared in LDS.
constexpr int kSharedWaves = 8;
// blocks of a request per key/value head
__host__ __device__ constexpr int shared_blocks(int nrows, int gh, int waves) {
  return ceil_div(ceil_div(nrows, 16) * gh, waves);
}
// SPLIT: blockIdx also counts the key splits, each a contiguous range of the
// request's key tiles; a block leaves its unnormalised O and (m, l) of every
// (row, head) in po and ml, [split][row][head], for attn_merge_kernel.
template <int DH, bool SPLIT, int NW>
__global__ __launch_bounds__(NW * 64) void attn_gqa_kernel(
    StepPlan p, const bf16* __restrict__ q, const bf16* __restrict__ kc,
    const bf16* __restrict__ vc, int s_max, int hq, int hkv, bf16* __restrict__ out,
    float scale_log2, int splits, float* __restrict__ po, float2* __restrict__ ml) {
  constexpr int NT = NW * 64;
  constexpr int SK = 64;                   // keys per tile
  constexpr int KRB = DH * 2;              // K row bytes
  constexpr int KCPR = DH / 8;             // 16-byte chunks per K row
  constexpr int KRPI = 1024 / KRB;         // K rows per load instruction
  constexpr int NKI = SK / KRPI;           // K load instructions per tile
  constexpr int NVI = DH / 8;              // V^T load instructions per tile (8 rows each)
  constexpr int NI = NKI + NVI;
  constexpr int IPW = (NI + NW - 1) / NW;  // load instructions per wave (at most)
  constexpr int KBYTES = SK * KRB;
  constexpr int STAGE = KBYTES + DH * SK * 2;
  constexpr int NDB = DH / 16;             // output dh blocks
  constexpr int NKS = DH / 32;             // k steps of S
  __shared__ __attribute__((aligned(1024))) char smem[2 * STAGE];

  // Block order: blocks are handed out in linear order round-robin over the
  // XCDs; the linear id is remapped so that each XCD receives one contiguous
  // range of (key/value head, query tile) with query tiles fastest, so the
  // row tiles of one request and key/value head run on one XCD at about the
  // same time and share its L2.
  int kvh, tile, split = 0;
  {
    const int total = gridDim.x, id = blockIdx.x;
    const int xcd = id % kXcds, per = total / kXcds, rem = total % kXcds;
    const int lid = xcd * per + min(xcd, rem) + id / kXcds;
    const int row = lid / p.n_tiles;              // (key/value head, split)
    tile = lid - row * p.n_tiles;
    if constexpr (SPLIT) {
      kvh = row / splits;
      split = row - kvh * splits;
    } else {
      kvh = row;
    }
  }
  const int gh = hq / hkv;
  const ReqPlan& rq = p.r[plan_req_of_tile(p, tile)];
  const int L = rq.seq_len;
  const bf16* kb = kc + ((long)(rq.slot * hkv + kvh) * s_max) * DH;
  const bf16* vb = vc + ((long)(rq.slot * hkv + kvh) * DH) * s_max;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int grp = (tile - rq.tile0) * NW + wave;        // this wave's (row group, head)
  const int row16 = grp / gh * 16;
  const int h = kvh * gh + grp % gh;              // query head
  const int qr = row16 + (lane & 15);             // query row of this lane in the request
  const bool q_ok = qr < rq.nrows;
  const bool w_ok = row16 < rq.nrows;             // uniform over the wave
  const long qrow = rq.row0 + qr;
  const int g = lane >> 4;

  // this wave's load instructions: j = wave + NW m over the tile's NI
  // instructions (the first NKI fill K, the rest V^T); per instruction the
  // lane's source at key 0 of the slot and the LDS byte offset in the stage
  const bf16* src[IPW];
  int dst[IPW];
#pragma unroll
  for (int m = 0; m < IPW; ++m) {
    const int j = wave + NW * m;
    if (j < NKI) {
      const int rho = KRPI * j + lane / KCPR;
      const int c = (lane % KCPR) ^ (rho & 7);
      const int key = (rho & ~31) | (((rho >> 2) & 3) << 3) | (((rho >> 4) & 1) << 2) | (rho & 3);
      src[m] = kb + (long)key * DH + c * 8;
      dst[m] = j * 1024;
    } else {
      const int jv = min(j, NI - 1) - NKI;
      const int d = 8 * jv + lane / 8;
      const int c = (lane % 8) ^ (d & 7);
      src[m] = vb + (long)d * s_max + c * 8;
      dst[m] = KBYTES + jv * 1024;
    }
  }
  auto issue = [&](int stage, int key0) {
    char* base = smem + stage * STAGE;
#pragma unroll
    for (int m = 0; m < IPW; ++m) {
      const int j = wave + NW * m;
      if (j < NI)
        load_lds16(src[m] + (j < NKI ? (long)key0 * DH : (long)key0), base + dst[m]);
    }
  };

  // Q fragments (B operand): col = query lane&15, k = dh 32*s + 8*g .. +7
  u32x4 qf[NKS];
#pragma unroll
  for (int s = 0; s < NKS; ++s) {
    if (q_ok)
      qf[s] = *reinterpret_cast<const u32x4*>(q + qrow * hq * DH + h * DH + s * 32 + g * 8);
    else
      qf[s] = u32x4{0u, 0u, 0u, 0u};
  }

  f32x4 o[NDB];
#pragma unroll
  for (int i = 0; i < NDB; ++i) o[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_ref = -INFINITY, l_run = 0.f;
  const int sw = (lane & 7) << 4;                 // chunk-slot XOR of rows 16 b + (lane & 15)

  int tbeg = 0, ntiles = ceil_div(L, SK);         // this block's key tiles [tbeg, ntiles)
  if constexpr (SPLIT) {
    const int per = ceil_div(ntiles, splits);
    tbeg = split * per;
    ntiles = min(ntiles, tbeg + per);
  }
  if (!SPLIT || tbeg < ntiles) issue(tbeg & 1, tbeg * SK);
  for (int t = tbeg; t < ntiles; ++t) {
    const int key0 = t * SK;
    wait_vmcnt<0>();
    __syncthreads();                              // tile t in LDS; stage (t + 1) & 1 free
    const char* kst = smem + (t & 1) * STAGE;
    const char* vst = kst + KBYTES;
    const bool tail = key0 + SK > L;
    if (tail) {                                   // clear V^T at keys >= L
      const int kl = L - key0;
      for (int idx = tid; idx < DH * 8; idx += NT) {
        const int d = idx >> 3, c = idx & 7;
        if (8 * c + 8 > kl) {
          u32x4* ptr = reinterpret_cast<u32x4*>(const_cast<char*>(vst) + d * 128 + ((c ^ (d & 7)) << 4));
          u32x4 v = *ptr;
#pragma unroll
          for (int w = 0; w < 4; ++w) {
            const uint32_t keep = (8 * c + 2 * w < kl ? 0x0000ffffu : 0u) |
                                  (8 * c + 2 * w + 1 < kl ? 0xffff0000u : 0u);
            v[w] &= keep;
          }
          *ptr = v;
        }
      }
      __syncthreads();
    }
    if (t + 1 < ntiles) issue((t + 1) & 1, key0 + SK);
    if (!w_ok) continue;                          // no rows: load and meet the barriers only

    // S^T blocks: sblk[kb][i] = raw score(key = key0 + pi(16 kb + 4 g + i), query = lane & 15)
    f32x4 sblk[4];
#pragma unroll
    for (int kbk = 0; kbk < 4; ++kbk) {
      f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
      const char* krow = kst + (kbk * 16 + (lane & 15)) * KRB;
#pragma unroll
      for (int s = 0; s < NKS; ++s) {
        const u32x4 a = *reinterpret_cast<const u32x4*>(krow + (((s * 4 + g) << 4) ^ sw));
        acc = mfma16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, qf[s]), acc);
      }
      sblk[kbk] = acc;
    }
    if (tail) {
#pragma unroll
      for (int kbk = 0; kbk < 4; ++kbk)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (key0 + 32 * (kbk >> 1) + 8 * g + 4 * (kbk & 1) + i >= L) sblk[kbk][i] = -INFINITY;
    }
    float mt = -INFINITY;
#pragma unroll
    for (int kbk = 0; kbk < 4; ++kbk)
#pragma unroll
      for (int i = 0; i < 4; ++i) mt = fmaxf(mt, sblk[kbk][i]);
    mt = fmaxf(mt, __shfl_xor(mt, 16, 64));
    mt = fmaxf(mt, __shfl_xor(mt, 32, 64));
    // move the reference maximum only on a large increase
    const bool grow = (mt - m_ref) * scale_log2 > 8.0f;
    if (__builtin_amdgcn_ballot_w64(grow)) {
      const float alpha = grow ? __builtin_amdgcn_exp2f((m_ref - mt) * scale_log2) : 1.0f;
      if (grow) m_ref = mt;
      l_run *= alpha;
#pragma unroll
      for (int i = 0; i < NDB; ++i) o[i] *= alpha;
    }
    const float nm = m_ref == -INFINITY ? 0.0f : -m_ref * scale_log2;
    float lsum = 0.f;
#pragma unroll
    for (int kbk = 0; kbk < 4; ++kbk)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float e = __builtin_amdgcn_exp2f(fmaf(sblk[kbk][i], scale_log2, nm));
        sblk[kbk][i] = e;
        lsum += e;
      }
    l_run += lsum;

    // O^T += V^T P^T over two 32-key steps; B operand slot 8 g + e <-> key
    // 32 j + 8 g + e, which lane group g holds as sblk[2 j + e / 4][e % 4]
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      bf16x8 ph, pl;
      split_p8(sblk[2 * j], sblk[2 * j + 1], ph, pl);
#pragma unroll
      for (int db = 0; db < NDB; ++db) {
        const u32x4 a = *reinterpret_cast<const u32x4*>(vst + (db * 16 + (lane & 15)) * 128 +
                                                        (((4 * j + g) << 4) ^ sw));
        o[db] = mfma16_bf16(__builtin_bit_cast(bf16x8, a), ph, o[db]);
        o[db] = mfma16_bf16(__builtin_bit_cast(bf16x8, a), pl, o[db]);
      }
    }
  }

  // finish: l over the 4 lanes sharing the query, normalise, store
  l_run += __shfl_xor(l_run, 16, 64);
  l_run += __shfl_xor(l_run, 32, 64);
  if constexpr (SPLIT) {                          // no tiles: (-inf, 0) and zeros
    if (q_ok) {
      const long at = ((long)split * p.n_rows + qrow) * hq + h;
#pragma unroll
      for (int db = 0; db < NDB; ++db)
        *reinterpret_cast<f32x4*>(po + at * DH + db * 16 + 4 * g) = o[db];
      if (g == 0) ml[at] = make_float2(m_ref, l_run);
    }
    return;
  }
  const float inv = 1.0f / l_run;
  if (q_ok) {
    bf16* dstp = out + qrow * hq * DH + h * DH;
#pragma unroll
    for (int db = 0; db < NDB; ++db) {
      bf16x4 v;
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = (bf16)(o[db][i] * inv);
      *reinterpret_cast<bf16x4*>(dstp + db * 16 + 4 * g) = v;
    }
  }
}

// Adds the key splits of each (row, head): DH / 4 lanes per item, the splits'
// loads in flight together, sums in split order.
constexpr int kMaxSplits = 8;   // more measured no faster
template <int DH>
__global__ __launch_bounds__(256) void attn_merge_kernel(const float* __restrict__ po,
                                                         const float2* __restrict__ ml, int items,
                                                         int splits, bf16* __restrict__ out,
                                                         float scale_log2) {
  constexpr int LPI = DH / 4;              // lanes per item
  const int item = blockIdx.x * (256 / LPI) + threadIdx.x / LPI, c = threadIdx.x % LPI * 4;
  if (item >= items) return;
  float mm = -INFINITY, l = 0.f;
  f32x4 o = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int s0 = 0; s0 < splits; s0 += 4) {
    float2 x[4];
    f32x4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const long at = (long)min(s0 + u, splits - 1) * items + item;
      x[u] = ml[at];
      v[u] = *reinterpret_cast<const f32x4*>(po + at * DH + c);
    }
    float mn = mm;
#pragma unroll
    for (int u = 0; u < 4; ++u) mn = fmaxf(mn, x[u].x);
    if (mn != mm) {                        // (mm = -inf: nothing added yet)
      const float a = __builtin_amdgcn_exp2f((mm - mn) * scale_log2);
      l *= a;
      o *= a;
      mm = mn;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (s0 + u >= splits || x[u].y == 0.f) continue;   // l = 0: the split has no keys
      const float a = __builtin_amdgcn_exp2f((x[u].x - mm) * scale_log2);
      l += x[u].y * a;
      o += v[u] * a;
    }
  }
  const float inv = 1.0f / l;
  bf16x4 r;
#pragma unroll
  for (int i = 0; i < 4; ++i) r[i] = (bf16)(o[i] * inv);
  *reinterpret_cast<bf16x4*>(out + (long)item * DH + c) = r;
}

// fp32 (the small fp32 model): one block = 16 query rows of one request x one
// query head, kF32Waves waves that take 32-key groups in turn, each with its own
// online softmax, merged in LDS at the end. Scores and outputs go through
// v_mfma_f32_16x16x4_f32 as S^T = K Q^T and O^T = V^T P^T: a lane's score
// accumulators (keys 4 g .. 4 g + 3 of a 16-key group, its own query; g = lane /
// 16) are the B operands of the PV products as they stand, and K rows and
// transposed V rows are read from the cache as the 16-byte fragments the MFMAs
// take, without LDS (a block reads each once). Latency bounds it at the sizes the
// model runs: 128 rows over 128 keys, 4 heads, took 324 us with one lane per query
// row in 8 blocks of one wave, and takes 9 us.
constexpr int kF32Waves = 4;
template <int DH>
__global__ __launch_bounds__(kF32Waves * 64) void attn_f32_kernel(
    StepPlan p, const float* __restrict__ q, const float* __restrict__ kc,
    const float* __restrict__ vc, int s_max, int hq, int hkv, float* __restrict__ out,
    float scale) {
  constexpr int NDB = DH / 16;             // 16-wide dh groups
  __shared__ float xm[kF32Waves][64], xl[kF32Waves][64];
  __shared__ f32x4 xo[kF32Waves][NDB][64];
  const int tile = blockIdx.x, h = blockIdx.y;
  const ReqPlan& rq = p.r[plan_req_of_tile(p, tile)];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = lane >> 4, c = lane & 15;
  const int qr = (tile - rq.tile0) * 16 + c;     // query row of this lane within the request
  const bool q_ok = qr < rq.nrows;
  const long qrow = rq.row0 + min(qr, rq.nrows - 1);
  const int L = rq.seq_len;
  const int kvh = h / (hq / hkv);
  const float* kb = kc + ((long)(rq.slot * hkv + kvh) * s_max) * DH;
  const float* vb = vc + ((long)(rq.slot * hkv + kvh) * DH) * s_max;

  // a lane's fragment element e of dh group j is dh index 16 j + 4 g + e, for Q and K alike
  f32x4 qf[NDB], o[NDB];
#pragma unroll
  for (int j = 0; j < NDB; ++j) {
    qf[j] = *reinterpret_cast<const f32x4*>(q + qrow * hq * DH + h * DH + 16 * j + 4 * g);
    o[j] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  float m_run = -INFINITY, l_run = 0.f;    // l: this lane's keys only
  // 32-key groups; a slot holds a multiple of 64 positions, so reads past L stay inside it
  for (int key0 = wave * 32; key0 < L; key0 += kF32Waves * 32) {
    f32x4 s[2], vf[2][NDB];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      f32x4 kf[NDB];
#pragma unroll
      for (int j = 0; j < NDB; ++j)
        kf[j] = *reinterpret_cast<const f32x4*>(kb + (long)(key0 + 16 * b + c) * DH + 16 * j + 4 * g);
      s[b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int j = 0; j < NDB; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) s[b] = mfma16_f32(kf[j][e], qf[j][e], s[b]);
    }
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int j = 0; j < NDB; ++j)
        vf[b][j] = *reinterpret_cast<const f32x4*>(vb + (long)(16 * j + c) * s_max + key0 + 16 * b + 4 * g);
    float mt = -INFINITY;
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bool in = key0 + 16 * b + 4 * g + e < L;
        s[b][e] = in ? s[b][e] * scale : -INFINITY;
        mt = fmaxf(mt, s[b][e]);
        if (!in) {                         // stale memory past the sequence: 0 x NaN is NaN
#pragma unroll
          for (int j = 0; j < NDB; ++j) vf[b][j][e] = 0.f;
        }
      }
    mt = fmaxf(mt, __shfl_xor(mt, 16, 64));
    mt = fmaxf(mt, __shfl_xor(mt, 32, 64));
    const float m_new = fmaxf(m_run, mt);
    // -inf while every score so far is (overflowed): weights of 0, not exp(-inf + inf)
    const float m_ref = m_new == -INFINITY ? 0.f : m_new;
    const float alpha = expf(m_run - m_ref);
    l_run *= alpha;
#pragma unroll
    for (int j = 0; j < NDB; ++j) o[j] *= alpha;
    m_run = m_new;
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float w = expf(s[b][e] - m_ref);
        l_run += w;
#pragma unroll
        for (int j = 0; j < NDB; ++j) o[j] = mfma16_f32(vf[b][j][e], w, o[j]);
      }
  }
  // merge the waves' key groups
  xm[wave][lane] = m_run;
  xl[wave][lane] = l_run;
#pragma unroll
  for (int j = 0; j < NDB; ++j) xo[wave][j][lane] = o[j];
  __syncthreads();
  float mm = -INFINITY;
#pragma unroll
  for (int w = 0; w < kF32Waves; ++w) mm = fmaxf(mm, xm[w][lane]);
  float a[kF32Waves], l = 0.f;
#pragma unroll
  for (int w = 0; w < kF32Waves; ++w) {
    a[w] = expf(xm[w][lane] - mm);         // 0 for a wave without keys
    l += xl[w][lane] * a[w];
  }
  l += __shfl_xor(l, 16, 64);
  l += __shfl_xor(l, 32, 64);
  const float inv = 1.0f / l;
  for (int j = wave; j < NDB; j += kF32Waves) {
    f32x4 t = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < kF32Waves; ++w) t += xo[w][j][lane] * a[w];
    if (q_ok)
      *reinterpret_cast<f32x4*>(out + qrow * hq * DH + h * DH + 16 * j + 4 * g) = t * inv;
  }
}

template <int DH, int QG, int KG>
static hipError_t launch_attn(const StepPlan& p, const bf16* q, const bf16* kc, const bf16* vc,
                              int s_max, int hq, int hkv, bf16* out, float scale_log2,
                              hipStream_t st) {
  const StepPlan t = plan_with_tiles(p, [](int n) { return ceil_div(n, 16 * QG); });
  if (t.n_tiles == 0) return hipSuccess;
  DLM_LAUNCH((attn_bf16_kernel<DH, QG, KG>), dim3(hq, t.n_tiles), dim3(QG * KG * 64), 0, st,
                     t, q, kc, vc, s_max, hq, hkv, out, scale_log2);
  return hipGetLastError();
}

template <int DH, bool SPLIT, int NW>
static hipError_t launch_shared(const StepPlan& p, const bf16* q, const bf16* kc, const bf16* vc,
                                int s_max, int hq, int hkv, bf16* out, float scale_log2, int splits,
                                float* scratch, hipStream_t st) {
  const StepPlan t = plan_with_tiles(p, [&](int n) { return shared_blocks(n, hq / hkv, NW); });
  if (t.n_tiles == 0) return hipSuccess;
  DLM_LAUNCH((attn_gqa_kernel<DH, SPLIT, NW>), dim3(hkv * t.n_tiles * splits), dim3(NW * 64), 0, st,
             t, q, kc, vc, s_max, hq, hkv, out, scale_log2, splits, scratch,
             reinterpret_cast<float2*>(scratch + (size_t)splits * p.n_rows * hq * DH));
  return hipGetLastError();
}

template <int DH>
static hipError_t attention_dh(const StepPlan& p, const bf16* q, const bf16* kc, const bf16* vc,
                               int s_max, int hq, int hkv, bf16* out, float scale_log2,
                               AttnPlan plan, float* scratch, hipStream_t st) {
  if (hkv < 1 || hq % hkv != 0 || plan.splits < 1 || plan.splits > kMaxSplits ||
      (plan.splits > 1 && plan.kernel != kAttnShared))
    return hipErrorInvalidValue;
#define ATTN_HEAD(QG_, KG_) launch_attn<DH, QG_, KG_>(p, q, kc, vc, s_max, hq, hkv, out, scale_log2, st)
#define ATTN_SHARED(SPLIT_, NW_)                                                            \
  launch_shared<DH, SPLIT_, NW_>(p, q, kc, vc, s_max, hq, hkv, out, scale_log2, plan.splits, \
                                 scratch, st)
  switch (plan.kernel) {
    case kAttnShared:
      return plan.splits > 1 ? ATTN_SHARED(true, kSharedWaves) : ATTN_SHARED(false, kSharedWaves);
    case kAttnHead32x4: return ATTN_HEAD(2, 4);
    case kAttnHead64x2: return ATTN_HEAD(4, 2);
    default: break;
  }
  if constexpr (DH == 64) {
    if (plan.kernel == kAttnShared4) return ATTN_SHARED(false, 4);
    if (plan.kernel == kAttnHead32x2) return ATTN_HEAD(2, 2);
  }
#undef ATTN_SHARED
#undef ATTN_HEAD
  return hipErrorInvalidValue;
}

// Kernel and key splits of a bf16 launch. Times are one layer's launch on MI355X
// (256 CUs) with cold caches, in us; head_dim 128 unless stated. What decides: blocks
// per CU; whether more than half of a shared-tile block's eight waves have rows
// ("full"); and the key tiles of 64 that a block walks one after the other.
//  * Key splits (shared tiles; attn_merge_kernel adds 4 us, and the partials' way
//    through memory a key tile's time per 16384 (row, head, split)) where the walk
//    gets shorter by enough tiles, about 1 us each: 5; 11 for multi-head head_dim
//    64, whose tiles take half as long; 4 more where the per-head kernel below fills
//    half the CUs. As many ranges as make a block per CU (28/4 heads, 8 x 48 rows
//    over 1280 keys, 96 blocks: two ranges 29.0, three 32.6, whole 31.9), or 9/8 of
//    that where blocks are not full (32 heads, 3 x 16 over 2304, 96 blocks: three
//    29.3, two 31.6). 32 x 517 6.8 + 4.0 against 15.5, 28/4 heads, 64 x 900 8.0 + 4.0
//    / 21.6; left whole: 512 x 512 15.1 + 4.6 / 16.0, head_dim 64, 2 x 200 over 1280
//    20.8 / 18.8.
//  * At most 32 rows per request: grouped queries fill the shared-tile blocks
//    (28/4, 20 x 32 over 1280 shared 40, per head 76; 48 x 16 over 320 15 / 90).
//    Multi-head: shared tiles over short sequences (8 x 32 over 640 20 / 26) and
//    where the per-head blocks start a second round (10 x 32 over 1280 43 /
//    56, 16 x 32 67 / 71, 20 x 32 98 / 94, 6 x 32 over 2304 52 / 47). head_dim 64:
//    per-head blocks of four waves, which fit twice as often on a CU (20 x 32 over
//    1280 shared 52, four key groups 49, two 44; 8 x 32 over 320 7.8 / 11.2 /
//    10.9); four key groups for long sequences (8 x 32 over 2304 30.7 / 32.5).
//  * head_dim 64, multi-head, at most 64 rows per request, more than two blocks
//    per CU: shared-tile blocks of four waves (20 x 64 over 1280 42.6, eight 53.4,
//    per head 48.8).
//  * Over one or three key tiles, or up to five in blocks that are not full: shared
//    (32 heads, 4 x 64 over 320 10.9 / 14.2; 128 rows over 128, full: 7.7 / 7.0;
//    160 over 160 10.0 / 10.8).
//  * Otherwise the per-head kernel while its blocks fit in one round: 32 rows and
//    four key groups where the 256-key turns are full (32 heads, 256 rows over 256
//    8.1 / 9.1; 200 over 200 10.9 / 10.8), else 64 rows and two (512 rows 14.7,
//    shared 17.6); then shared tiles (600 rows 21.7 / 32.5, 1024 34.3 / 44.7).
AttnPlan attention_plan(const StepPlan& p, int hq, int hkv, int dh, size_t elem,
                        size_t scratch_bytes, int num_cu) {
  if (elem != 2 || hkv < 1 || hq % hkv != 0 || p.n_rows < 1) return AttnPlan{};
  const int gh = hq / hkv;
  int max_rows = 0, max_len = 0;
  long blocks = 0, groups = 0, t32 = 0, t64 = 0;
  for (int r = 0; r < p.n_req; ++r) {
    const int n = p.r[r].nrows;
    max_rows = std::max(max_rows, n);
    max_len = std::max(max_len, p.r[r].seq_len);
    blocks += (long)hkv * shared_blocks(n, gh, kSharedWaves);
    groups += (long)hq * ceil_div(n, 16);
    t32 += (long)hq * ceil_div(n, 32);
    t64 += (long)hq * ceil_div(n, 64);
  }
  const int nt = ceil_div(max_len, 64);
  const bool few = max_rows <= 32, mha = gh == 1, narrow = dh == 64;
  const bool full = 2 * groups > blocks * kSharedWaves;

  const long room = full ? num_cu : num_cu + num_cu / 8;
  const size_t one = (size_t)p.n_rows * hq * (dh * sizeof(float) + sizeof(float2));
  long s = std::min({(long)kMaxSplits, room / blocks, (long)(scratch_bytes / one)});
  for (; s > 1; --s) {                     // ranges of equal length: as many as are not empty
    const int per = ceil_div(nt, (int)s), used = ceil_div(nt, per);
    if (blocks * used > room) continue;
    const long need = (narrow && mha ? 11 : 5) +
                      (full && !few && t64 <= num_cu && 2 * t64 > num_cu ? 4 : 0) +
                      (long)p.n_rows * hq * used * dh / (128 * 16384);
    if (used > 1 && nt - per >= need) return AttnPlan{kAttnShared, used};
    break;
  }
  if (few) {
    if (!mha || nt <= (narrow ? 5 : 10)) return AttnPlan{kAttnShared, 1};
    if (narrow)
      return AttnPlan{nt >= 16 && t32 <= num_cu ? kAttnHead32x4 : kAttnHead32x2, 1};
    return AttnPlan{t32 > num_cu && t32 <= 2 * num_cu ? kAttnShared : kAttnHead32x4, 1};
  }
  if (narrow && mha && max_rows <= 64 && t64 > 2 * num_cu) return AttnPlan{kAttnShared4, 1};
  if (nt == 1 || nt == 3 || (nt <= 5 && !full)) return AttnPlan{kAttnShared, 1};
  const int turns = ceil_div(max_len, 256) * 256;
  if (t32 <= num_cu && nt >= 4 && (turns - max_len) * 8 <= turns) return AttnPlan{kAttnHead32x4, 1};
  return AttnPlan{t64 <= num_cu ? kAttnHead64x2 : kAttnShared, 1};
}

hipError_t attention_merge(const StepPlan& p, int hq, int dh, int splits, const float* scratch,
                           bf16* out, hipStream_t st) {
  const int items = p.n_rows * hq;
  if (items == 0) return hipSuccess;
  const float scale_log2 = 1.4426950408889634f / sqrtf((float)dh);
  const float2* ml = reinterpret_cast<const float2*>(scratch + (size_t)splits * items * dh);
  if (dh == 128)
    DLM_LAUNCH(attn_merge_kernel<128>, dim3(ceil_div(items, 8)), dim3(256), 0, st, scratch, ml,
               items, splits, out, scale_log2);
  else if (dh == 64)
    DLM_LAUNCH(attn_merge_kernel<64>, dim3(ceil_div(items, 16)), dim3(256), 0, st, scratch, ml,
               items, splits, out, scale_log2);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

template <>
hipError_t attention<bf16>(const StepPlan& p, const bf16* q, const bf16* kc, const bf16* vc,
                           int s_max, int hq, int hkv, int dh, bf16* out, AttnPlan plan,
                           float* scratch, hipStream_t st) {
  if (p.n_rows == 0) return hipSuccess;
  const float scale_log2 = 1.4426950408889634f / sqrtf((float)dh);
  if (dh == 128) return attention_dh<128>(p, q, kc, vc, s_max, hq, hkv, out, scale_log2, plan, scratch, st);
  if (dh == 64) return attention_dh<64>(p, q, kc, vc, s_max, hq, hkv, out, scale_log2, plan, scratch, st);
  return hipErrorInvalidValue;
}

template <>
hipError_t attention<float>(const StepPlan& p, const float* q, const float* kc, const float* vc,
                            int s_max, int hq, int hkv, int dh, float* out, AttnPlan plan, float*,
                            hipStream_t st) {
  if (plan.splits != 1) return hipErrorInvalidValue;
  if (p.n_rows == 0) return hipSuccess;
  const float scale = 1.0f / sqrtf((float)dh);
  const StepPlan t = plan_with_tiles(p, [](int n) { return ceil_div(n, 16); });
  dim3 g(t.n_tiles, hq);
  if (dh == 64)
    DLM_LAUNCH(attn_f32_kernel<64>, g, dim3(kF32Waves * 64), 0, st, t, q, kc, vc, s_max, hq, hkv,
                       out, scale);
  else if (dh == 128)
    DLM_LAUNCH(attn_f32_kernel<128>, g, dim3(kF32Waves * 64), 0, st, t, q, kc, vc, s_max, hq, hkv,
                       out, scale);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace dlm
