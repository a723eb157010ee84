// Fused masked attention in fp32 on the matrix cores (v_mfma_f32_32x32x2_f32), forward and
// backward, for head sizes up to 128 (multiples of 16; a kernel instance is built for each multiple of
// 32 and the next smaller size runs on it with its upper 16 columns read as zeros and never stored).
//
// Same operator, same decomposition and same orientation of the score blocks as the bf16 kernels
// in attention_mfma.hip (the paper's matmul / exp / max / sum primitives, Section 4.1.1, fused with
// a pre-fused gradient function, Section 5.2.1): a wavefront owns 32 query rows (forward, dQ) or
// 32 key rows (dK/dV) and walks the other sequence dimension in LDS tiles; the MFMA that produces
// a score block leaves the index contracted NEXT in a lane's registers, so probabilities go from
// accumulator registers straight into the next MFMA.
//
// The fp32 MFMA contracts two k per instruction: lanes 0..31 supply k = 0, lanes 32..63 k = 1, one
// value per lane for each operand.  With fp32 there is nothing to pack and nothing to transpose:
//   "row" fragments  (contraction along the head dimension): lane reads tile[row0 + lane%32][2*kk + lane/32]
//   "column" fragments (contraction along the walked rows): lane reads tile[krow][col0 + lane%32],
//       where krow is the tile row whose score sits in register t of THIS lane half -- the two
//       halves of a wavefront hold different rows in the same register, and the instruction only
//       needs both operands to agree on which row is "k = lane/32".
// Along the head dimension the order of k is free as long as both operands agree on it: MFMA 4j + e of a score block
// contracts elements (2j + h)*4 + e, h = lane/32, so that a lane takes four MFMAs' operands with one 16-byte read
// (rows of the LDS tiles, and the wavefront's own row straight from memory).
// Tiles are row-major fp32 with four floats of padding per row.
//
// A wavefront's chain of dependent MFMAs (64 clocks for two k) sets the time, so the four wavefronts of a workgroup
// are split between rows and keys: KG of them share 32 rows and take the blocks of the walked dimension in turn,
// each with its own statistics and accumulators, which meet in LDS at the end.  KG = 4 where the problem has few
// (sequence, head, 128-row block) triples, KG = 1 -- no duplicated tile loads -- where they fill the chip.
#include "devutil.h"
#include "kernels.h"
#include "philox.h"

namespace fl {
namespace {

constexpr int NT = 256;        // threads per workgroup (4 wavefronts)
constexpr float LOG2E = 1.4426950408889634f, LN2 = 0.6931471805599453f;

// rows of the walked dimension per LDS tile: at least one 32-row block for each of the KG wavefronts on the same rows
constexpr int tile_rows(int dh, int kg) { return kg == 4 ? 128 : dh <= 64 || kg == 2 ? 64 : 32; }
constexpr int rows_wg(int kg) { return 128 / kg; }   // rows owned by a workgroup (32 per group of KG wavefronts)
constexpr int row_stride(int dh) { return dh + 4; }

__device__ __forceinline__ int acc_row(int r, int h) { return (r >> 2) * 8 + h * 4 + (r & 3); }

__device__ __forceinline__ f32x16_t mfma2(float a, float b, f32x16_t c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ void zero16(f32x16_t &v) {
#pragma unroll
  for (int r = 0; r < 16; ++r) v[r] = 0.f;
}

// A tile of up to TILE rows of DH floats on its way from global memory to LDS (rows >= nvalid are zero):
// load() issues the global reads, store() writes the tile; the kernels load tile t+1 right after storing
// tile t so that the reads are in flight during the MFMAs.
template <int DH, int KG> struct TileRegsF {
  static constexpr int TILE = tile_rows(DH, KG), CPR = DH / 4, N = TILE * CPR / NT;
  static_assert(TILE * CPR % NT == 0, "tile must divide among the threads");
  float4 r[N];
  __device__ __forceinline__ void load(const float *src, size_t ld, int nvalid, int dh) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int c = threadIdx.x + NT * i, row = c / CPR, ch = c % CPR;
      r[i] = row < nvalid && ch * 4 < dh ? *reinterpret_cast<const float4 *>(src + (size_t)row * ld + ch * 4)
                                         : make_float4(0, 0, 0, 0);
    }
  }
  __device__ __forceinline__ void store(float *dst) const {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int c = threadIdx.x + NT * i, row = c / CPR, ch = c % CPR;
      *reinterpret_cast<float4 *>(dst + row * row_stride(DH) + ch * 4) = r[i];
    }
  }
};

// this lane's operand values of its own row: element (2j + lane/32)*4 + e at [4j + e] (zeros without a row)
template <int DH> __device__ __forceinline__ void own_row(const float *row, int h2, int dh, float (&f)[DH / 2]) {
#pragma unroll
  for (int j = 0; j < DH / 8; ++j) {
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    if (row && 8 * j < dh) v = *reinterpret_cast<const float4 *>(row + (2 * j + h2) * 4);
    f[4 * j] = v.x; f[4 * j + 1] = v.y; f[4 * j + 2] = v.z; f[4 * j + 3] = v.w;
  }
}
// s += tile row (at `row`, offset by the lane half already) x own values, along the head dimension
template <int DH> __device__ __forceinline__ f32x16_t row_dot(const float *row, const float (&own)[DH / 2], f32x16_t s) {
#pragma unroll
  for (int j = 0; j < DH / 8; ++j) {
    const float4 v = *reinterpret_cast<const float4 *>(row + 8 * j);
    s = mfma2(v.x, own[4 * j], s);
    s = mfma2(v.y, own[4 * j + 1], s);
    s = mfma2(v.z, own[4 * j + 2], s);
    s = mfma2(v.w, own[4 * j + 3], s);
  }
  return s;
}
// Position of a wavefront: group of rows, and its place among the KG wavefronts on those rows.
template <int KG> struct WavePos {
  int rg, kg;
  __device__ __forceinline__ WavePos() : rg((int)(threadIdx.x >> 6) / KG), kg((int)(threadIdx.x >> 6) % KG) {}
};
// Adds up what the KG wavefronts on the same rows hold, through LDS ([wavefront][register][lane]): wavefront kg returns
// with the sums of registers 4g .. 4g+3, g = kg * 4/KG .. , of every 32-column block; `w` weighs the wavefronts.
template <int NB, int KG> __device__ __forceinline__ void park(float *red, const f32x16_t (&acc)[NB]) {
  float *mine = red + (threadIdx.x >> 6) * (NB * 16 * 64) + (threadIdx.x & 63);
#pragma unroll
  for (int db = 0; db < NB; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) mine[(db * 16 + r) * 64] = acc[db][r];
}
template <int NB, int KG>
__device__ __forceinline__ void gather(const float *red, int rg, int db, int g, const float (&w)[KG], float (&v)[4]) {
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = 0.f;
#pragma unroll
  for (int k = 0; k < KG; ++k) {
    const float *src = red + ((rg * KG + k) * NB * 16 + db * 16 + g * 4) * 64 + (threadIdx.x & 63);
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] += src[e * 64] * w[k];
  }
}
template <int DH, int KG> constexpr size_t f32_lds_floats() {   // two tiles, the query statistics, and the merge
  const size_t tiles = (size_t)2 * tile_rows(DH, KG) * row_stride(DH) + 2 * tile_rows(DH, KG);
  const size_t merge = KG > 1 ? (size_t)4 * (DH / 32) * 16 * 64 + 4 * 2 * 64 : 0;
  return tiles > merge ? tiles : merge;
}

// ------------------------------------------------------------------------------------------ forward
template <int DH, bool CAUSAL, bool DROP, int KG>
__global__ __launch_bounds__(NT) void attn_fwd_mfma_f32(const float *__restrict__ qkv, const int32_t *__restrict__ lengths,
                                                        DropSpec drop, int Tn, int H, int dh, float scale,
                                                        float *__restrict__ o, float *__restrict__ lse) {
  constexpr int TILE = tile_rows(DH, KG), ST = row_stride(DH), NB = DH / 32, ROWS_WG = rows_wg(KG);
  extern __shared__ __attribute__((aligned(16))) float smem[];
  float *const sK = smem, *const sV = smem + TILE * ST;
  const int lane = threadIdx.x & 63, h2 = lane >> 5, l32 = lane & 31;
  const WavePos<KG> wave;
  const AttnBlock blk = attn_block<CAUSAL>();
  const int b = blk.b, hd = blk.hd, rb = blk.rb;
  const int D = H * dh;
  const size_t ld = (size_t)3 * D;
  const int len = lengths ? min(max(lengths[b], 1), Tn) : Tn;  // a length outside 1..T is treated as the nearest valid one
  const float *base = qkv + (size_t)b * Tn * ld + hd * dh;
  const int q = rb * ROWS_WG + wave.rg * 32 + l32;
  float qf[DH / 2];
  own_row<DH>(q < Tn ? base + (size_t)q * ld : nullptr, h2, dh, qf);
  const float c = scale * LOG2E;
  float m = -INFINITY, l = 0.f;
  f32x16_t oacc[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) zero16(oacc[i]);

  // causal: the workgroup needs keys up to its last query, a wavefront up to the last of its 32 queries
  const int kend = CAUSAL ? min(len, (int)(rb * ROWS_WG + ROWS_WG)) : len;
  const int wend = CAUSAL ? min(len, (int)(rb * ROWS_WG + wave.rg * 32 + 32)) : len;
  TileRegsF<DH, KG> tk, tv;
  tk.load(base + D, ld, min(TILE, Tn), dh);
  tv.load(base + 2 * D, ld, min(TILE, Tn), dh);
  for (int k0 = 0; k0 < kend; k0 += TILE) {
    __syncthreads();
    tk.store(sK);
    tv.store(sV);
    __syncthreads();
    if (k0 + TILE < kend) {
      tk.load(base + (size_t)(k0 + TILE) * ld + D, ld, min(TILE, Tn - k0 - TILE), dh);
      tv.load(base + (size_t)(k0 + TILE) * ld + 2 * D, ld, min(TILE, Tn - k0 - TILE), dh);
    }
#pragma unroll
    for (int kb = wave.kg; kb < TILE / 32; kb += KG) {
      if (k0 + kb * 32 >= wend) break;
      f32x16_t s;
      zero16(s);
      s = row_dot<DH>(sK + (kb * 32 + l32) * ST + h2 * 4, qf, s);   // S^T[key, q]
      float mloc = -INFINITY;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int key = k0 + kb * 32 + acc_row(r, h2);
        s[r] = (key < len && (!CAUSAL || key <= q)) ? s[r] * c : -INFINITY;
        mloc = fmaxf(mloc, s[r]);
      }
      mloc = half_pair_max(mloc);
      const float mnew = fmaxf(m, mloc);   // finite: every block a wavefront visits holds an allowed key for each query
      float rs = 0.f;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        s[r] = exp2f(s[r] - mnew);
        rs += s[r];
      }
      rs = half_pair_sum(rs);
      const float corr = exp2f(m - mnew);
      l = l * corr + rs;   // the softmax denominator ignores dropout
      m = mnew;
      if constexpr (DROP) {  // registers 4g..4g+3 hold four consecutive keys: one generator call
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          float kp[4];
          drop_keep4(drop, (uint32_t)(k0 + kb * 32 + g * 8 + h2 * 4) >> 2, (uint32_t)q, (uint32_t)(b * H + hd), kp);
#pragma unroll
          for (int e = 0; e < 4; ++e) s[g * 4 + e] *= kp[e];
        }
      }
#pragma unroll
      for (int db = 0; db < NB; ++db) {
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[db][r] *= corr;
#pragma unroll
        for (int t = 0; t < 16; ++t)   // O^T[d, q] += V^T[d, key] P^T[key, q], key = the one register t holds
          oacc[db] = mfma2(sV[(kb * 32 + acc_row(t, h2)) * ST + db * 32 + l32], s[t], oacc[db]);
      }
    }
  }
  if constexpr (KG > 1) {
    // merged to the common maximum; a wavefront that saw no block has m = -inf, l = 0 and weight 2^-inf = 0
    // (the first wavefront of a group has seen key 0, so the maximum is finite)
    float *const stat = smem + 4 * NB * 16 * 64;
    __syncthreads();   // the tiles are no longer being read
    park<NB, KG>(smem, oacc);
    stat[(threadIdx.x >> 6) * 128 + lane] = m;
    stat[(threadIdx.x >> 6) * 128 + 64 + lane] = l;
    __syncthreads();
    float w[KG], mk[KG];
    m = -INFINITY;
#pragma unroll
    for (int k = 0; k < KG; ++k) {
      mk[k] = stat[(wave.rg * KG + k) * 128 + lane];
      m = fmaxf(m, mk[k]);
    }
    l = 0.f;
#pragma unroll
    for (int k = 0; k < KG; ++k) {
      w[k] = exp2f(mk[k] - m);
      l += w[k] * stat[(wave.rg * KG + k) * 128 + 64 + lane];
    }
    const float inv = 1.0f / l;
#pragma unroll
    for (int k = 0; k < KG; ++k) w[k] *= inv;
    float *orow = o + ((size_t)b * Tn + q) * D + hd * dh;
#pragma unroll
    for (int db = 0; db < NB; ++db)
#pragma unroll
      for (int i = 0; i < 4 / KG; ++i) {
        const int qd = wave.kg * (4 / KG) + i;
        float v[4];
        gather<NB, KG>(smem, wave.rg, db, qd, w, v);
        if (q < Tn && db * 32 + qd * 8 + h2 * 4 < dh) VecIO<float, 4>::store(orow + db * 32 + qd * 8 + h2 * 4, v);
      }
    if (q < Tn && h2 == 0 && wave.kg == 0) lse[((size_t)b * H + hd) * Tn + q] = (m + log2f(l)) * LN2;
    return;
  }
  if (q < Tn) {
    const float inv = 1.0f / l;
    float *orow = o + ((size_t)b * Tn + q) * D + hd * dh;
#pragma unroll
    for (int db = 0; db < NB; ++db)
#pragma unroll
      for (int qd = 0; qd < 4; ++qd) {
        float v[4] = {oacc[db][qd * 4] * inv, oacc[db][qd * 4 + 1] * inv, oacc[db][qd * 4 + 2] * inv,
                      oacc[db][qd * 4 + 3] * inv};
        if (db * 32 + qd * 8 + h2 * 4 < dh) VecIO<float, 4>::store(orow + db * 32 + qd * 8 + h2 * 4, v);
      }
    if (h2 == 0) lse[((size_t)b * H + hd) * Tn + q] = (m + log2f(l)) * LN2;
  }
}

// ------------------------------------------------------------------------------------------ dQ (+ delta)
template <int DH, bool CAUSAL, bool DROP, int KG, bool WRITE_DELTA>
__device__ __forceinline__ void dq_block(const AttnBlock blk, float *const smem, const float *__restrict__ qkv,
                                         const float *__restrict__ o, const float *__restrict__ dout,
                                         const float *__restrict__ lse, const int32_t *__restrict__ lengths, const DropSpec &drop,
                                         int Tn, int H, int dh, float scale, float *__restrict__ dqkv, float *__restrict__ delta) {
  constexpr int TILE = tile_rows(DH, KG), ST = row_stride(DH), NB = DH / 32, ROWS_WG = rows_wg(KG);
  float *const sK = smem, *const sV = smem + TILE * ST;
  const int lane = threadIdx.x & 63, h2 = lane >> 5, l32 = lane & 31;
  const WavePos<KG> wave;
  const int b = blk.b, hd = blk.hd, rb = blk.rb;
  const int D = H * dh;
  const size_t ld = (size_t)3 * D;
  const int len = lengths ? min(max(lengths[b], 1), Tn) : Tn;  // a length outside 1..T is treated as the nearest valid one
  const float *base = qkv + (size_t)b * Tn * ld + hd * dh;
  const int q = rb * ROWS_WG + wave.rg * 32 + l32;
  const bool qok = q < Tn;
  float qf[DH / 2], dof[DH / 2];
  own_row<DH>(qok ? base + (size_t)q * ld : nullptr, h2, dh, qf);
  own_row<DH>(qok ? dout + ((size_t)b * Tn + q) * D + hd * dh : nullptr, h2, dh, dof);
  float dl = 0.f;
  {
    float of[DH / 2];
    own_row<DH>(qok ? o + ((size_t)b * Tn + q) * D + hd * dh : nullptr, h2, dh, of);
#pragma unroll
    for (int kk = 0; kk < DH / 2; ++kk) dl += dof[kk] * of[kk];
  }
  dl = half_pair_sum(dl);
  const size_t st_idx = ((size_t)b * H + hd) * Tn + (qok ? q : 0);
  const float L2 = qok ? lse[st_idx] * LOG2E : 0.f;
  if (WRITE_DELTA && qok && h2 == 0 && wave.kg == 0) delta[st_idx] = dl;
  const float c = scale * LOG2E;
  f32x16_t acc[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) zero16(acc[i]);

  const int kend = CAUSAL ? min(len, (int)(rb * ROWS_WG + ROWS_WG)) : len;       // as in the forward kernel
  const int wend = CAUSAL ? min(len, (int)(rb * ROWS_WG + wave.rg * 32 + 32)) : len;
  TileRegsF<DH, KG> tk, tv;
  tk.load(base + D, ld, min(TILE, Tn), dh);
  tv.load(base + 2 * D, ld, min(TILE, Tn), dh);
  for (int k0 = 0; k0 < kend; k0 += TILE) {
    __syncthreads();
    tk.store(sK);
    tv.store(sV);
    __syncthreads();
    if (k0 + TILE < kend) {
      tk.load(base + (size_t)(k0 + TILE) * ld + D, ld, min(TILE, Tn - k0 - TILE), dh);
      tv.load(base + (size_t)(k0 + TILE) * ld + 2 * D, ld, min(TILE, Tn - k0 - TILE), dh);
    }
#pragma unroll
    for (int kb = wave.kg; kb < TILE / 32; kb += KG) {
      if (k0 + kb * 32 >= wend) break;
      f32x16_t s, dp;
      zero16(s);
      zero16(dp);
      s = row_dot<DH>(sK + (kb * 32 + l32) * ST + h2 * 4, qf, s);      // S^T[key, q]
      dp = row_dot<DH>(sV + (kb * 32 + l32) * ST + h2 * 4, dof, dp);   // dP^T[key, q]
      if constexpr (DROP) {  // dP = (dO V^T) * keep
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          float kp[4];
          drop_keep4(drop, (uint32_t)(k0 + kb * 32 + g * 8 + h2 * 4) >> 2, (uint32_t)q, (uint32_t)(b * H + hd), kp);
#pragma unroll
          for (int e = 0; e < 4; ++e) dp[g * 4 + e] *= kp[e];
        }
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int key = k0 + kb * 32 + acc_row(r, h2);
        const float p = (key < len && (!CAUSAL || key <= q)) ? exp2f(s[r] * c - L2) : 0.f;
        s[r] = p * (dp[r] - dl);   // dS^T
      }
#pragma unroll
      for (int db = 0; db < NB; ++db)
#pragma unroll
        for (int t = 0; t < 16; ++t)   // dQ^T[d, q] += K^T[d, key] dS^T[key, q]
          acc[db] = mfma2(sK[(kb * 32 + acc_row(t, h2)) * ST + db * 32 + l32], s[t], acc[db]);
    }
  }
  if constexpr (KG > 1) {
    __syncthreads();   // the tiles are no longer being read
    park<NB, KG>(smem, acc);
    __syncthreads();
    float w[KG];
#pragma unroll
    for (int k = 0; k < KG; ++k) w[k] = scale;
    float *drow = dqkv + ((size_t)b * Tn + q) * ld + hd * dh;
#pragma unroll
    for (int db = 0; db < NB; ++db)
#pragma unroll
      for (int i = 0; i < 4 / KG; ++i) {
        const int qd = wave.kg * (4 / KG) + i;
        float v[4];
        gather<NB, KG>(smem, wave.rg, db, qd, w, v);
        if (qok && db * 32 + qd * 8 + h2 * 4 < dh) VecIO<float, 4>::store(drow + db * 32 + qd * 8 + h2 * 4, v);
      }
    return;
  }
  if (qok) {
    float *drow = dqkv + ((size_t)b * Tn + q) * ld + hd * dh;
#pragma unroll
    for (int db = 0; db < NB; ++db)
#pragma unroll
      for (int qd = 0; qd < 4; ++qd) {
        float v[4] = {acc[db][qd * 4] * scale, acc[db][qd * 4 + 1] * scale, acc[db][qd * 4 + 2] * scale,
                      acc[db][qd * 4 + 3] * scale};
        if (db * 32 + qd * 8 + h2 * 4 < dh) VecIO<float, 4>::store(drow + db * 32 + qd * 8 + h2 * 4, v);
      }
  }
}

// ------------------------------------------------------------------------------------------ dK, dV
// OWN_DELTA: the queries' delta = dO . O is computed here instead of read.
template <int DH, bool CAUSAL, bool DROP, int KG, bool OWN_DELTA>
__device__ __forceinline__ void dkv_block(const AttnBlock blk, float *const smem, const float *__restrict__ qkv,
                                          const float *__restrict__ o, const float *__restrict__ dout,
                                          const float *__restrict__ lse, const int32_t *__restrict__ lengths, const DropSpec &drop,
                                          int Tn, int H, int dh, float scale, float *__restrict__ dqkv, const float *__restrict__ delta) {
  constexpr int TILE = tile_rows(DH, KG), ST = row_stride(DH), NB = DH / 32, ROWS_WG = rows_wg(KG);
  float *const sQ = smem, *const sDO = smem + TILE * ST;
  float *const sL = sDO + TILE * ST, *const sDl = sL + TILE;   // lse*log2(e) and delta of the tile's queries
  const int lane = threadIdx.x & 63, h2 = lane >> 5, l32 = lane & 31;
  const WavePos<KG> wave;
  const int b = blk.b, hd = blk.hd, rb = blk.rb;
  const int D = H * dh;
  const size_t ld = (size_t)3 * D;
  const int len = lengths ? min(max(lengths[b], 1), Tn) : Tn;  // a length outside 1..T is treated as the nearest valid one
  const float *base = qkv + (size_t)b * Tn * ld + hd * dh;
  const int key = rb * ROWS_WG + wave.rg * 32 + l32;
  const bool kok = key < Tn;
  float kf[DH / 2], vf[DH / 2];
  own_row<DH>(kok ? base + (size_t)key * ld + D : nullptr, h2, dh, kf);
  own_row<DH>(kok ? base + (size_t)key * ld + 2 * D : nullptr, h2, dh, vf);
  const float c = scale * LOG2E;
  const bool live = key < len;   // a masked key has probability 0 against every query
  f32x16_t dk[NB], dv[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    zero16(dk[i]);
    zero16(dv[i]);
  }
  const bool wg_live = rb * ROWS_WG < len;   // a workgroup whose keys are all masked only writes zeros
  const size_t stat0 = ((size_t)b * H + hd) * Tn;
  const float *dobase = dout + (size_t)b * Tn * D + hd * dh;

  const float *obase = o + (size_t)b * Tn * D + hd * dh;

  TileRegsF<DH, KG> tq, tdo;
  float rl = INFINITY, rd = 0.f;   // lse and delta of a query of the tile, held by the first of its TPR threads
  constexpr int TPR = NT / TILE;   // threads that share a query's delta = dO . O
  const int drow = threadIdx.x / TPR, dpart = threadIdx.x % TPR;
  auto load_tile = [&](int q0) {
    const int nvalid = min(TILE, Tn - q0);
    tq.load(base + (size_t)q0 * ld, ld, nvalid, dh);
    tdo.load(dobase + (size_t)q0 * D, (size_t)D, nvalid, dh);
    const bool ok = drow < nvalid;
    rl = ok ? lse[stat0 + q0 + drow] * LOG2E : INFINITY;   // exp2(-inf) = 0 beyond T
    rd = 0.f;
    if constexpr (!OWN_DELTA) {
      if (ok) rd = delta[stat0 + q0 + drow];
      return;
    }
    if (ok) {
      const size_t at = (size_t)(q0 + drow) * D;
#pragma unroll
      for (int i = 0; i < DH / 4 / TPR; ++i) {
        const int ch = (dpart + i * TPR) * 4;
        if (ch < dh) {
          const float4 x = *reinterpret_cast<const float4 *>(dobase + at + ch), y = *reinterpret_cast<const float4 *>(obase + at + ch);
          rd += (x.x * y.x + x.y * y.y) + (x.z * y.z + x.w * y.w);
        }
      }
    }
    rd += dpp_lane<0xB1>(rd);                       // the TPR = 2, 4 or 8 lanes are neighbours
    if constexpr (TPR >= 4) rd += dpp_lane<0x4E>(rd);
    if constexpr (TPR >= 8) rd += dpp_lane<0x141>(rd);
  };
  // causal: only queries at or after a key see it
  const int qbeg = CAUSAL ? (int)(rb * ROWS_WG) / TILE * TILE : 0;
  const int wkey0 = rb * ROWS_WG + wave.rg * 32;
  if (wg_live) load_tile(qbeg);
  for (int q0 = qbeg; wg_live && q0 < Tn; q0 += TILE) {
    __syncthreads();
    tq.store(sQ);
    tdo.store(sDO);
    if (dpart == 0) {
      sL[drow] = rl;
      sDl[drow] = rd;
    }
    __syncthreads();
    if (q0 + TILE < Tn) load_tile(q0 + TILE);
#pragma unroll
    for (int qb = wave.kg; qb < TILE / 32; qb += KG) {
      if (q0 + qb * 32 >= Tn) break;
      if (CAUSAL && q0 + qb * 32 + 31 < wkey0) continue;
      f32x16_t s, dp;
      zero16(s);
      zero16(dp);
      s = row_dot<DH>(sQ + (qb * 32 + l32) * ST + h2 * 4, kf, s);      // S[q, key]
      dp = row_dot<DH>(sDO + (qb * 32 + l32) * ST + h2 * 4, vf, dp);   // dP[q, key]
      float kp[4][4];
      if constexpr (DROP) {
#pragma unroll
        for (int g = 0; g < 4; ++g)
          drop_keep_rows4(drop, (uint32_t)key, (uint32_t)(q0 + qb * 32 + g * 8 + h2 * 4), (uint32_t)(b * H + hd), kp[g]);
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int qi = qb * 32 + acc_row(r, h2);
        const float p = (live && (!CAUSAL || q0 + qi >= key)) ? exp2f(s[r] * c - sL[qi]) : 0.f;
        float keep = 1.f;
        if constexpr (DROP) keep = kp[r >> 2][r & 3];
        dp[r] = p * (dp[r] * keep - sDl[qi]);   // dS
        s[r] = p * keep;                        // dV sees the dropped-out probabilities
      }
#pragma unroll
      for (int db = 0; db < NB; ++db)
#pragma unroll
        for (int t = 0; t < 16; ++t) {
          const int row = (qb * 32 + acc_row(t, h2)) * ST + db * 32 + l32;
          dv[db] = mfma2(sDO[row], s[t], dv[db]);    // dV^T[d, key] += dO^T[d, q] P[q, key]
          dk[db] = mfma2(sQ[row], dp[t], dk[db]);    // dK^T[d, key] += Q^T[d, q] dS[q, key]
        }
    }
  }
  if constexpr (KG > 1) {
    float wk[KG], wv[KG];
#pragma unroll
    for (int k = 0; k < KG; ++k) wk[k] = scale, wv[k] = 1.f;
    float *row = dqkv + ((size_t)b * Tn + key) * ld + D + hd * dh;
#pragma unroll
    for (int part = 0; part < 2; ++part) {
      __syncthreads();   // the tiles, then the first part's sums, are no longer being read
      park<NB, KG>(smem, part == 0 ? dk : dv);
      __syncthreads();
#pragma unroll
      for (int db = 0; db < NB; ++db)
#pragma unroll
        for (int i = 0; i < 4 / KG; ++i) {
          const int qd = wave.kg * (4 / KG) + i;
          float v[4];
          gather<NB, KG>(smem, wave.rg, db, qd, part == 0 ? wk : wv, v);
          if (kok && db * 32 + qd * 8 + h2 * 4 < dh) VecIO<float, 4>::store(row + part * D + db * 32 + qd * 8 + h2 * 4, v);
        }
    }
    return;
  }
  if (kok) {
    float *dkrow = dqkv + ((size_t)b * Tn + key) * ld + D + hd * dh;
    float *dvrow = dkrow + D;
#pragma unroll
    for (int db = 0; db < NB; ++db)
#pragma unroll
      for (int qd = 0; qd < 4; ++qd) {
        float a[4] = {dk[db][qd * 4] * scale, dk[db][qd * 4 + 1] * scale, dk[db][qd * 4 + 2] * scale,
                      dk[db][qd * 4 + 3] * scale};
        float v[4] = {dv[db][qd * 4], dv[db][qd * 4 + 1], dv[db][qd * 4 + 2], dv[db][qd * 4 + 3]};
        if (db * 32 + qd * 8 + h2 * 4 < dh) {
          VecIO<float, 4>::store(dkrow + db * 32 + qd * 8 + h2 * 4, a);
          VecIO<float, 4>::store(dvrow + db * 32 + qd * 8 + h2 * 4, v);
        }
      }
  }
}

template <int DH, bool CAUSAL, bool DROP, int KG>
__global__ __launch_bounds__(NT) void attn_bwd_dq_mfma_f32(const float *__restrict__ qkv, const float *__restrict__ o,
                                                           const float *__restrict__ dout, const float *__restrict__ lse,
                                                           const int32_t *__restrict__ lengths, DropSpec drop, int Tn, int H,
                                                           int dh, float scale, float *__restrict__ dqkv,
                                                           float *__restrict__ delta) {
  extern __shared__ __attribute__((aligned(16))) float smem[];
  dq_block<DH, CAUSAL, DROP, KG, true>(attn_block<CAUSAL>(), smem, qkv, o, dout, lse, lengths, drop, Tn, H, dh, scale, dqkv, delta);
}
template <int DH, bool CAUSAL, bool DROP, int KG>
__global__ __launch_bounds__(NT) void attn_bwd_dkv_mfma_f32(const float *__restrict__ qkv, const float *__restrict__ dout,
                                                            const float *__restrict__ lse, const float *__restrict__ delta,
                                                            const int32_t *__restrict__ lengths, DropSpec drop, int Tn, int H,
                                                            int dh, float scale, float *__restrict__ dqkv) {
  extern __shared__ __attribute__((aligned(16))) float smem[];
  dkv_block<DH, CAUSAL, DROP, KG, false>(attn_block<CAUSAL>(), smem, qkv, nullptr, dout, lse, lengths, drop, Tn, H, dh, scale, dqkv, delta);
}
// dQ and dK/dV in one launch, for problems whose workgroups all run at once: they only share their inputs (each computes
// the delta it needs), and side by side they take the time of the longer instead of the sum (8 x 128 tokens, 4 heads of
// 64: 22.7 -> 14.5 us; with more workgroups than CUs the larger of the two register budgets costs more than that: 4 x
// 1000, 8 heads of 64: 301 -> 383).  The first nrb_q row blocks of a (batch, head) are dQ's.
template <int DH, bool CAUSAL, bool DROP, int KG>
__global__ __launch_bounds__(NT) void attn_bwd_both_mfma_f32(const float *__restrict__ qkv, const float *__restrict__ o,
                                                             const float *__restrict__ dout, const float *__restrict__ lse,
                                                             const int32_t *__restrict__ lengths, DropSpec drop, int Tn, int H,
                                                             int dh, float scale, float *__restrict__ dqkv, int nrb_q) {
  extern __shared__ __attribute__((aligned(16))) float smem[];
  AttnBlock blk = attn_block<false>();
  if (blk.rb < nrb_q) {
    dq_block<DH, CAUSAL, DROP, KG, false>(blk, smem, qkv, o, dout, lse, lengths, drop, Tn, H, dh, scale, dqkv, nullptr);
  } else {
    blk.rb -= nrb_q;
    dkv_block<DH, CAUSAL, DROP, KG, true>(blk, smem, qkv, o, dout, lse, lengths, drop, Tn, H, dh, scale, dqkv, nullptr);
  }
}

// The most wavefronts on one group of rows that an instance takes: beyond, the tiles in flight (registers) spill.
template <int DH> constexpr int MAX_DQ = DH <= 96 ? 4 : 2;
template <int DH> constexpr int MAX_DKV = DH <= 64 ? 4 : DH <= 96 ? 2 : 1;
// How many wavefronts share a group of rows: more than one where 128-row workgroups leave SIMDs without a wavefront (and
// never more than there are 32-row blocks to share).  Forward / backward in us at KG = 1, 2, 4: 32 workgroups (8 x 128
// tokens, 4 heads of 64) 15.0, 10.1, 7.6 / 47.9, 31.6, 22.7; 96 (3 x 489, 8 of 32) 29.6, 18.3, 17.8 / 93, 57, 52;
// 128 (16 x 128, 8 of 64) 15.3, 10.8, 14.0 / 49, 34, 44; 264 (22 x 115, 12 of 64) 25.7, 24.2, 31.8 / 91, 83, 103.
// One wavefront per 32 rows and scalar operand reads, as before: 18.5 / 62 on the first.
int key_groups(int B, int T, int H) {
  const int forced = forced_f32_key_groups();
  if (forced) return forced;
  if (T <= 32) return 1;
  const long wgs = (long)B * H * ((T + 127) / 128);   // workgroups at KG = 1
  return wgs <= 96 && T > 64 ? 4 : wgs <= 288 ? 2 : 1;
}

template <typename K> hipError_t raise_lds(K kern, size_t lds, bool &raised) {
  if (lds <= 64 * 1024 || raised) return hipSuccess;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  raised = e == hipSuccess;
  return e;
}

template <int DH, bool CAUSAL, bool DROP, int KG>
hipError_t fwd_k(const float *qkv, const int32_t *lengths, const DropSpec &drop, int B, int T, int H, int dh, float scale,
                 float *o, float *lse, hipStream_t s) {
  constexpr size_t lds = f32_lds_floats<DH, KG>() * sizeof(float);
  static_assert(lds <= 160 * 1024, "the tiles fit in LDS");
  static bool raised = false;
  hipError_t e = raise_lds(attn_fwd_mfma_f32<DH, CAUSAL, DROP, KG>, lds, raised);
  if (e != hipSuccess) return e;
  dim3 grid((T + rows_wg(KG) - 1) / rows_wg(KG), H, B);
  hipLaunchKernelGGL((attn_fwd_mfma_f32<DH, CAUSAL, DROP, KG>), grid, dim3(NT), lds, s, qkv, lengths, drop, T, H, dh, scale, o, lse);
  return hipGetLastError();
}
template <int DH, bool CAUSAL, bool DROP, int KG>
hipError_t dq_k(const float *qkv, const float *o, const float *dout, const float *lse, const int32_t *lengths,
                const DropSpec &drop, int B, int T, int H, int dh, float scale, float *dqkv, float *delta, hipStream_t s) {
  constexpr size_t lds = f32_lds_floats<DH, KG>() * sizeof(float);
  static bool raised = false;
  auto kern = attn_bwd_dq_mfma_f32<DH, CAUSAL, DROP, KG>;
  hipError_t e = raise_lds(kern, lds, raised);
  if (e != hipSuccess) return e;
  dim3 grid((T + rows_wg(KG) - 1) / rows_wg(KG), H, B);
  hipLaunchKernelGGL(kern, grid, dim3(NT), lds, s, qkv, o, dout, lse, lengths, drop, T, H, dh, scale, dqkv, delta);
  return hipGetLastError();
}
template <int DH, bool CAUSAL, bool DROP, int KG>
hipError_t dkv_k(const float *qkv, const float *dout, const float *lse, const float *delta, const int32_t *lengths,
                 const DropSpec &drop, int B, int T, int H, int dh, float scale, float *dqkv, hipStream_t s) {
  constexpr size_t lds = f32_lds_floats<DH, KG>() * sizeof(float);
  static bool raised = false;
  auto kern = attn_bwd_dkv_mfma_f32<DH, CAUSAL, DROP, KG>;
  hipError_t e = raise_lds(kern, lds, raised);
  if (e != hipSuccess) return e;
  dim3 grid((T + rows_wg(KG) - 1) / rows_wg(KG), H, B);
  hipLaunchKernelGGL(kern, grid, dim3(NT), lds, s, qkv, dout, lse, delta, lengths, drop, T, H, dh, scale, dqkv);
  return hipGetLastError();
}
template <int DH, bool CAUSAL, bool DROP, int KG>
hipError_t both_k(const float *qkv, const float *o, const float *dout, const float *lse, const int32_t *lengths,
                  const DropSpec &drop, int B, int T, int H, int dh, float scale, float *dqkv, hipStream_t s) {
  constexpr size_t lds = f32_lds_floats<DH, KG>() * sizeof(float);
  static bool raised = false;
  auto kern = attn_bwd_both_mfma_f32<DH, CAUSAL, DROP, KG>;
  hipError_t e = raise_lds(kern, lds, raised);
  if (e != hipSuccess) return e;
  const int nrb = (T + rows_wg(KG) - 1) / rows_wg(KG);
  hipLaunchKernelGGL(kern, dim3(2 * nrb, H, B), dim3(NT), lds, s, qkv, o, dout, lse, lengths, drop, T, H, dh, scale, dqkv, nrb);
  return hipGetLastError();
}

template <int DH, bool CAUSAL, bool DROP>
hipError_t fwd_t(const float *qkv, const int32_t *lengths, const DropSpec &drop, int B, int T, int H, int dh, float scale,
                 float *o, float *lse, hipStream_t s) {
  switch (key_groups(B, T, H)) {
    case 4: return fwd_k<DH, CAUSAL, DROP, 4>(qkv, lengths, drop, B, T, H, dh, scale, o, lse, s);
    case 2: return fwd_k<DH, CAUSAL, DROP, 2>(qkv, lengths, drop, B, T, H, dh, scale, o, lse, s);
    default: return fwd_k<DH, CAUSAL, DROP, 1>(qkv, lengths, drop, B, T, H, dh, scale, o, lse, s);
  }
}
template <int DH, bool CAUSAL, bool DROP>
hipError_t bwd_t(const float *qkv, const float *o, const float *dout, const float *lse, const int32_t *lengths,
                 const DropSpec &drop, int B, int T, int H, int dh, float scale, float *dqkv, float *delta, hipStream_t s) {
  const int kg = key_groups(B, T, H);
  if constexpr (DH <= 64) {
    if (2l * B * H * ((T + rows_wg(kg) - 1) / rows_wg(kg)) <= 256) switch (kg) {
      case 4: return both_k<DH, CAUSAL, DROP, 4>(qkv, o, dout, lse, lengths, drop, B, T, H, dh, scale, dqkv, s);
      case 2: return both_k<DH, CAUSAL, DROP, 2>(qkv, o, dout, lse, lengths, drop, B, T, H, dh, scale, dqkv, s);
      default: return both_k<DH, CAUSAL, DROP, 1>(qkv, o, dout, lse, lengths, drop, B, T, H, dh, scale, dqkv, s);
    }
  }
  constexpr int QMAX = MAX_DQ<DH>, KMAX = MAX_DKV<DH>;
  hipError_t e;
  if (kg == 4 && QMAX == 4) e = dq_k<DH, CAUSAL, DROP, QMAX>(qkv, o, dout, lse, lengths, drop, B, T, H, dh, scale, dqkv, delta, s);
  else if (kg >= 2) e = dq_k<DH, CAUSAL, DROP, 2>(qkv, o, dout, lse, lengths, drop, B, T, H, dh, scale, dqkv, delta, s);
  else e = dq_k<DH, CAUSAL, DROP, 1>(qkv, o, dout, lse, lengths, drop, B, T, H, dh, scale, dqkv, delta, s);
  if (e != hipSuccess) return e;
  if (kg >= KMAX) return dkv_k<DH, CAUSAL, DROP, KMAX>(qkv, dout, lse, delta, lengths, drop, B, T, H, dh, scale, dqkv, s);
  if (kg == 2) return dkv_k<DH, CAUSAL, DROP, (KMAX > 2 ? 2 : KMAX)>(qkv, dout, lse, delta, lengths, drop, B, T, H, dh, scale, dqkv, s);
  return dkv_k<DH, CAUSAL, DROP, 1>(qkv, dout, lse, delta, lengths, drop, B, T, H, dh, scale, dqkv, s);
}

template <int DH>
hipError_t fwd_pick(int causal, const float *qkv, const int32_t *lengths, const DropSpec &drop, int B, int T, int H,
                    int dh, float scale, float *o, float *lse, hipStream_t s) {
  if (causal)
    return drop.thr ? fwd_t<DH, true, true>(qkv, lengths, drop, B, T, H, dh, scale, o, lse, s)
                    : fwd_t<DH, true, false>(qkv, lengths, drop, B, T, H, dh, scale, o, lse, s);
  return drop.thr ? fwd_t<DH, false, true>(qkv, lengths, drop, B, T, H, dh, scale, o, lse, s)
                  : fwd_t<DH, false, false>(qkv, lengths, drop, B, T, H, dh, scale, o, lse, s);
}

template <int DH>
hipError_t bwd_pick(int causal, const float *qkv, const float *o, const float *dout, const float *lse,
                    const int32_t *lengths, const DropSpec &drop, int B, int T, int H, int dh, float scale,
                    float *dqkv, float *delta, hipStream_t s) {
  if (causal)
    return drop.thr ? bwd_t<DH, true, true>(qkv, o, dout, lse, lengths, drop, B, T, H, dh, scale, dqkv, delta, s)
                    : bwd_t<DH, true, false>(qkv, o, dout, lse, lengths, drop, B, T, H, dh, scale, dqkv, delta, s);
  return drop.thr ? bwd_t<DH, false, true>(qkv, o, dout, lse, lengths, drop, B, T, H, dh, scale, dqkv, delta, s)
                  : bwd_t<DH, false, false>(qkv, o, dout, lse, lengths, drop, B, T, H, dh, scale, dqkv, delta, s);
}

}  // namespace

bool attention_mfma_f32_supported(int dh) { return dh >= 16 && dh <= 128 && dh % 16 == 0; }

hipError_t launch_attention_fwd_mfma_f32(const void *qkv, const int32_t *lengths, int causal, const DropSpec &drop,
                                         int B, int T, int H, int dh, void *o, float *lse, hipStream_t s) {
  const float scale = 1.0f / sqrtf((float)dh);
  const float *x = static_cast<const float *>(qkv);
  float *y = static_cast<float *>(o);
  if (!attention_mfma_f32_supported(dh)) return hipErrorInvalidValue;
  switch ((dh + 31) / 32) {
    case 1: return fwd_pick<32>(causal, x, lengths, drop, B, T, H, dh, scale, y, lse, s);
    case 2: return fwd_pick<64>(causal, x, lengths, drop, B, T, H, dh, scale, y, lse, s);
    case 3: return fwd_pick<96>(causal, x, lengths, drop, B, T, H, dh, scale, y, lse, s);
    case 4: return fwd_pick<128>(causal, x, lengths, drop, B, T, H, dh, scale, y, lse, s);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_attention_bwd_mfma_f32(const void *qkv, const void *o, const void *dout, const float *lse,
                                         const int32_t *lengths, int causal, const DropSpec &drop, int B, int T, int H,
                                         int dh, void *dqkv, float *delta, hipStream_t s) {
  const float scale = 1.0f / sqrtf((float)dh);
  const float *x = static_cast<const float *>(qkv), *oo = static_cast<const float *>(o);
  const float *g = static_cast<const float *>(dout);
  float *dx = static_cast<float *>(dqkv);
  if (!attention_mfma_f32_supported(dh)) return hipErrorInvalidValue;
  switch ((dh + 31) / 32) {
    case 1: return bwd_pick<32>(causal, x, oo, g, lse, lengths, drop, B, T, H, dh, scale, dx, delta, s);
    case 2: return bwd_pick<64>(causal, x, oo, g, lse, lengths, drop, B, T, H, dh, scale, dx, delta, s);
    case 3: return bwd_pick<96>(causal, x, oo, g, lse, lengths, drop, B, T, H, dh, scale, dx, delta, s);
    case 4: return bwd_pick<128>(causal, x, oo, g, lse, lengths, drop, B, T, H, dh, scale, dx, delta, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace fl
