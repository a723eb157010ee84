// Body of the GEMM kernels for problems with few output tiles (fp32 and bf16): C[M,N] = sum_k A(m,k) B(n,k) on
// tiles of (TM*32) x (TN*32) whose W wavefronts SPLIT K.  Shared by the single-problem kernel (gemm_small.hip) and
// the kernel that runs all weight gradients of a layer in one launch (gemm_dw_small.hip).
//
// What bounds such a problem is not the matrix cores but how long one workgroup takes to pull its operand panels
// and how many CUs pull at the same time.  So: tiles small enough that most CUs get one; and every wavefront walks
// k-tiles of its own (wavefront w takes k-tiles w, w + W, ...) through a private piece of LDS, so that the operand
// bytes of a tile are fetched once, no barrier separates the k-tiles, and W * S k-tiles are in flight per
// workgroup.  A k-tile is 128 bytes of k per row (64 bf16, 32 fp32) and travels with direct-to-LDS loads; it is
// read into registers in one go, and the next one is requested before its MFMAs are issued.  The W partial
// accumulators meet in LDS at the end (fixed order), where every thread of the workgroup picks up eight
// consecutive outputs for the epilogue.
//
// LDS layouts (16-byte chunks, one wavefront's private tile):
//   k-contiguous operand [rows][128 B]:   chunk c of row r sits at c ^ ((r >> 1) & 7); a fragment is one 16-byte
//     read per lane.  For fp32 the four values of a lane's chunk feed four MFMAs of two k each: both operands
//     enumerate k in the same order, and a sum does not care which.
//   k-major operand [k][rows]: as it lies in memory; bf16 fragments through the transposing read
//     (ds_read_b64_tr_b16), whose 32-lane halves touch four k-rows of 64 bytes each: with 64-row tiles those would
//     share banks, so chunk c of k-row k sits at c ^ (((k >> 1) & 1) << 2); fp32 fragments are single words.
#pragma once
#include "devutil.h"
#include "gemm_dev.h"
#include "lds_dma.h"

namespace fl {

template <typename T> struct KTile;   // V: a lane's part of a fragment
template <> struct KTile<bf16_t> { static constexpr int KT = 64, EPC = 8; typedef bf16x8_t V; };
template <> struct KTile<float> { static constexpr int KT = 32, EPC = 4; typedef f32x4_t V; };

// One operand of a wavefront's private k-tile: TR*32 rows.
template <typename T, bool KC, int TR> struct SmallFeed {
  static constexpr int EPC = KTile<T>::EPC, KT = KTile<T>::KT, R = TR * 32;
  static constexpr int NOPS = TR * 4;         // TR*32 rows * 128 bytes / 1 KiB per wave-level load
  static constexpr int BYTES = R * 128;
  static constexpr int CPR = R / EPC;         // k-major: chunks per k-row
  static constexpr bool SWZ = !KC && sizeof(T) == 2 && TR == 2;
  int off[NOPS];
  static __device__ __forceinline__ int chunk_k(int j, int lane) {   // first k of this lane's chunk inside the tile
    if (KC) return ((lane & 7) ^ (((j * 8 + (lane >> 3)) >> 1) & 7)) * EPC;
    return (j * 64 + lane) / CPR;
  }
  __device__ __forceinline__ void init(int ld, int row0, int nrows, int lane) {
#pragma unroll
    for (int j = 0; j < NOPS; ++j) {
      const int P = j * 64 + lane;
      if (KC) {
        off[j] = min(row0 + (P >> 3), nrows - 1) * ld + chunk_k(j, lane);
      } else {
        const int k = P / CPR, c = (P % CPR) ^ (SWZ ? ((k >> 1) & 1) << 2 : 0);
        off[j] = k * ld + min(row0 + c * EPC, nrows - EPC);
      }
    }
  }
  // Requests the k-tile that starts at k0.  Chunks past kend are fetched from the last valid place instead (their
  // products are masked out by the reader).
  __device__ __forceinline__ void issue(const T *base, int ld, int k0, int kend, unsigned lds, int lane) const {
    const T *src = base + (KC ? (size_t)k0 : (size_t)k0 * ld);
    if (k0 + KT <= kend) {
#pragma unroll
      for (int j = 0; j < NOPS; ++j) lds_dma16(src + off[j], lds + j * 1024u);
    } else {
#pragma unroll
      for (int j = 0; j < NOPS; ++j) {
        const int over = k0 + chunk_k(j, lane) - (KC ? kend - EPC : kend - 1);
        lds_dma16(src + off[j] - (over > 0 ? (KC ? over : over * ld) : 0), lds + j * 1024u);
      }
    }
  }
  // Fragment of the 32 rows of block i at step kk (two chunks of k: lane half h holds chunk kk*2 + h).
  static __device__ __forceinline__ typename KTile<T>::V frag(const unsigned char *t, int i, int kk, int lane) {
    typedef typename KTile<T>::V V;
    if constexpr (KC) {
      const int r = i * 32 + (lane & 31), c = (kk * 2 + (lane >> 5)) ^ ((r >> 1) & 7);
      return *reinterpret_cast<const V *>(t + r * 128 + c * 16);
    } else if constexpr (sizeof(T) == 2) {
      typedef __attribute__((address_space(3))) s16x4_t *lds_s16x4_ptr;
      typedef short s16x8_t __attribute__((ext_vector_type(8)));
      const int g = lane >> 4, s = lane & 15;
      const int kb = kk * 16 + (g >> 1) * 8 + (s >> 2), row = i * 32 + (g & 1) * 16 + 4 * (s & 3);
      const int c = (row >> 3) ^ (SWZ ? ((kb >> 1) & 1) << 2 : 0);
      const unsigned char *a = t + kb * (R * 2) + c * 16 + (row & 7) * 2;
      const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)a);
      const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(a + 4 * R * 2));
      const s16x8_t v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
      return __builtin_bit_cast(V, v);
    } else {
      const float *f = reinterpret_cast<const float *>(t) + (kk * 2 + (lane >> 5)) * 4 * R + i * 32 + (lane & 31);
      return V{f[0], f[R], f[2 * R], f[3 * R]};
    }
  }
};

template <typename T, int TM, int TN, int W, int S> constexpr int small_slot_bytes() { return (TM + TN) * 4096 * S; }
template <typename T, int TM, int TN, int W, int S> constexpr size_t small_lds_bytes() {
  return (size_t)W * small_slot_bytes<T, TM, TN, W, S>();   // the accumulators (TM*TN*4 KiB per wavefront) fit: TM*TN <= TM+TN
}

// One tile: rows row0.., columns col0.., k in [kbeg, kend).  p.partial, if set, already points at the k-range's slab.
template <typename T, bool AKC, bool BKC, int TM, int TN, int W, int S, bool DROP, int EPI>
__device__ __forceinline__ void gemm_small_tile(const GemmDev &p, int row0, int col0, int kbeg, int kend,
                                                unsigned char *smem) {
  static_assert(TM * TN <= (TM + TN) * S, "the accumulators reuse the operand tiles' LDS");
  static_assert(S == 1 || S == 2, "one or two k-tiles in flight per wavefront");
  typedef SmallFeed<T, AKC, TM> FA;
  typedef SmallFeed<T, BKC, TN> FB;
  typedef typename KTile<T>::V V;
  constexpr int KT = KTile<T>::KT, EPC = KTile<T>::EPC, NTHR = W * 64;
  constexpr int SLOT = small_slot_bytes<T, TM, TN, W, S>(), STAGE = FA::BYTES + FB::BYTES;
  constexpr int OPS = FA::NOPS + FB::NOPS;
  constexpr int OPR = TN * 4, OCTS = TM * 32 * OPR, NOCT = (OCTS + NTHR - 1) / NTHR;   // octs: eight outputs of a row
  const int lane = threadIdx.x & 63, h2 = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const T *A = static_cast<const T *>(p.A), *B = static_cast<const T *>(p.B);
  FA fa;
  FB fb;
  fa.init(p.lda, row0, p.M, lane);
  fb.init(p.ldb, col0, p.N, lane);
  const unsigned lds = lds_address(smem) + wave * SLOT;
  auto issue = [&](int k0, int st) {
    fa.issue(A, p.lda, k0, kend, lds + st * STAGE, lane);
    fb.issue(B, p.ldb, k0, kend, lds + st * STAGE + FA::BYTES, lane);
  };
  int k0 = kbeg + wave * KT;
#pragma unroll
  for (int s = 0; s < S; ++s)
    if (k0 + s * W * KT < kend) issue(k0 + s * W * KT, s);

  f32x16_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  for (int it = 0; k0 < kend; k0 += W * KT, ++it) {
    const int st = S == 1 ? 0 : (it & 1);
    if (S == 2 && k0 + W * KT < kend) FL_WAIT_VMCNT(OPS);   // the younger k-tile stays in flight
    else FL_WAIT_VMCNT(0);
    asm volatile("" ::: "memory");
    const unsigned char *tA = smem + wave * SLOT + st * STAGE, *tB = tA + FA::BYTES;
    V va[4][TM], vb[4][TN];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
#pragma unroll
      for (int i = 0; i < TM; ++i) va[kk][i] = FA::frag(tA, i, kk, lane);
#pragma unroll
      for (int j = 0; j < TN; ++j) vb[kk][j] = FB::frag(tB, j, kk, lane);
    }
    if (k0 + S * W * KT < kend) {   // refill this stage: its contents are in registers once the reads are done
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
#pragma unroll
        for (int i = 0; i < TM; ++i) asm volatile("" : "+v"(va[kk][i]));
#pragma unroll
        for (int j = 0; j < TN; ++j) asm volatile("" : "+v"(vb[kk][j]));
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      issue(k0 + S * W * KT, st);
    }
    if (k0 + KT > kend) {   // the ragged last k-tile: what lies past the end of k counts as zero
#pragma unroll
      for (int kk = 0; kk < 4; ++kk)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int e = 0; e < EPC; ++e)
            if (k0 + (kk * 2 + h2) * EPC + e >= kend) {
              va[kk][i][e] = T(0.f);
#pragma unroll
              for (int j = 0; j < TN; ++j) vb[kk][j][e] = T(0.f);
            }
    }
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          // D = B_frag x A_frag: register q*4+e of a lane ends up as C[i*32 + lane%32, j*32 + q*8 + (lane/32)*4 + e]
          if constexpr (sizeof(T) == 2) {
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vb[kk][j], va[kk][i], acc[i][j], 0, 0, 0);
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(vb[kk][j][e], va[kk][i][e], acc[i][j], 0, 0, 0);
          }
        }
  }

  // What the epilogue reads from memory is requested before the accumulators are exchanged.
  float bias8[NOCT][8];
  bf16x8_t pre_res[NOCT], pre_aux[NOCT];
  constexpr bool PRE = sizeof(T) == 2 && EPI != EPI_PARTIAL;
#pragma unroll
  for (int o = 0; o < NOCT; ++o) {
    const int t = threadIdx.x + o * NTHR, m = row0 + t / OPR, n0 = col0 + (t % OPR) * 8;
    const bool ok = t < OCTS && m < p.M && n0 < p.N && EPI != EPI_PARTIAL && !p.partial;
#pragma unroll
    for (int e = 0; e < 8; ++e) bias8[o][e] = 0.f;
    pre_res[o] = bf16x8_t{};
    pre_aux[o] = bf16x8_t{};
    if (ok && p.bias) Oct<T>::load(static_cast<const T *>(p.bias) + n0, bias8[o]);
    if constexpr (PRE) {
      const size_t at = (size_t)m * p.ldc + n0;
      if (ok && p.residual) pre_res[o] = *reinterpret_cast<const bf16x8_t *>(static_cast<const bf16_t *>(p.residual) + at);
      if (EPI != EPI_PLAIN && EPI != EPI_GELU_FWD && ok && p.dact)
        pre_aux[o] = *reinterpret_cast<const bf16x8_t *>(static_cast<const bf16_t *>(p.aux) + at);
    }
  }
  // Accumulators to LDS, one TM*TN*4 KiB tile per wavefront, row-major, float4 chunk c of row r at c ^ (r % chunks):
  // every wavefront overwrites its own operand tiles only, which nobody else reads.
  constexpr int CH = TN * 8;   // float4 chunks of a row
  float *mine = reinterpret_cast<float *>(smem + wave * SLOT);
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int r = i * 32 + (lane & 31), c = (j * 8 + q * 2 + h2) ^ (r & (CH - 1));
        *reinterpret_cast<float4 *>(mine + (r * CH + c) * 4) =
            make_float4(acc[i][j][q * 4], acc[i][j][q * 4 + 1], acc[i][j][q * 4 + 2], acc[i][j][q * 4 + 3]);
      }
  static_assert((CH & (CH - 1)) == 0, "the swizzle needs a power of two");
  __syncthreads();
#pragma unroll
  for (int o = 0; o < NOCT; ++o) {
    const int t = threadIdx.x + o * NTHR, r = t / OPR, c8 = t % OPR;
    const int m = row0 + r, n0 = col0 + c8 * 8;
    if (t < OCTS && m < p.M && n0 < p.N) {
      float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      const int c0 = (c8 * 2) ^ (r & (CH - 1)), c1 = (c8 * 2 + 1) ^ (r & (CH - 1));
#pragma unroll
      for (int w = 0; w < W; ++w) {   // fixed order: the result does not depend on timing
        const float *s = reinterpret_cast<const float *>(smem + w * SLOT) + r * CH * 4;
        const float4 lo = *reinterpret_cast<const float4 *>(s + c0 * 4), hi = *reinterpret_cast<const float4 *>(s + c1 * 4);
        v[0] += lo.x; v[1] += lo.y; v[2] += lo.z; v[3] += lo.w;
        v[4] += hi.x; v[5] += hi.y; v[6] += hi.z; v[7] += hi.w;
      }
      gemm_epilogue_oct<T, DROP, PRE, PRE, EPI>(p, m, n0, v, bias8[o], pre_res[o], pre_aux[o]);
    }
  }
}

}  // namespace fl
