// Pipelined bf16 MFMA GEMM for gfx950 (same contraction and epilogue as gemm.hip;
// this is the kernel the layer's large GEMMs run on).
//
//   C[M,N] = sum_k A(m,k) B(n,k),  k-range a multiple of 64.
//
// * Operand tiles travel HBM/L2 -> LDS with the direct-to-LDS load
//   (global_load_lds_dwordx4): no VGPRs and no LDS-write instructions are spent on
//   staging, so NS stages (k-tiles) can be in flight; one workgroup barrier per k-tile.
//   A wave-level load writes 64 consecutive 16-byte chunks of LDS; WHICH global chunk a
//   lane fetches is free, and that is where the bank-conflict swizzle is applied:
//     k-contiguous tile  [rows][64 k]   : chunk c of row r sits at position c ^ ((r>>1)&7)
//     k-major tile       [64 k][rows]   : chunk c of k-row k sits at position c ^ km_swizzle(k)
//   Both make the MFMA fragment reads (16-byte row reads, and the transposing
//   ds_read_b64_tr_b16 for k-major tiles) touch every bank once per 32 lanes.
// * Rows past the end of an operand are clamped to the last valid row (their products land in
//   output rows/columns that are never stored), so no lane ever reads out of bounds.
// * 256 threads = 4 wavefronts in a 2x2 grid over a BM x BN tile (other grids: see the instances in
//   launch_layout); each wavefront owns
//   (BM/2) x (BN/2) = TM x TN MFMA tiles of 32x32 (v_mfma_f32_32x32x16_bf16), issued as
//   D = B_frag x A_frag so that a lane ends with four consecutive n of one m.
#include "devutil.h"
#include "gemm_dev.h"
#include "kernels.h"
#include "lds_dma.h"

namespace fl {
namespace {

constexpr int KT = 64;

typedef __attribute__((address_space(3))) void *lds_void_ptr;
typedef const __attribute__((address_space(1))) void *glb_void_ptr;
typedef __attribute__((address_space(3))) s16x4_t *lds_s16x4_ptr;

template <int N> __device__ __forceinline__ void wait_vmcnt_le() { FL_WAIT_VMCNT(N); }

// Chunk swizzle of a k-major tile of R rows.  A transposing read touches 64 bytes of each of four consecutive k-rows,
// which must fall into different quarters of the 256 bytes of banks: rows of a multiple of 256 bytes (R = 128, 256) need
// all four shifted apart, rows of an odd multiple of 128 (R = 192) the two pairs, odd multiples of 64 none.
template <int R> __device__ __forceinline__ int km_swizzle(int k) {
  return R % 128 == 0 ? (k & 3) << 2 : R % 64 == 0 ? ((k >> 1) & 1) << 2 : 0;
}

// One operand's staging plan for this wave: element offsets (from the operand base) of the chunks
// its lanes fetch, for each of its NOPS wave-level loads per k-tile.
template <bool KC, int R, int NW> struct Stager {
  static constexpr int NOPS = R / (8 * NW);  // R*128 bytes per stage / 1 KiB per load / NW waves
  int off[NOPS];
  int kstep;  // element offset from one k-tile to the next
  __device__ __forceinline__ void init(int ld, int row0, int nrows, int kbeg, int lane, int wave) {
#pragma unroll
    for (int j = 0; j < NOPS; ++j) {
      const int P = (wave + NW * j) * 64 + lane;  // chunk position inside the stage
      if (KC) {
        const int r = P >> 3, c = (P & 7) ^ ((r >> 1) & 7);
        off[j] = min(row0 + r, nrows - 1) * ld + kbeg + c * 8;
      } else {
        constexpr int CPR = R / 8;
        const int k = P / CPR, c = (P % CPR) ^ km_swizzle<R>(k);
        off[j] = (kbeg + k) * ld + min(row0 + c * 8, nrows - 8);
      }
    }
    kstep = KC ? KT : KT * ld;
  }
  // stage_lds: LDS byte address of the stage's first byte; wave: wave-uniform (a scalar)
  __device__ __forceinline__ void issue(const bf16_t *base, int kt, unsigned stage_lds, int wave) const {
#pragma unroll
    for (int j = 0; j < NOPS; ++j) {
      const bf16_t *src = base + (size_t)off[j] + (size_t)kt * kstep;
      lds_dma16(src, stage_lds + (unsigned)(wave + NW * j) * 1024u);
    }
  }
};

// Fragment (32 rows starting at tile row r0, k-step kk) out of a swizzled stage.
template <bool KC, int R>
__device__ __forceinline__ bf16x8_t frag(const unsigned char *stage, int r0, int kk, int lane) {
  if (KC) {
    const int r = r0 + (lane & 31);
    const int c = (kk * 2 + (lane >> 5)) ^ ((r >> 1) & 7);
    return *reinterpret_cast<const bf16x8_t *>(stage + r * 128 + c * 16);
  } else {
    const int g = lane >> 4, s = lane & 15;
    const int kb = kk * 16 + (g >> 1) * 8 + (s >> 2);
    const int rowpos = r0 + (g & 1) * 16 + 4 * (s & 3);
    const int c = (rowpos >> 3) ^ km_swizzle<R>(kb);
    const unsigned char *a = stage + kb * (R * 2) + c * 16 + (rowpos & 7) * 2;
    s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)a);
    s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(a + 4 * R * 2));
    typedef short s16x8_t __attribute__((ext_vector_type(8)));
    s16x8_t v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8_t, v);
  }
}

// WM x WN wavefronts share a BM x BN tile; each owns TM x TN MFMA tiles of 32x32.  KG > 1: KG such
// groups of wavefronts work on the same tile, group g taking the g-th part of every k-tile, and their
// accumulators are added through LDS at the end, half of the tile by either group.  For outputs with few tiles (one workgroup per CU)
// this puts two wavefronts on every SIMD, so that one's LDS reads overlap the other's MFMAs.
template <bool AKC, bool BKC, int BM, int BN, int NS, int WM, int WN, bool DROP, int KG, int EPI = EPI_FULL>
__global__ __launch_bounds__(WM *WN *KG * 64) void gemm_bf16_pipe(GemmDev p) {
  constexpr int NW = WM * WN * KG;
  constexpr int KKS = KT / 16 / KG;  // 16-wide k-steps of a k-tile per group
  static_assert(KKS >= 1 && KKS * KG * 16 == KT, "k-groups must divide the k-tile");
  constexpr int TM = BM / (32 * WM), TN = BN / (32 * WN);
  constexpr int A_BYTES = BM * 128, STAGE = (BM + BN) * 128;
  constexpr int OPS = Stager<AKC, BM, NW>::NOPS + Stager<BKC, BN, NW>::NOPS;  // loads per wave per k-tile
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];

  int split, tile_m, tile_n;
  xcd_work_coords(blockIdx.x, p.tiles_m, p.tiles_n, p.splits, 1024 / BM, split, tile_m, tile_n);
  const int row0 = tile_m * BM, col0 = tile_n * BN;
  const int kbeg = split * p.k_per_split;
  if (p.partial) p.partial += (size_t)split * p.M * p.N;
  const int kend = min(p.K, kbeg + p.k_per_split);
  const int nk = (kend - kbeg) / KT;
  const bf16_t *A = static_cast<const bf16_t *>(p.A);
  const bf16_t *B = static_cast<const bf16_t *>(p.B);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // in a scalar register: LDS addresses below are scalars too
  const unsigned smem_lds = lds_address(smem);
  const int kg = wave / (WM * WN), wpos = wave % (WM * WN);  // k-group, position in the tile
  const int wm = wpos / WN, wn = wpos % WN;

  Stager<AKC, BM, NW> sa;
  Stager<BKC, BN, NW> sb;
  sa.init(p.lda, row0, p.M, kbeg, lane, wave);
  sb.init(p.ldb, col0, p.N, kbeg, lane, wave);

  f32x16_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  // prologue: NS-1 k-tiles in flight
#pragma unroll
  for (int s = 0; s < NS - 1; ++s) {
    if (s < nk) {
      sa.issue(A, s, smem_lds + s * STAGE, wave);
      sb.issue(B, s, smem_lds + s * STAGE + A_BYTES, wave);
    }
  }
  for (int kt = 0; kt < nk; ++kt) {
    // k-tile kt must have landed: allow the loads of the (up to NS-2) younger k-tiles to stay in flight
    const int younger = min(NS - 2, nk - 1 - kt);
    if (NS >= 4 && younger >= 2) wait_vmcnt_le<2 * OPS>();
    else if (NS >= 3 && younger == 1) wait_vmcnt_le<OPS>();
    else wait_vmcnt_le<0>();
    // every wave's part of k-tile kt is in LDS; everyone is done reading k-tile kt-1.  A bare
    // s_barrier: __syncthreads() would add a fence that waits for ALL loads, younger k-tiles included.
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (kt + NS - 1 < nk) {
      const unsigned st = smem_lds + ((kt + NS - 1) % NS) * STAGE;
      sa.issue(A, kt + NS - 1, st, wave);
      sb.issue(B, kt + NS - 1, st + A_BYTES, wave);
    }
    const unsigned char *sA = smem + (kt % NS) * STAGE, *sB = sA + A_BYTES;
    // fragments of k-step kk+1 are requested before the MFMAs of k-step kk are issued.  Left to itself the
    // scheduler sinks those reads behind the MFMAs and into the registers the MFMAs have just read, so that
    // every k-step waits out a full LDS round trip; the scheduling barriers keep the two groups apart where
    // the wavefront tile is small enough for the second fragment set to cost no occupancy.
    constexpr bool PIN = TM * TN <= 4;
    bf16x8_t fa[2][TM], fb[2][TN];
    const int kk0 = kg * KKS;
#pragma unroll
    for (int i = 0; i < TM; ++i) fa[0][i] = frag<AKC, BM>(sA, wm * (BM / WM) + i * 32, kk0, lane);
#pragma unroll
    for (int j = 0; j < TN; ++j) fb[0][j] = frag<BKC, BN>(sB, wn * (BN / WN) + j * 32, kk0, lane);
#pragma unroll
    for (int kk = 0; kk < KKS; ++kk) {
      if (kk + 1 < KKS) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
          fa[(kk + 1) & 1][i] = frag<AKC, BM>(sA, wm * (BM / WM) + i * 32, kk0 + kk + 1, lane);
#pragma unroll
        for (int j = 0; j < TN; ++j)
          fb[(kk + 1) & 1][j] = frag<BKC, BN>(sB, wn * (BN / WN) + j * 32, kk0 + kk + 1, lane);
      }
      if constexpr (PIN) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[kk & 1][j], fa[kk & 1][i], acc[i][j], 0, 0, 0);
      if constexpr (PIN) __builtin_amdgcn_sched_barrier(0);
    }
  }

  // Epilogue through LDS (see gemm_staged_epilogue): the operand stages are reused.
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();  // every wave is done reading the operand stages
  asm volatile("" ::: "memory");
  if constexpr (KG == 2) {
    // each group finishes half of the tile's 32-row blocks: it parks its sums of the other half in LDS ([position][register]
    // [lane]: lane-contiguous, no bank conflicts), adds the other group's to its own, and both walk the epilogue
    static_assert(TM == 2, "one block of rows for each group");
    constexpr int PER_WAVE = TN * 16 * 64;
    float *red = reinterpret_cast<float *>(smem) + (size_t)wpos * PER_WAVE + lane;
    float *dst = red + (size_t)kg * (WM * WN) * PER_WAVE;
    const float *src = red + (size_t)(1 - kg) * (WM * WN) * PER_WAVE;
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) dst[(j * 16 + r) * 64] = kg == 0 ? acc[1][j][r] : acc[0][j][r];
    __syncthreads();
    f32x16_t fin[1][TN];
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) fin[0][j][r] = (kg == 0 ? acc[0][j][r] : acc[1][j][r]) + src[(j * 16 + r) * 64];
    __syncthreads();  // the epilogue's staging area overlaps what other wavefronts have just read
    float *cw = reinterpret_cast<float *>(smem) + (size_t)wave * 32 * (TN * 32 + 4);
    gemm_staged_epilogue<bf16_t, 1, TN, DROP, EPI>(p, fin, cw, row0 + wm * (BM / WM) + kg * 32, col0 + wn * (BN / WN), lane);
  } else {
    static_assert(KG == 1, "one or two k-groups");
    float *cw = reinterpret_cast<float *>(smem) + (size_t)wpos * 32 * (TN * 32 + 4);
    gemm_staged_epilogue<bf16_t, TM, TN, DROP, EPI>(p, acc, cw, row0 + wm * (BM / WM), col0 + wn * (BN / WN), lane);
  }
}

template <bool AKC, bool BKC, int BM, int BN, int NS, int WM, int WN, bool DROP, int KG, int EPI = EPI_FULL>
hipError_t launch_cfg_d(GemmDev d, int splits, hipStream_t s) {
  constexpr size_t stage_lds = (size_t)NS * (BM + BN) * 128;
  constexpr size_t epi_lds = (size_t)WM * WN * KG * 32 * (BN / WN + 4) * sizeof(float);
  constexpr size_t red_lds = KG > 1 ? (size_t)BM * BN * sizeof(float) : 0;
  constexpr size_t lds0 = stage_lds > epi_lds ? stage_lds : epi_lds;
  constexpr size_t lds = lds0 > red_lds ? lds0 : red_lds;
  static_assert(lds <= 160 * 1024, "stages do not fit in LDS");
  auto kern = gemm_bf16_pipe<AKC, BKC, BM, BN, NS, WM, WN, DROP, KG, EPI>;
  if (lds > 64 * 1024) {
    static bool raised = false;
    if (!raised) {
      hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                         hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      if (e != hipSuccess) return e;
      raised = true;
    }
  }
  d.tiles_m = (d.M + BM - 1) / BM;
  d.tiles_n = (d.N + BN - 1) / BN;
  d.splits = splits;
  dim3 grid(d.tiles_m * d.tiles_n * splits);
  hipLaunchKernelGGL(kern, grid, dim3(WM * WN * KG * 64), lds, s, d);
  return hipGetLastError();
}

// the epilogue kinds of the instances the layer runs on (see gemm_epi_kind), with or without the dropout steps
template <bool AKC, bool BKC, int BM, int BN, int NS, int WM, int WN, int KG, bool DROP>
hipError_t launch_kind(const GemmDev &d, int splits, hipStream_t s) {
  const int kind = gemm_epi_kind(d.partial != nullptr, d.act, d.dact, d.preact != nullptr);
  if (kind == EPI_PLAIN) return launch_cfg_d<AKC, BKC, BM, BN, NS, WM, WN, DROP, KG, EPI_PLAIN>(d, splits, s);
  if (!DROP && kind == EPI_PARTIAL) return launch_cfg_d<AKC, BKC, BM, BN, NS, WM, WN, false, KG, EPI_PARTIAL>(d, splits, s);
  if (kind == EPI_LIGHT) return launch_cfg_d<AKC, BKC, BM, BN, NS, WM, WN, DROP, KG, EPI_LIGHT>(d, splits, s);
  if (kind == EPI_GELU_FWD) return launch_cfg_d<AKC, BKC, BM, BN, NS, WM, WN, DROP, KG, EPI_GELU_FWD>(d, splits, s);
  if (kind == EPI_GELU_BWD) return launch_cfg_d<AKC, BKC, BM, BN, NS, WM, WN, DROP, KG, EPI_GELU_BWD>(d, splits, s);
  return launch_cfg_d<AKC, BKC, BM, BN, NS, WM, WN, DROP, KG>(d, splits, s);
}
template <bool AKC, bool BKC, int BM, int BN, int NS, int WM = 2, int WN = 2, int KG = 1>
hipError_t launch_cfg(const GemmDev &d, int splits, hipStream_t s) {
  constexpr bool specialised = (BM == 128 && BN == 128 && WM == 2 && WN == 2 && ((NS == 2 && KG == 1) || (NS == 3 && KG == 2))) ||
                               (BM == 256 && BN == 192) || (BN == 128 && (BM == 160 || BM == 96)) || (BM == 256 && BN == 256 && WN == 4);
  if (d.drop_where) {   // (see gemm_pipe_takes_dropout)
    if constexpr (AKC && specialised && (BM <= 160 || BN == 192)) return launch_kind<AKC, BKC, BM, BN, NS, WM, WN, KG, true>(d, splits, s);
    else return hipErrorInvalidValue;
  }
  if constexpr (specialised) return launch_kind<AKC, BKC, BM, BN, NS, WM, WN, KG, false>(d, splits, s);
  else return launch_cfg_d<AKC, BKC, BM, BN, NS, WM, WN, false, KG>(d, splits, s);
}

template <bool AKC, bool BKC>
hipError_t launch_layout(const GemmDev &d, int splits, int variant, hipStream_t s) {
  switch (variant) {
    case 0: return launch_cfg<AKC, BKC, 128, 128, 2>(d, splits, s);
    case 1: return launch_cfg<AKC, BKC, 128, 128, 4>(d, splits, s);
    case 2: return launch_cfg<AKC, BKC, 256, 128, 3>(d, splits, s);
    case 3: return launch_cfg<AKC, BKC, 256, 128, 2>(d, splits, s);
    case 4: return launch_cfg<AKC, BKC, 256, 256, 2>(d, splits, s);
    case 5: return launch_cfg<AKC, BKC, 256, 256, 2, 2, 4>(d, splits, s);
    case 6: return launch_cfg<AKC, BKC, 256, 128, 3, 4, 2>(d, splits, s);
    case 8: return launch_cfg<AKC, BKC, 128, 128, 2, 2, 2, 2>(d, splits, s);
    case 9: return launch_cfg<AKC, BKC, 128, 128, 3, 2, 2, 2>(d, splits, s);
    case 10:
      if constexpr (AKC) return launch_cfg<AKC, BKC, 160, 128, 2, 1, 4>(d, splits, s);
      else return hipErrorInvalidValue;
    case 11:
      if constexpr (AKC) return launch_cfg<AKC, BKC, 96, 128, 2, 1, 4>(d, splits, s);
      else return hipErrorInvalidValue;
    case 7:  // used for y = x W^T and dx = dy W only
      if constexpr (AKC) return launch_cfg<AKC, BKC, 256, 192, 2, 4, 2>(d, splits, s);
      else return hipErrorInvalidValue;
  }
  return hipErrorInvalidValue;
}

}  // namespace

bool gemm_pipe_eligible(const GemmArgs &a, int kps) {
  // whole k-tiles only; operands must hold at least one full 8-element chunk per clamped row
  return kps % KT == 0 && a.K % KT == 0 && a.M >= 8 && a.N >= 8 && (long)a.M * a.lda < (1l << 31) &&
         (long)a.N * a.ldb < (1l << 31) && (long)a.K * (a.a_kc ? 1 : a.lda) < (1l << 31) &&
         (long)a.K * (a.b_kc ? 1 : a.ldb) < (1l << 31);
}

void gemm_pipe_tile(int variant, int *bm, int *bn) {
  static const int t[12][2] = {{128, 128}, {128, 128}, {256, 128}, {256, 128}, {256, 256}, {256, 256}, {256, 128}, {256, 192}, {128, 128}, {128, 128}, {160, 128}, {96, 128}};
  *bm = t[variant][0];
  *bn = t[variant][1];
}

// dropout steps in the epilogue: not with the large wavefront tiles, which have no registers for the generator
bool gemm_pipe_takes_dropout(int variant) { return variant == 0 || variant == 7 || variant == 9 || variant == 10 || variant == 11; }

namespace {
// Time of a launch that has the chip to itself, in us: tiles per CU (of the fullest) x k-tiles x what a CU takes for one
// k-tile of one tile, plus a fixed part (per tile, where a CU holds one workgroup).  Fitted to launches of 4096-16384
// rows, N, K = 768..4096, k-contiguous and k-major B alike (they do not differ); within 6 % of all of them.
double pipe_time(int variant, int M, int N, int K) {
  int bm, bn;
  gemm_pipe_tile(variant, &bm, &bn);
  const double n = (double)(((long)((M + bm - 1) / bm) * ((N + bn - 1) / bn) + 255) / 256), nk = K / (double)KT;
  switch (variant) {
    case 0: return 4.0 + n * nk * 0.617;
    case 5: return n * (8.2 + nk * 1.65);
    case 7: return n * (8.5 + nk * 1.06);
    case 9: return n * (5.2 + nk * 0.54);
    case 10: return 5.5 + n * nk * (n > 2 ? 0.70 : 0.59);
    case 11: return 5.5 + n * nk * (n > 2 ? 0.515 : 0.42);
  }
  return 1e30;
}
// What was found by hand inside whole training steps.
int pipe_base_variant(bool b_kc, int M, int N, bool alone) {
  // More 128x128 tiles than the chip holds at two workgroups per CU, but not with 160x128 tiles: one round
  // instead of one and a bit (12608 x 768 outputs: 594 tiles against 474; dy W at k = 3072 / 2304 / 768 alone:
  // 83 -> 66, 64 -> 51, 28 -> 22 us).
  const long slots = 512, tiles128 = (long)((M + 127) / 128) * ((N + 127) / 128);
  const bool one_round_160 = tiles128 > slots && (long)((M + 159) / 160) * ((N + 127) / 128) <= slots;
  // One round of 128x128 tiles that leaves a quarter of the places empty, where 96x128 tiles fill them (8000 x 768
  // outputs: 378 tiles against 504; on their own 57 -> 48, 42 -> 38, 20 -> 17.5 us at k = 3072 / 2304 / 768).  Only with
  // more tiles than CUs (below that the two-k-group variant is ahead), and only for a launch that has the chip to itself.
  const bool one_round_96 = alone && tiles128 > 256 && 5 * tiles128 <= 4 * slots && (long)((M + 95) / 96) * ((N + 127) / 128) <= slots;
  if (one_round_160) return 10;
  if (b_kc && N % 192 == 0) {
    // 256x192 tiles on 8 wavefronts halve the L1 and LDS traffic per flop and win when they fill the
    // chip in whole rounds (one workgroup per CU); otherwise 128x128 / 2 stages, two workgroups per CU.
    const long tiles = (long)((M + 255) / 256) * (N / 192), rounds = (tiles + 255) / 256;
    if (tiles >= 160 && 100 * tiles >= (rounds == 1 ? 74 : 90) * rounds * 256) return 7;
  }
  // at most one 128x128 tile per CU: three stages and two k-groups of wavefronts per tile (eight wavefronts on
  // the CU instead of four) keep more loads in flight.
  if (b_kc && tiles128 <= 256) return 9;
  return one_round_96 ? 11 : 0;
}
}  // namespace

int gemm_pipe_pick_variant(bool a_kc, bool b_kc, int M, int N, int K, bool alone, bool drop) {
  const int forced = forced_gemm_pipe_variant();
  if (forced != -1) return forced >= 7 && forced != 8 && forced != 9 && !a_kc ? -2 : forced;
  if (!a_kc) return b_kc ? -2 : 0;
  const int base = pipe_base_variant(b_kc, M, N, alone);
  // Another variant where the time model says that it is clearly ahead: 16384 x 4096 x 1024 on 256x256 tiles 158 -> 141
  // us, 12608 x 3072 x 768 on 160x128 79 -> 74, 4096 x 3072 x 768 with a k-major B on 256x192 29 -> 24.
  const int all[6] = {0, 5, 7, 9, 10, 11};
  int best = drop && !gemm_pipe_takes_dropout(base) ? 0 : base;
  double best_us = pipe_time(best, M, N, K) * (alone ? 0.95 : 0.90);
  for (int v : all) {
    if (drop && !gemm_pipe_takes_dropout(v)) continue;
    if (!alone && v == 11) continue;
    // columns of 192 that are not full: 7420 x 1024 x 4096 takes 94 us on 256x192 tiles (76 by the model), 83 on 128x128
    if (v == 7 && N % 192) continue;
    const double us = pipe_time(v, M, N, K);
    if (us < best_us) best_us = us, best = v;
  }
  return best;
}

hipError_t launch_gemm_bf16_pipe(const GemmArgs &a, const void *dev, int splits, int variant, hipStream_t s) {
  const GemmDev &d = *static_cast<const GemmDev *>(dev);
  if (a.a_kc && a.b_kc) return launch_layout<true, true>(d, splits, variant, s);
  if (a.a_kc && !a.b_kc) return launch_layout<true, false>(d, splits, variant, s);
  if (!a.a_kc && !a.b_kc) return launch_layout<false, false>(d, splits, variant, s);
  return launch_layout<false, true>(d, splits, variant, s);
}

}  // namespace fl
