// All weight gradients of a backward pass in one launch (bf16): out[N, K] = sum over tokens of gy[m, n] x[m, k] for up
// to DW_MAX_JOBS problems with one token count, plus the column sums that ride along (see gemm_dw.h).
//
// The main loop is that of gemm_pipe.hip with both operands k-major: token tiles of 64 travel to LDS with
// direct-to-LDS loads as they lie in memory ([64 tokens][rows], 16-byte chunk c of token t at c ^ ((t & 3) << 2)) and
// are read with the transposing ds_read_b64_tr_b16.  What bounds it per k-tile and CU is the L1 feed on small tiles
// and the matrix cores on large ones: 128 x 128 tiles take 0.56 us (3.7 TFLOP/s per CU), 256 x 128 on eight wavefronts
// 0.94 us (4.5), 256 x 256 1.41 us (6.0).  Alone on the chip there is no second kernel to leave room for, so the
// tile and the token split are picked by those rates (dw_plan).
// A token count that is not a multiple of 64: the last k-tile's rows past the end are fetched from the last token and
// zeroed in the fragments of gy and x (0 times an infinity of the last token would be a NaN).
#include "gemm_dw.h"
#include "lds_dma.h"

namespace fl {
namespace {

constexpr int KT = 64;
template <int N> __device__ __forceinline__ void wait_vmcnt_le() { FL_WAIT_VMCNT(N); }

template <int R, int NW> struct Stager {
  static constexpr int NOPS = R / (8 * NW), CPR = R / 8;
  int off[NOPS];
  static __device__ __forceinline__ int token(int j, int lane, int wave) { return ((wave + NW * j) * 64 + lane) / CPR; }
  __device__ __forceinline__ void init(int ld, int row0, int nrows, int lane, int wave) {
#pragma unroll
    for (int j = 0; j < NOPS; ++j) {
      const int P = (wave + NW * j) * 64 + lane, k = P / CPR, c = (P % CPR) ^ ((k & 3) << 2);
      off[j] = k * ld + min(row0 + c * 8, nrows - 8);
    }
  }
  __device__ __forceinline__ void issue(const bf16_t *base, int ld, int k0, int kend, unsigned lds, int lane, int wave) const {
    const bf16_t *src = base + (size_t)k0 * ld;
    if (k0 + KT <= kend) {
#pragma unroll
      for (int j = 0; j < NOPS; ++j) lds_dma16(src + off[j], lds + (unsigned)(wave + NW * j) * 1024u);
    } else {
#pragma unroll
      for (int j = 0; j < NOPS; ++j) {
        const int over = k0 + token(j, lane, wave) - (kend - 1);
        lds_dma16(src + off[j] - (over > 0 ? (size_t)over * ld : 0), lds + (unsigned)(wave + NW * j) * 1024u);
      }
    }
  }
};

template <int R> __device__ __forceinline__ bf16x8_t frag(const unsigned char *stage, int r0, int kk, int lane) {
  typedef __attribute__((address_space(3))) s16x4_t *lds_s16x4_ptr;
  typedef short s16x8_t __attribute__((ext_vector_type(8)));
  const int g = lane >> 4, s = lane & 15;
  const int kb = kk * 16 + (g >> 1) * 8 + (s >> 2), row = r0 + (g & 1) * 16 + 4 * (s & 3);
  const int c = (row >> 3) ^ ((kb & 3) << 2);
  const unsigned char *a = stage + kb * (R * 2) + c * 16 + (row & 7) * 2;
  const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)a);
  const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(a + 4 * R * 2));
  const s16x8_t v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_bit_cast(bf16x8_t, v);
}

template <int BM, int BN, int NS, int WM, int WN, bool PARTIAL>
__global__ __launch_bounds__(WM *WN * 64) void gemm_dw_pipe(DwDev d) {
  constexpr int NW = WM * WN, TM = BM / (32 * WM), TN = BN / (32 * WN);
  constexpr int A_BYTES = BM * 128, STAGE = (BM + BN) * 128;
  typedef Stager<BM, NW> SA;
  typedef Stager<BN, NW> SB;
  constexpr int OPS = SA::NOPS + SB::NOPS;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const int tiles = d.first[d.njobs] * d.splits;
  if ((int)blockIdx.x >= tiles) {
    dw_columns<bf16_t, NW * 64>(d, blockIdx.x - tiles, reinterpret_cast<float *>(smem));
    return;
  }
  GemmDev p;
  int tile_m, tile_n, kbeg, kend;
  dw_tile(d, blockIdx.x, 1024 / BM, p, tile_m, tile_n, kbeg, kend);
  const int row0 = tile_m * BM, col0 = tile_n * BN, nk = (kend - kbeg + KT - 1) / KT;
  const bf16_t *A = static_cast<const bf16_t *>(p.A), *B = static_cast<const bf16_t *>(p.B);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const unsigned smem_lds = lds_address(smem);
  const int wm = wave / WN, wn = wave % WN;
  SA sa;
  SB sb;
  sa.init(p.lda, row0, p.M, lane, wave);
  sb.init(p.ldb, col0, p.N, lane, wave);
  auto issue = [&](int kt) {
    const unsigned st = smem_lds + (kt % NS) * STAGE;
    sa.issue(A, p.lda, kbeg + kt * KT, kend, st, lane, wave);
    sb.issue(B, p.ldb, kbeg + kt * KT, kend, st + A_BYTES, lane, wave);
  };
  f32x16_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
#pragma unroll
  for (int s = 0; s < NS - 1; ++s)
    if (s < nk) issue(s);
  for (int kt = 0; kt < nk; ++kt) {
    if (NS >= 3 && kt + 1 < nk) wait_vmcnt_le<OPS>();   // the younger k-tile may stay in flight
    else wait_vmcnt_le<0>();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();   // k-tile kt is in LDS, and everyone is done with k-tile kt-1
    asm volatile("" ::: "memory");
    if (kt + NS - 1 < nk) issue(kt + NS - 1);
    const unsigned char *sA = smem + (kt % NS) * STAGE, *sB = sA + A_BYTES;
    constexpr bool PIN = TM * TN <= 4;
    bf16x8_t fa[2][TM], fb[2][TN];
    auto read = [&](int kk) {
#pragma unroll
      for (int i = 0; i < TM; ++i) fa[kk & 1][i] = frag<BM>(sA, wm * (BM / WM) + i * 32, kk, lane);
#pragma unroll
      for (int j = 0; j < TN; ++j) fb[kk & 1][j] = frag<BN>(sB, wn * (BN / WN) + j * 32, kk, lane);
    };
    const bool ragged = kbeg + (kt + 1) * KT > kend;
    read(0);
#pragma unroll
    for (int kk = 0; kk < KT / 16; ++kk) {
      if (kk + 1 < KT / 16) read(kk + 1);
      if constexpr (PIN) __builtin_amdgcn_sched_barrier(0);
      if (ragged) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int e = 0; e < 8; ++e)
            if (kbeg + kt * KT + kk * 16 + (lane >> 5) * 8 + e >= kend) {
              fa[kk & 1][i][e] = (bf16_t)0.f;
#pragma unroll
              for (int j = 0; j < TN; ++j) fb[kk & 1][j][e] = (bf16_t)0.f;
            }
      }
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[kk & 1][j], fa[kk & 1][i], acc[i][j], 0, 0, 0);
      if constexpr (PIN) __builtin_amdgcn_sched_barrier(0);
    }
  }
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();   // every wavefront is done reading the operand stages
  asm volatile("" ::: "memory");
  float *cw = reinterpret_cast<float *>(smem) + (size_t)wave * 32 * (TN * 32 + 4);
  gemm_staged_epilogue<bf16_t, TM, TN, false, PARTIAL ? EPI_PARTIAL : EPI_PLAIN>(p, acc, cw, row0 + wm * (BM / WM), col0 + wn * (BN / WN), lane);
}

template <int BM, int BN, int NS, int WM, int WN, bool PARTIAL>
hipError_t launch_p(const DwJob *jobs, int njobs, const ColJob *cols, int ncols, int M, int splits, bool accumulate, hipStream_t s) {
  constexpr size_t stages = (size_t)NS * (BM + BN) * 128, epi = (size_t)WM * WN * 32 * (BN / WN + 4) * sizeof(float);
  constexpr size_t lds = stages > epi ? stages : epi;
  static_assert(lds <= 160 * 1024 && lds >= (size_t)WM * WN * 64 * 8 * sizeof(float), "stages and column sums fit in LDS");
  auto kern = gemm_dw_pipe<BM, BN, NS, WM, WN, PARTIAL>;
  if (lds > 64 * 1024) {
    static bool raised = false;
    if (!raised) {
      hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      if (e != hipSuccess) return e;
      raised = true;
    }
  }
  DwDev d;
  const int grid = dw_fill(d, jobs, njobs, cols, ncols, M, splits, KT, BM, BN, accumulate);
  hipLaunchKernelGGL(kern, dim3(grid), dim3(WM * WN * 64), lds, s, d);
  return hipGetLastError();
}
template <int BM, int BN, int NS, int WM, int WN>
hipError_t launch_t(const DwJob *jobs, int njobs, const ColJob *cols, int ncols, int M, int splits, bool accumulate, hipStream_t s) {
  return splits > 1 ? launch_p<BM, BN, NS, WM, WN, true>(jobs, njobs, cols, ncols, M, splits, accumulate, s)
                    : launch_p<BM, BN, NS, WM, WN, false>(jobs, njobs, cols, ncols, M, splits, accumulate, s);
}

long tiles_of(const DwJob *jobs, int n, int bm, int bn) {
  long t = 0;
  for (int j = 0; j < n; ++j) t += (long)((jobs[j].N + bm - 1) / bm) * ((jobs[j].K + bn - 1) / bn);
  return t;
}

// kernel of a plan: its tile, the part of a launch that does not depend on the tokens, and microseconds per k-tile (64
// tokens; fp32: 32) of a CU that works on one tile, and per tile when it works on several
struct DwKernel { int bm, bn; double fix, one, more; };
const DwKernel kBf16[5] = {{256, 256, 8.0, 1.60, 1.60}, {256, 128, 7.0, 1.05, 1.05}, {128, 128, 6.0, 0.56, 0.56}, {64, 64, 4.5, 0.20, 0.20}, {32, 32, 3.5, 0.10, 0.16}};
const DwKernel kF32[2] = {{64, 64, 5.0, 0.53, 0.72}, {32, 32, 3.5, 0.18, 0.24}};

}  // namespace

// The kernel and token split with the least time by that table, splits paying for their partial sums (written and read
// at 5 TB/s) and a second launch.  BERT-base shape (4096 tokens): 256 x 128 unsplit, 76 us where the four launches and
// their second stages took 124; 12608 tokens: 256 x 256 in two ranges, 190 us against 250.
DwPlan dw_plan(int dt, const DwJob *jobs, int njobs, int M) {
  DwPlan best{dt == DT_F32 ? DW_SMALL32 : DW_128, 1};
  const int forced = forced_dw_kernel();
  double best_us = 1e30;
  long elems = 0;
  for (int j = 0; j < njobs; ++j) elems += (long)jobs[j].N * jobs[j].K;
  for (int k = 0; k < 5; ++k) {
    if (forced >= 0 ? k != forced : dt == DT_F32 && k < DW_SMALL64) continue;
    const DwKernel &K = dt == DT_F32 ? kF32[k - DW_SMALL64] : kBf16[k];
    const int kt = dt == DT_F32 ? 32 : KT, nk = (M + kt - 1) / kt;
    const long tiles = tiles_of(jobs, njobs, K.bm, K.bn);
    for (int s = 1; s <= 16 && s <= nk; ++s) {
      const int per_split = (nk + s - 1) / s;
      if ((long)(s - 1) * per_split >= nk) continue;   // an empty range
      const long n = (tiles * s + 255) / 256;          // tiles of the fullest CU
      double us = K.fix + n * per_split * (n > 1 ? K.more : K.one) + (n - 1) * (k <= DW_256x128 ? K.fix : 1.0);
      if (s > 1) us += 5.0 + (double)elems * s * 8 / 5.0e6;
      if (us < best_us) best_us = us, best = {k, s};
    }
  }
  return best;
}

hipError_t launch_dw_batch(int dt, const DwPlan &plan, const DwJob *jobs, int njobs, const ColJob *cols, int ncols, int M,
                           bool accumulate, hipStream_t s) {
  if (njobs < 1 || njobs > DW_MAX_JOBS || ncols < 0 || ncols > DW_MAX_COLS || M < 1 || plan.splits < 1) return hipErrorInvalidValue;
  for (int j = 0; j < njobs; ++j) {
    const DwJob &J = jobs[j];
    if (!J.gy || !J.x || !J.out || (plan.splits > 1 && !J.partial) || J.N < 8 || J.K < 8 || J.N % 8 || J.K % 8)
      return hipErrorInvalidValue;
  }
  for (int j = 0; j < ncols; ++j)
    if (!cols[j].in || !cols[j].out || cols[j].rows < 1 || cols[j].n < 8 || cols[j].n % 8 || cols[j].ld % 8) return hipErrorInvalidValue;
  switch (plan.kernel) {
    case DW_SMALL32: return launch_dw_small(dt, 32, jobs, njobs, cols, ncols, M, plan.splits, accumulate, s);
    case DW_SMALL64: return launch_dw_small(dt, 64, jobs, njobs, cols, ncols, M, plan.splits, accumulate, s);
  }
  if (dt != DT_BF16) return hipErrorInvalidValue;
  switch (plan.kernel) {
    case DW_256: return launch_t<256, 256, 2, 2, 4>(jobs, njobs, cols, ncols, M, plan.splits, accumulate, s);
    case DW_256x128: return launch_t<256, 128, 3, 4, 2>(jobs, njobs, cols, ncols, M, plan.splits, accumulate, s);
    case DW_128: return launch_t<128, 128, 2, 2, 2>(jobs, njobs, cols, ncols, M, plan.splits, accumulate, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace fl
