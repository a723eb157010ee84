// GEMM for problems with few output tiles, fp32 and bf16: y = x W^T and dx = dy W on tiles of 32x32 to 64x64 whose four
// wavefronts split k (see gemm_small.h for the kernel's body and why).
#include "gemm_small.h"
#include "kernels.h"

namespace fl {
namespace {

template <typename T, bool AKC, bool BKC, int TM, int TN, int W, int S, bool DROP, int EPI>
__global__ __launch_bounds__(W * 64) void gemm_small(GemmDev p) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  int split, tile_m, tile_n;
  xcd_work_coords(blockIdx.x, p.tiles_m, p.tiles_n, p.splits, 1024 / (TM * 32), split, tile_m, tile_n);
  const int kbeg = split * p.k_per_split, kend = min(p.K, kbeg + p.k_per_split);
  if (p.partial) p.partial += (size_t)split * p.M * p.N;
  gemm_small_tile<T, AKC, BKC, TM, TN, W, S, DROP, EPI>(p, tile_m * TM * 32, tile_n * TN * 32, kbeg, kend, smem);
}

template <typename T, bool AKC, bool BKC, int TM, int TN, int W, int S, bool DROP, int EPI>
hipError_t launch_k(GemmDev d, int splits, hipStream_t s) {
  constexpr size_t lds = small_lds_bytes<T, TM, TN, W, S>();
  static_assert(lds <= 160 * 1024, "the wavefronts' k-tiles fit in LDS");
  auto kern = gemm_small<T, AKC, BKC, TM, TN, W, S, DROP, EPI>;
  if (lds > 64 * 1024) {
    static bool raised = false;
    if (!raised) {
      hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      if (e != hipSuccess) return e;
      raised = true;
    }
  }
  d.tiles_m = (d.M + TM * 32 - 1) / (TM * 32);
  d.tiles_n = (d.N + TN * 32 - 1) / (TN * 32);
  d.splits = splits;
  hipLaunchKernelGGL(kern, dim3(d.tiles_m * d.tiles_n * splits), dim3(W * 64), lds, s, d);
  return hipGetLastError();
}

// the epilogue kinds exist apart for bf16, where the instances' straight-line code matters (see gemm_dev.h)
template <typename T, bool AKC, bool BKC, int TM, int TN, int W, int S>
hipError_t launch_e(const GemmDev &d, int splits, hipStream_t s) {
  if (d.drop_where) return launch_k<T, AKC, BKC, TM, TN, W, S, true, EPI_FULL>(d, splits, s);
  if constexpr (sizeof(T) == 2) {
    const int kind = gemm_epi_kind(d.partial != nullptr, d.act, d.dact, d.preact != nullptr);
    if (kind == EPI_PLAIN) return launch_k<T, AKC, BKC, TM, TN, W, S, false, EPI_PLAIN>(d, splits, s);
    if (kind == EPI_LIGHT) return launch_k<T, AKC, BKC, TM, TN, W, S, false, EPI_LIGHT>(d, splits, s);
    if (kind == EPI_GELU_FWD) return launch_k<T, AKC, BKC, TM, TN, W, S, false, EPI_GELU_FWD>(d, splits, s);
    if (kind == EPI_GELU_BWD) return launch_k<T, AKC, BKC, TM, TN, W, S, false, EPI_GELU_BWD>(d, splits, s);
  }
  return launch_k<T, AKC, BKC, TM, TN, W, S, false, EPI_FULL>(d, splits, s);
}
// (A is k-contiguous in both of the layouts that come here: y = x W^T and dx = dy W)
template <typename T, int TM, int TN, int W, int S>
hipError_t launch_l(const GemmArgs &a, const GemmDev &d, int splits, hipStream_t s) {
  return a.b_kc ? launch_e<T, true, true, TM, TN, W, S>(d, splits, s) : launch_e<T, true, false, TM, TN, W, S>(d, splits, s);
}
template <typename T>
hipError_t launch_v(const GemmArgs &a, const GemmDev &d, int splits, int v, hipStream_t s) {
  switch (v) {
    case 0: return launch_l<T, 1, 1, 4, 2>(a, d, splits, s);
    case 1: return launch_l<T, 1, 2, 4, 1>(a, d, splits, s);
    case 2: return launch_l<T, 2, 2, 4, 1>(a, d, splits, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace

// The variant for a problem (0: 32x32 tiles, 1: 32x64, 2: 64x64), or -1 where the larger tiles of the other kernels
// are ahead.  By time, as measured on 400 shapes of M = 16..3000 tokens (N, K from d_model 256..1024), in us:
//   bf16: a fixed part plus the operand bytes that the fullest CU pulls at 85 KB/us (32x32 tiles 50 when a CU gets
//   several); the 128x128 tiles of gemm_pipe.hip: 4.6 us plus 69 KB/us.  24 x 768 x 3072: 26.8 -> 5.7; 744 x 768 x
//   3072: 28.3 -> 13.0; 1001 x 2048 x 512: 8.9 -> 7.2.
//   fp32: a fixed part plus the matrix cores' time for the fullest CU's tiles, 5-7.5 ns per k and 32x32 block (the
//   64 x 64 tiles reuse fragments: 4.1, 6.1 where a CU gets several).  1024 x 256 x 1024: 12.4 -> 8.9; 2048 x 512 x 2048: 51 -> 39.
int gemm_small_pick(int dt, bool a_kc, int M, int N, int K, bool pipe_eligible, bool gelu) {
  if (!a_kc) return -1;
  const int rows[3] = {64, 96, 128};
  const long tm32 = (M + 31) / 32, tn32 = (N + 31) / 32, tn64 = (N + 63) / 64, tm64 = (M + 63) / 64;
  const long tiles[3] = {tm32 * tn32, tm32 * tn64, tm64 * tn64};
  int best = -1;
  double best_us = 1e30;
  for (int v = 0; v < 3; ++v) {
    const double n = (double)((tiles[v] + 255) / 256);   // tiles of the fullest CU
    double us;
    if (dt == DT_F32) {
      const double fix[3] = {3.5, 3.5, 4.8}, one[3] = {0.0057, 0.010, 0.0164}, more[3] = {0.0075, 0.0125, 0.0245};
      us = fix[v] + n * K * (n > 1 ? more[v] : one[v]);
    } else {
      const double fix[3] = {2.6, 3.0, 4.0}, rate = v == 0 && n > 1 ? 50e3 : 85e3;
      us = fix[v] + n * rows[v] * K * 2 / rate;
    }
    if (us < best_us) best_us = us, best = v;
  }
  if (dt == DT_F32) return gemm_f32_small_applies(M, N) ? best : -1;
  if (!pipe_eligible) return tiles[2] <= 2048 ? best : -1;   // a ragged k: the alternative is the register-staged kernel
  const long t128 = (long)((M + 127) / 128) * ((N + 127) / 128);
  // (GELU and its derivative: every thread of a workgroup walks the epilogue here, half of them there)
  const double pipe_us = 4.6 + (gelu ? 3.0 : 0.0) + (double)((t128 + 255) / 256) * 256 * K * 2 / 69e3;
  return tiles[2] <= 1024 && best_us < pipe_us ? best : -1;
}

// Fewer than one 64 x 128 tile per CU: the tiles of gemm.hip would leave most of the chip idle.
bool gemm_f32_small_applies(int M, int N) { return (long)((M + 63) / 64) * ((N + 127) / 128) < 256; }

hipError_t launch_gemm_small(int dt, const GemmArgs &a, const void *dev, int splits, int variant, hipStream_t s) {
  if (!a.a_kc) return hipErrorInvalidValue;
  const GemmDev &d = *static_cast<const GemmDev *>(dev);
  return dt == DT_F32 ? launch_v<float>(a, d, splits, variant, s) : launch_v<bf16_t>(a, d, splits, variant, s);
}

}  // namespace fl
