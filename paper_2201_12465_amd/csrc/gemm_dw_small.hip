// All weight gradients of a backward pass in one launch, for problems whose tiles do not fill the chip in the
// pipelined kernel of gemm_dw.hip, and for fp32: tiles as in gemm_small.h (both operands k-major, the contraction runs
// over the tokens), any token count.
#include "gemm_dw.h"
#include "gemm_small.h"

namespace fl {
namespace {

template <typename T, int TM, int TN, int W, int S>
__global__ __launch_bounds__(W * 64) void gemm_dw_small(DwDev d) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const int tiles = d.first[d.njobs] * d.splits;
  if ((int)blockIdx.x >= tiles) {
    dw_columns<T, W * 64>(d, blockIdx.x - tiles, reinterpret_cast<float *>(smem));
    return;
  }
  GemmDev p;
  int tm, tn, kbeg, kend;
  dw_tile(d, blockIdx.x, 1024 / (TM * 32), p, tm, tn, kbeg, kend);
  gemm_small_tile<T, false, false, TM, TN, W, S, false, EPI_PLAIN>(p, tm * TM * 32, tn * TN * 32, kbeg, kend, smem);
}

template <typename T, int TM, int TN, int W, int S>
hipError_t launch(const DwJob *jobs, int njobs, const ColJob *cols, int ncols, int M, int splits, bool accumulate, hipStream_t s) {
  constexpr size_t lds = small_lds_bytes<T, TM, TN, W, S>();
  auto kern = gemm_dw_small<T, TM, TN, W, S>;
  if (lds > 64 * 1024) {
    static bool raised = false;
    if (!raised) {
      hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      if (e != hipSuccess) return e;
      raised = true;
    }
  }
  DwDev d;
  const int grid = dw_fill(d, jobs, njobs, cols, ncols, M, splits, KTile<T>::KT, TM * 32, TN * 32, accumulate);
  hipLaunchKernelGGL(kern, dim3(grid), dim3(W * 64), lds, s, d);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_dw_small(int dt, int tile, const DwJob *jobs, int njobs, const ColJob *cols, int ncols, int M, int splits,
                           bool accumulate, hipStream_t s) {
  if (dt == DT_F32)
    return tile == 32 ? launch<float, 1, 1, 4, 2>(jobs, njobs, cols, ncols, M, splits, accumulate, s)
                      : launch<float, 2, 2, 4, 1>(jobs, njobs, cols, ncols, M, splits, accumulate, s);
  return tile == 32 ? launch<bf16_t, 1, 1, 4, 2>(jobs, njobs, cols, ncols, M, splits, accumulate, s)
                    : launch<bf16_t, 2, 2, 4, 1>(jobs, njobs, cols, ncols, M, splits, accumulate, s);
}

}  // namespace fl
