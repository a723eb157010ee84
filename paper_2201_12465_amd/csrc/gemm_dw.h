// What the two weight-gradient kernels (gemm_dw.hip, gemm_dw_small.hip) share: the table of a launch, the walk over
// its tiles, and the column sums that ride along.
//
// All parameter gradients of a layer's backward pass that are sums over tokens -- the four dW = dy^T x, the bias
// sums of the linears whose dy no LayerNorm backward has summed, and the second stage of the LayerNorm sums -- wait
// until the pass has produced every dy and then run as ONE launch on the layer's stream.  Launched one by one they
// are short kernels of 36-144 output tiles that either leave CUs idle or have to be cut over the tokens, with fp32
// partial sums to add up afterwards; together their tiles fill the chip once or twice over, mostly without a cut.
// Beside the input-gradient chain on a second stream (where they used to run) they cost the chain as much as they
// gained, and an event record plus wait per operator on the host (195 us of host time per pass).
#pragma once
#include "devutil.h"
#include "gemm_dev.h"
#include "kernels.h"

namespace fl {

struct DwDev {
  struct Job {
    const void *gy, *x;
    void *out;
    float *partial;
    int N, K, tiles_n, tiles_k;   // out[N, K] = sum over tokens of gy[m, n] x[m, k]
  } job[DW_MAX_JOBS];
  ColJob col[DW_MAX_COLS];
  int first[DW_MAX_JOBS + 1];        // first tile of each job
  int first_col[DW_MAX_COLS + 1];    // first strip of each column-sum job, counted from the end of the tiles
  int njobs, ncols, M, splits, m_per_split, accumulate;
};

// Fills the launch's table for BM x BN tiles; returns the number of workgroups.
inline int dw_fill(DwDev &d, const DwJob *jobs, int njobs, const ColJob *cols, int ncols, int M, int splits, int kt, int bm,
                   int bn, bool accumulate) {
  int at = 0;
  for (int j = 0; j < njobs; ++j) {
    d.first[j] = at;
    d.job[j] = {jobs[j].gy, jobs[j].x, jobs[j].out, splits > 1 ? jobs[j].partial : nullptr, jobs[j].N, jobs[j].K,
                (jobs[j].N + bm - 1) / bm, (jobs[j].K + bn - 1) / bn};
    at += d.job[j].tiles_n * d.job[j].tiles_k;
  }
  d.first[njobs] = at;
  int strips = 0;
  for (int j = 0; j < ncols; ++j) {
    d.first_col[j] = strips;
    d.col[j] = cols[j];
    const int w = cols[j].f32 ? 32 : 64;   // columns of a strip: 128 bytes of a row
    strips += (cols[j].n + w - 1) / w;
  }
  d.first_col[ncols] = strips;
  d.njobs = njobs; d.ncols = ncols; d.M = M; d.splits = splits; d.accumulate = accumulate ? 1 : 0;
  d.m_per_split = ((M + splits - 1) / splits + kt - 1) / kt * kt;
  return at * splits + strips;
}

// Tile of workgroup `bid` (< tiles * splits): its job, tile coordinates and token range, as the argument block of the
// shared epilogue.  XCD-contiguous order: token range first, then job, then groups of `gm` row-tiles.
__device__ __forceinline__ void dw_tile(const DwDev &d, int bid, int gm, GemmDev &p, int &tm, int &tn, int &kbeg, int &kend) {
  const int tiles = d.first[d.njobs];
  int id = xcd_tile_order(bid, tiles * d.splits);
  const int split = id / tiles;
  id -= split * tiles;
  int j = 0;
  while (j + 1 < d.njobs && id >= d.first[j + 1]) ++j;
  const DwDev::Job &J = d.job[j];
  id -= d.first[j];
  const int per_group = gm * J.tiles_k, g = id / per_group, r = id - g * per_group;
  const int rows = min(gm, J.tiles_n - g * gm);
  tn = r / rows;
  tm = g * gm + (r - tn * rows);
  kbeg = split * d.m_per_split;
  kend = min(d.M, kbeg + d.m_per_split);
  p.A = J.gy; p.B = J.x; p.C = J.out;
  p.M = J.N; p.N = J.K; p.K = d.M; p.lda = J.N; p.ldb = J.K; p.ldc = J.K;
  p.bias = nullptr; p.aux = nullptr; p.preact = nullptr; p.act = 0; p.dact = 0; p.drop_where = 0;
  p.residual = d.accumulate ? J.out : nullptr;   // in place: each lane reads the elements it then writes
  p.partial = J.partial ? J.partial + (size_t)split * J.N * J.K : nullptr;
}

// out[n] = sum over rows of in[r][n] for one strip of 128 bytes of columns: eight lanes per row, the other threads on
// other rows, one pass through LDS (NTHR * 16 / sizeof(TIN) floats) in a fixed order.
template <typename TIN, typename TOUT, int NTHR>
__device__ __forceinline__ void column_strip(const ColJob &c, int strip, int accumulate, float *red) {
  constexpr int VEC = Elem<TIN>::VEC, COLS = 8 * VEC, RL = NTHR / 8;
  const int t = threadIdx.x, rl = t >> 3, c0 = (t & 7) * VEC, n0 = strip * COLS + c0;
  float a[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) a[e] = 0.f;
  if (n0 < c.n) {
    const TIN *src = static_cast<const TIN *>(c.in) + n0;
#pragma unroll 8
    for (int r = rl; r < c.rows; r += RL) {
      float v[VEC];
      VecIO<TIN, VEC>::load(src + (size_t)r * c.ld, v);
#pragma unroll
      for (int e = 0; e < VEC; ++e) a[e] += v[e];
    }
  }
#pragma unroll
  for (int e = 0; e < VEC; e += 4) *reinterpret_cast<float4 *>(red + rl * COLS + c0 + e) = make_float4(a[e], a[e + 1], a[e + 2], a[e + 3]);
  __syncthreads();
  const int n = strip * COLS + t;
  if (t < COLS && n < c.n) {
    float s[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int r = 0; r < RL; r += 4)
#pragma unroll
      for (int u = 0; u < 4; ++u) s[u] += red[(r + u) * COLS + t];
    float v = (s[0] + s[1]) + (s[2] + s[3]);
    TOUT *out = static_cast<TOUT *>(c.out) + n;
    if (accumulate) v += to_f32(*out);
    *out = from_f32<TOUT>(v);
  }
}
template <typename T, int NTHR> __device__ __forceinline__ void dw_columns(const DwDev &d, int strip, float *red) {
  int j = 0;
  while (j + 1 < d.ncols && strip >= d.first_col[j + 1]) ++j;
  strip -= d.first_col[j];
  if (d.col[j].f32) column_strip<float, T, NTHR>(d.col[j], strip, d.accumulate, red);
  else column_strip<bf16_t, T, NTHR>(d.col[j], strip, d.accumulate, red);
}

}  // namespace fl
