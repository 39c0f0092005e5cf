// Gram matrix of thin rows in FP64 on the matrix cores, one partial per block.
//
// part[p w + q] = sum over the block's rows of x_p x_q (p, q < w <= 16 NB).  A lane of
// v_mfma_f64_16x16x4f64 holds column lane % 16 of row lane / 16 of a group of four, as the
// A and as the B operand alike, so one load per 16 columns feeds the product; the blocks on
// and above the diagonal are formed and mirrored.  Waves take groups of four rows in turn,
// eight groups in flight (four with more blocks); the waves' sums are added in LDS in wave order.
//
// Bound by latency (3 to 6 MB of rows): 76800 x 20 rows for the certificate took 34.3 us with
// one thread per entry and the rows in LDS, 8.2 here; 76800 x 10 for the preconditioner
// 25.7, 5.0 here.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace rpca_rows {

typedef double d4 __attribute__((ext_vector_type(4)));
constexpr int TH = 256;  // threads per block

// The columns come in SIDES sides of `per` columns each, a side in blocks of 16 of its own
// (NB blocks in all); column p of the result is column p % per of side p / per.  load(o, x)
// fills x[i] with the lane's column of block i in the row at offset o = row * stride; what
// it gives past a side's columns or past the rows is masked.
template <int NB, int SIDES, typename Load>
__device__ __forceinline__ void rows_gram(int64_t rows, int stride, int per, Load load, double* part) {
  constexpr int UN = NB <= 2 ? 8 : 4, TRI = NB * (NB + 1) / 2, NBS = NB / SIDES;
  static_assert(NB % SIDES == 0, "whole sides");
  __shared__ double sG[TRI * 256];
  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  d4 acc[TRI];
#pragma unroll
  for (int t = 0; t < TRI; ++t) acc[t] = d4{0., 0., 0., 0.};
  const int64_t step = (int64_t)gridDim.x * (TH / 64) * 4, ostep = step * stride;
  int64_t r0 = ((int64_t)blockIdx.x * (TH / 64) + wave) * 4, o0 = (r0 + lk) * stride;
  for (; r0 < rows; r0 += UN * step, o0 += UN * ostep) {
    double x[UN][NB];
#pragma unroll
    for (int u = 0; u < UN; ++u) load(r0 + u * step + lk < rows ? o0 + u * ostep : 0, x[u]);
#pragma unroll
    for (int u = 0; u < UN; ++u) {
#pragma unroll
      for (int i = 0; i < NB; ++i)
        x[u][i] = r0 + u * step + lk < rows && 16 * (i % NBS) + li < per ? x[u][i] : 0.0;
#pragma unroll
      for (int i = 0, t = 0; i < NB; ++i)
#pragma unroll
        for (int j = i; j < NB; ++j, ++t) acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[u][i], x[u][j], acc[t], 0, 0, 0);
    }
  }
#pragma unroll 1
  for (int q = 0; q < TH / 64; ++q) {
    if (wave == q) {
#pragma unroll
      for (int t = 0; t < TRI; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          double& s = sG[t * 256 + (4 * r + lk) * 16 + li];  // row 4 r + lk, column li
          s = q == 0 ? acc[t][r] : s + acc[t][r];
        }
    }
    __syncthreads();
  }
  const int w = SIDES * per;
  for (int e = threadIdx.x; e < w * w; e += TH) {
    const int p = e / w, c = e % w;
    const int lo = p < c ? p : c, hi = p < c ? c : p;
    const int cl = lo % per, ch = hi % per;
    const int i = lo / per * NBS + (cl >> 4), j = hi / per * NBS + (ch >> 4);  // i <= j
    const int t = i * NB - i * (i - 1) / 2 + (j - i);
    part[e] = sG[t * 256 + (cl & 15) * 16 + (ch & 15)];
  }
}

}  // namespace rpca_rows
