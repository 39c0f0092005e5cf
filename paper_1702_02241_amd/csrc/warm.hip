// Learned warm start: window statistics, a 2-layer MLP (forward, backward,
// Adam) on FP32 MFMA, and the row pooling / upsampling that maps factors
// between full and low resolution.  The declarations and the definitions of
// every quantity are in rpca_warm.h.
//
// GEMM.  C = op(A) op(B) with op = identity or transpose, row-major storage, one
// 64 x 64 output tile per wave (4 x 4 accumulators of v_mfma_f32_16x16x4f32).  The
// operands go from memory to registers as 16-byte loads and straight into the
// matrix unit, one block of 16 K values ahead of the products: no LDS staging and
// no barrier in the K loop.  When the output has few tiles K is split over the
// waves of a workgroup (summed through LDS) and over workgroups (partials summed
// by a second kernel), or, with K in order, the tile's rows over the waves; always in a
// fixed order, so every result is bitwise
// reproducible.  The epilogue adds a bias, applies ReLU or gates by a previous
// activation (the ReLU derivative in the backward pass).  Products of at most four rows
// (one window's prediction) take a matrix-vector kernel instead, but for the first layer of a
// training step.

#include <hip/hip_runtime.h>
#include <math.h>
#include <string.h>

#include <algorithm>
#include <type_traits>
#include <vector>

#include "rpca.h"
#include "rpca_warm.h"

namespace {

typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int GT = 256;
constexpr int BM = 64, BN = 64, BK = 16;
constexpr int KMAX_LOSS = 32;

// 16-byte accesses at any 4-byte aligned address (rows of odd length)
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
typedef double d4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f4 mfma_f32(float a, float b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

struct GemmArgs {
  const float* A;
  const float* B;
  float* C;
  int64_t M, N, K;
  int64_t lda, ldb, ldc;
  int64_t kchunk;       // K range per wave of a split (multiple of BK)
  const float* bias;    // N values or null
  const float* gate;    // M x N (leading dimension ldg) or null: C = acc * (gate > 0)
  int64_t ldg;
  int32_t relu;
  float* part;          // [splits][M][N] partial products, or null (direct epilogue)
};

__device__ __forceinline__ float epilogue(const GemmArgs& a, int64_t i, int64_t j, float v) {
  if (a.bias) v += a.bias[j];
  if (a.relu) v = fmaxf(v, 0.f);
  if (a.gate && !(a.gate[i * a.ldg + j] > 0.f)) v = 0.f;
  return v;
}

// One operand's 16 values of a K block: o[t][q] is element (16-wide tile t, K = k0 + 4 lk + q)
// of this lane.  K order and the order of a tile's rows are free as long as both
// operands and the output agree, so every load is 16 contiguous bytes:
//   KMAJ (element (x, k) at p[k ld + x]): row k, x = x0 + 4 li + t -- tile t holds x0 + 4 i + t
//   else (p[x ld + k]): row x = x0 + 16 t + li, four K values -- tile t holds x0 + 16 t + i
// Elements past X or kend read as zero.  SEQ: K = k0 + 4 q + lk instead, so that the products
// run through K in order (the rows of a non-KMAJ operand then take four loads of 4 bytes).
template <bool KMAJ, bool SEQ>
__device__ __forceinline__ void load_operand(const float* __restrict__ p, int64_t ld, int64_t x0, int64_t X, int64_t k0,
                                             int64_t kend, int li, int lk, float (&o)[4][4]) {
  auto kof = [&](int q) -> int64_t { return k0 + (SEQ ? 4 * q + lk : 4 * lk + q); };
  if (KMAJ) {
    if (x0 + 64 <= X && k0 + BK <= kend) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f4 v = *reinterpret_cast<const f4u*>(p + kof(q) * ld + x0 + 4 * li);
#pragma unroll
        for (int t = 0; t < 4; ++t) o[t][q] = v[t];
      }
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int64_t k = kof(q), x = x0 + 4 * li + t;
          o[t][q] = (k < kend && x < X) ? p[k * ld + x] : 0.f;
        }
    }
  } else {
    if (x0 + 64 <= X && k0 + BK <= kend) {
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const float* row = p + (x0 + 16 * t + li) * ld;
        const f4 v = SEQ ? f4{row[kof(0)], row[kof(1)], row[kof(2)], row[kof(3)]}
                         : f4(*reinterpret_cast<const f4u*>(row + k0 + 4 * lk));
#pragma unroll
        for (int q = 0; q < 4; ++q) o[t][q] = v[q];
      }
    } else {
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int64_t k = kof(q), x = x0 + 16 * t + li;
          o[t][q] = (k < kend && x < X) ? p[x * ld + k] : 0.f;
        }
    }
  }
}

// The same of one 16-wide tile t, with no branch per element: past X or kend the last element
// is loaded and replaced by zero.
template <bool KMAJ, bool SEQ>
__device__ __forceinline__ void load_tile_operand(const float* __restrict__ p, int64_t ld, int64_t x0, int64_t X, int64_t k0,
                                                  int64_t kend, int li, int lk, int t, float (&o)[4]) {
  auto kof = [&](int q) -> int64_t { return k0 + (SEQ ? 4 * q + lk : 4 * lk + q); };
  const int64_t x = x0 + (KMAJ ? 4 * li + t : 16 * t + li), xc = x < X ? x : X - 1;
  if (!KMAJ && !SEQ && k0 + BK <= kend) {
    const f4 v = *reinterpret_cast<const f4u*>(p + xc * ld + k0 + 4 * lk);
#pragma unroll
    for (int q = 0; q < 4; ++q) o[q] = v[q];
  } else {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t k = kof(q) < kend ? kof(q) : kend - 1;
      o[q] = KMAJ ? p[k * ld + xc] : p[xc * ld + k];
    }
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) o[q] = x < X && kof(q) < kend ? o[q] : 0.f;
}

// FP32 MFMA-bound (64 products of 32 cycles per 16 loads of a lane): 64 x 64 a wave makes
// each 16-byte load feed 16 products.  At 64 rows of the 9700-512-49000 network: y = h W2
// 91 -> 59 us, dz = dy W2^T 158 -> 70 us, dW2 = h^T dy 70 -> 53 us against a 64 x 64
// workgroup tile staged through LDS with two barriers per 16 K values; the products alone
// are 20 us each at the matrix unit's rate.
//
// op(A) is KMAJ when TA, op(B) when !TB.  WK = 4: the workgroup's waves split the K range
// of one tile and meet in LDS; WK = 1 (K of a few blocks): each wave has its own tile;
// WK = 0: each wave takes a K range of its own through K in order and writes it as a partial
// (or the result, if there is one range), so an entry's rounding depends on the ranges alone.
// ROWS (WK = 0, 1; products whose tiles and ranges leave most of the chip idle): a workgroup per
// tile (and range), a 16-row tile of it per wave, with the same sums: a quarter of the products
// per block of K, and none for rows past M.  300-16-360 at 64 rows, forward: 15.8 us for 32.0,
// 620-128-2240 at 17: 16.4 for 33.8 (18.0 and 21.9 with 64 x 64 workgroup tiles in LDS).
template <bool TA, bool TB, int WK, bool ROWS>
__global__ __launch_bounds__(GT) void k_gemm(GemmArgs a) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lk = lane >> 4;
  static_assert(!ROWS || WK != 4, "the waves share a tile in one way");
  constexpr int MI = ROWS ? 1 : 4;  // row tiles of a wave
  constexpr bool NW = WK == 1 && !ROWS;  // the waves take tiles of their own
  const int64_t m0 = (int64_t)blockIdx.y * BM, n0 = ((int64_t)blockIdx.x * (NW ? 4 : 1) + (NW ? w : 0)) * BN;
  const int64_t z = WK == 0 && !ROWS ? (int64_t)blockIdx.z * 4 + w : blockIdx.z;  // partial
  const int64_t kbeg = (WK == 4 ? z * 4 + w : z) * a.kchunk;
  int64_t kend = kbeg + a.kchunk;
  if (kend > a.K) kend = a.K;
  if (NW && n0 >= a.N) return;
  if (WK == 0 && kbeg >= a.K) return;
  if (ROWS && m0 + (TA ? w : 16 * w) >= a.M) return;  // no row of this wave's tile
  f4 acc[MI][4];
  auto load_a = [&](int64_t k0, float (&o)[MI][4]) {
    if constexpr (ROWS) load_tile_operand<TA, WK == 0>(a.A, a.lda, m0, a.M, k0, kend, li, lk, w, o[0]);
    else load_operand<TA, WK == 0>(a.A, a.lda, m0, a.M, k0, kend, li, lk, o);
  };
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};

  if (kbeg < kend) {
    float av[MI][4], bv[4][4];
    load_a(kbeg, av);
    load_operand<!TB, WK == 0>(a.B, a.ldb, n0, a.N, kbeg, kend, li, lk, bv);
    for (int64_t k0 = kbeg; k0 < kend; k0 += BK) {
      float an[MI][4], bn[4][4];
      const bool more = k0 + BK < kend;
      if (more) {
        load_a(k0 + BK, an);
        load_operand<!TB, WK == 0>(a.B, a.ldb, n0, a.N, k0 + BK, kend, li, lk, bn);
      }
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j) acc[i][j] = mfma_f32(av[i][q], bv[j][q], acc[i][j]);
      if (more) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            if (i < MI) av[i < MI ? i : 0][q] = an[i < MI ? i : 0][q];
            bv[i][q] = bn[i][q];
          }
      }
    }
  }
  // lane holds rows 4 lk + r, column li of each 16 x 16 tile (i, j)
  auto row = [&](int i, int r) -> int64_t { return m0 + (TA ? 4 * (4 * lk + r) + i : 16 * i + 4 * lk + r); };
  auto put = [&](int i, int r, const f4& v) {  // v[j]: the four N tiles
    const int64_t gm = row(i, r);
    if (gm >= a.M) return;
    float* dst = a.part ? a.part + z * a.M * a.N + gm * a.N : a.C + gm * a.ldc;
    const int64_t gn = n0 + (TB ? li : 4 * li);
    if (!TB && gn + 4 <= a.N) {
      f4 o = v;
      if (!a.part)
#pragma unroll
        for (int j = 0; j < 4; ++j) o[j] = epilogue(a, gm, gn + j, v[j]);
      *reinterpret_cast<f4u*>(dst + gn) = o;
      return;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int64_t g = gn + (TB ? 16 * j : j);
      if (g < a.N) dst[g] = a.part ? v[j] : epilogue(a, gm, g, v[j]);
    }
  };
  if constexpr (WK != 4) {
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) put(ROWS ? w : i, r, f4{acc[i][0][r], acc[i][1][r], acc[i][2][r], acc[i][3][r]});
  } else {
    // wave w finishes the row tile i = w: the others' accumulators of it through LDS,
    // added in wave order
    __shared__ f4 sP[4][4][4][64];  // [row tile][wave][j][lane]
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) sP[i][w][j][lane] = acc[i][j];
    __syncthreads();
    f4 s[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) s[j] = ((sP[w][0][j][lane] + sP[w][1][j][lane]) + sP[w][2][j][lane]) + sP[w][3][j][lane];
#pragma unroll
    for (int r = 0; r < 4; ++r) put(w, r, f4{s[0][r], s[1][r], s[2][r], s[3][r]});
  }
}

__global__ __launch_bounds__(GT) void k_splitk_reduce(GemmArgs a, int splits) {
  const int64_t mn = a.M * a.N;
  for (int64_t o = (int64_t)blockIdx.x * GT + threadIdx.x; o < mn; o += (int64_t)gridDim.x * GT) {
    float s = 0.f;
    int z = 0;
    for (; z + 7 < splits; z += 8) {  // eight loads in flight, added in order
      float x[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = a.part[(int64_t)(z + e) * mn + o];
#pragma unroll
      for (int e = 0; e < 8; ++e) s += x[e];
    }
    for (; z < splits; ++z) s += a.part[(int64_t)z * mn + o];
    const int64_t i = o / a.N, j = o % a.N;
    a.C[i * a.ldc + j] = epilogue(a, i, j, s);
  }
}

// C = A B for at most MV rows of A (row-major, B K-major: the forward pass of one or a few
// windows).  Memory-bound on B (100 MB of W2 in 21.6 us, 4.6 TB/s; the 64-row tile took
// 68 us, padding one row to 64): a workgroup of 32 lane columns (VEC values each) x 32 K
// groups streams its K range once, the groups' sums meet in LDS in group order.
constexpr int MV = 4, MV_T = 1024, MV_L = 32, MV_G = MV_T / MV_L, MV_K = 512;
template <int VEC>
__global__ __launch_bounds__(MV_T) void k_gemv(GemmArgs a) {
  __shared__ float sx[MV][MV_K];
  __shared__ float sp[MV_G][MV_L * VEC];
  const int tid = threadIdx.x, c = tid & (MV_L - 1), gk = tid / MV_L;
  const int M = (int)a.M;
  const int64_t n = ((int64_t)blockIdx.x * MV_L + c) * VEC;
  const int64_t kbeg = (int64_t)blockIdx.z * a.kchunk;
  const int64_t kend = kbeg + a.kchunk < a.K ? kbeg + a.kchunk : a.K;
  float acc[MV][VEC] = {};
  for (int64_t k0 = kbeg; k0 < kend; k0 += MV_K) {
    const int nk = (int)(kend - k0 < MV_K ? kend - k0 : MV_K);
    __syncthreads();
    for (int e = tid; e < M * MV_K; e += MV_T) {
      const int b = e / MV_K, kk = e % MV_K;
      if (kk < nk) sx[b][kk] = a.A[b * a.lda + k0 + kk];
    }
    __syncthreads();
    if (n < a.N) {
#pragma unroll 8
      for (int kk = gk; kk < nk; kk += MV_G) {
        const float* src = a.B + (k0 + kk) * a.ldb + n;
        float v[VEC];
        if (VEC == 4) {
          const f4 x = *reinterpret_cast<const f4*>(src);
#pragma unroll
          for (int e = 0; e < VEC; ++e) v[e] = x[e & 3];
        } else {
          v[0] = src[0];
        }
#pragma unroll
        for (int b = 0; b < MV; ++b)
          if (b < M)
#pragma unroll
            for (int e = 0; e < VEC; ++e) acc[b][e] = fmaf(sx[b][kk], v[e], acc[b][e]);
      }
    }
  }
#pragma unroll
  for (int b = 0; b < MV; ++b) {
    if (b >= M) break;
    __syncthreads();
#pragma unroll
    for (int e = 0; e < VEC; ++e) sp[gk][c * VEC + e] = acc[b][e];
    __syncthreads();
    const int64_t j = (int64_t)blockIdx.x * MV_L * VEC + tid;
    if (tid < MV_L * VEC && j < a.N) {
      float s = 0.f;
#pragma unroll
      for (int q = 0; q < MV_G; ++q) s += sp[q][tid];
      if (a.part)
        a.part[(int64_t)blockIdx.z * a.M * a.N + b * a.N + j] = s;
      else
        a.C[b * a.ldc + j] = epilogue(a, b, j, s);
    }
  }
}

// out[j] = sum over rows of A (rows x cols, row-major), added in row order; two
// matrices in one launch (blockIdx.y)
struct ColsumArgs {
  const float* A[2];
  int64_t rows, cols[2];
  float* out[2];
};
__global__ __launch_bounds__(GT) void k_colsum(ColsumArgs a) {
  const int y = blockIdx.y;
  const float* __restrict__ A = a.A[y];
  const int64_t cols = a.cols[y], rows = a.rows;
  const int64_t j = (int64_t)blockIdx.x * GT + threadIdx.x;
  if (j >= cols) return;
  float s = 0.f;
  int64_t r = 0;
  for (; r + 15 < rows; r += 16) {  // sixteen loads in flight
    float x[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) x[e] = A[(r + e) * cols + j];
#pragma unroll
    for (int e = 0; e < 16; ++e) s += x[e];
  }
  for (; r < rows; ++r) s += A[r * cols + j];
  a.out[y][j] = s;
}

// ---------------------------------------------------------------------------
// Loss on the factored target.  For batch element b with prediction (Uh, Vh)
// and target factors (TU, TV):
//   Guu = Uh^T Uh, Mtu = TU^T Uh, Gtu = TU^T TU  (k x k, over the mu rows)
//   Gvv = Vh^T Vh, Mtv = TV^T Vh, Gtv = TV^T TV  (k x k, over the nv rows)
//   ||Uh Vh^T - TU TV^T||^2 = <Guu, Gvv> - 2 <Mtu, Mtv> + <Gtu, Gtv>
//   d/dUh = 2 (Uh Gvv - TU Mtv),   d/dVh = 2 (Vh Guu - TV Mtu).
// All of it in FP64 on v_mfma_f64_16x16x4f64 (KB = 1: k <= 16, 2: k <= 32).  One FP64
// lane layout serves both kernels: A and B operands hold row / column li at K = lk, the
// output holds rows 4 r + lk, column li.
//
// k_loss_grams: a workgroup takes one row chunk of one batch element, its waves
// interleaved groups of four rows, four of them in flight (64 windows of 4900 rows: 19 us; one workgroup per
// window with one thread per entry took 367 us); the waves' sums meet in LDS in wave order and the
// chunk's three matrices go to gpart[b][chunk][3][k][k].  Chunks [0, cu) cover the
// mu rows of U, [cu, cu + cv) the nv rows of V.
struct LossArgs {
  const float* y;
  const float* TU;
  const float* TV;
  int mu, nv, k, batch;
  int per, cu, cv;  // rows per chunk, chunks of each side
  int64_t d_out;
  double* gpart;
  double* grams;  // [batch][6][k][k]
  double* lossb;  // [batch]
  double* loss;
  float* dy;
};

__device__ __forceinline__ d4 mfma_f64(double a, double b, d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

template <int KB>
__global__ __launch_bounds__(GT) void k_loss_grams(LossArgs a) {
  constexpr int NTL = 3 * KB * KB;
  __shared__ double sG[GT / 64][NTL * 256];
  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int b = blockIdx.y, ch = blockIdx.x, k = a.k;
  const bool us = ch < a.cu;
  const int rows = us ? a.mu : a.nv, r0 = (us ? ch : ch - a.cu) * a.per;
  const int r1 = r0 + a.per < rows ? r0 + a.per : rows;
  const float* P = a.y + (int64_t)b * a.d_out + (us ? 0 : (int64_t)a.mu * k);
  const float* T = us ? a.TU + (int64_t)b * a.mu * k : a.TV + (int64_t)b * a.nv * k;
  d4 acc[3][KB][KB];
#pragma unroll
  for (int m = 0; m < 3; ++m)
#pragma unroll
    for (int i = 0; i < KB; ++i)
#pragma unroll
      for (int j = 0; j < KB; ++j) acc[m][i][j] = d4{0., 0., 0., 0.};
  constexpr int UN = 4;  // groups of rows whose loads are in flight together
  for (int rb = r0 + 4 * w; rb < r1; rb += 16 * UN) {
    float pv[UN][KB], tv[UN][KB];
#pragma unroll
    for (int u = 0; u < UN; ++u)
#pragma unroll
      for (int i = 0; i < KB; ++i) {
        const int r = rb + 16 * u + lk, c = 16 * i + li;
        const bool ok = r < r1 && c < k;
        const int64_t o = ok ? (int64_t)r * k + c : 0;
        pv[u][i] = P[o];
        tv[u][i] = T[o];
        pv[u][i] = ok ? pv[u][i] : 0.f;
        tv[u][i] = ok ? tv[u][i] : 0.f;
      }
#pragma unroll
    for (int u = 0; u < UN; ++u)
#pragma unroll
      for (int i = 0; i < KB; ++i)
#pragma unroll
        for (int j = 0; j < KB; ++j) {
          const double p = pv[u][i], t = tv[u][i], q = pv[u][j], v = tv[u][j];
          acc[0][i][j] = mfma_f64(p, q, acc[0][i][j]);
          acc[1][i][j] = mfma_f64(t, q, acc[1][i][j]);
          acc[2][i][j] = mfma_f64(t, v, acc[2][i][j]);
        }
  }
#pragma unroll
  for (int m = 0; m < 3; ++m)
#pragma unroll
    for (int i = 0; i < KB; ++i)
#pragma unroll
      for (int j = 0; j < KB; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) sG[w][((m * KB + i) * KB + j) * 256 + (4 * r + lk) * 16 + li] = acc[m][i][j][r];
  __syncthreads();
  const int kk2 = k * k;
  double* out = a.gpart + ((int64_t)b * (a.cu + a.cv) + ch) * 3 * kk2;
  for (int e = threadIdx.x; e < 3 * kk2; e += GT) {
    const int m = e / kk2, p = (e % kk2) / k, q = e % k;
    const int o = ((m * KB + (p >> 4)) * KB + (q >> 4)) * 256 + (p & 15) * 16 + (q & 15);
    double s = 0.0;
#pragma unroll
    for (int ww = 0; ww < GT / 64; ++ww) s += sG[ww][o];
    out[e] = s;
  }
}

// grams[b] = the chunks' sums in chunk order, and b's share of the loss
__global__ __launch_bounds__(GT) void k_loss_finish(LossArgs a) {
  __shared__ double sh[GT / 64];
  const int b = blockIdx.x, kk2 = a.k * a.k;
  double acc = 0.0;
  for (int e = threadIdx.x; e < kk2; e += GT) {
    double g[6] = {0., 0., 0., 0., 0., 0.};
    const double* src = a.gpart + (int64_t)b * (a.cu + a.cv) * 3 * kk2 + e;
    for (int ch = 0; ch < a.cu; ++ch, src += 3 * kk2)
#pragma unroll
      for (int m = 0; m < 3; ++m) g[m] += src[m * kk2];
    for (int ch = 0; ch < a.cv; ++ch, src += 3 * kk2)
#pragma unroll
      for (int m = 0; m < 3; ++m) g[3 + m] += src[m * kk2];
#pragma unroll
    for (int m = 0; m < 6; ++m) a.grams[((int64_t)b * 6 + m) * kk2 + e] = g[m];
    acc += g[0] * g[3] - 2.0 * g[1] * g[4] + g[2] * g[5];
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) acc += __shfl_xor(acc, o, 64);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int w = 0; w < GT / 64; ++w) s += sh[w];
    a.lossb[b] = s;
  }
}

// dy rows of one batch element, 16 rows a wave at a time: (2 / B) (P G - T M) with G, M in
// registers (15 us for 64 windows; 55 us with one thread per entry reading G from memory); the first block also forms loss = (1/B) sum_b in a fixed order.  Rows
// [0, mu) are U's (G = Gvv, M = Mtv), the rest V's (Guu, Mtu).
template <int KB>
__global__ __launch_bounds__(GT) void k_loss_dy(LossArgs a) {
  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int b = blockIdx.y, k = a.k, kk2 = k * k;
  if (blockIdx.x == 0 && b == 0 && w == 0) {
    double s = 0.0;
    for (int q = lane; q < a.batch; q += 64) s += a.lossb[q];
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o, 64);
    if (lane == 0) *a.loss = s / a.batch;
  }
  const int ub = (a.mu + 15) >> 4, nb = ub + ((a.nv + 15) >> 4);  // 16-row blocks of each side
  const int stride = gridDim.x * (GT / 64);
  const double sc = 2.0 / a.batch;
  const double* g = a.grams + (int64_t)b * 6 * kk2;
  double G[4 * KB][KB], Mt[4 * KB][KB];  // B operands: K = 4 s + lk, column 16 j + li
  int side = -1;
  for (int blk = blockIdx.x * (GT / 64) + w; blk < nb; blk += stride) {
    const bool us = blk < ub;
    if ((int)us != side) {
      side = us;
      const double* Gp = g + (us ? 3 : 0) * kk2;
      const double* Mp = g + (us ? 4 : 1) * kk2;
#pragma unroll
      for (int s = 0; s < 4 * KB; ++s)
#pragma unroll
        for (int j = 0; j < KB; ++j) {
          const int kr = 4 * s + lk, c = 16 * j + li;
          const bool ok = kr < k && c < k;
          G[s][j] = ok ? Gp[kr * k + c] : 0.0;
          Mt[s][j] = ok ? -Mp[kr * k + c] : 0.0;
        }
    }
    const int rows = us ? a.mu : a.nv, r0 = 16 * (us ? blk : blk - ub);
    const int64_t off = (int64_t)b * a.d_out + (us ? 0 : (int64_t)a.mu * k);
    const float* T = us ? a.TU + (int64_t)b * a.mu * k : a.TV + (int64_t)b * a.nv * k;
    const bool rok = r0 + li < rows;
    const int64_t ro = (int64_t)(rok ? r0 + li : rows - 1) * k;
    d4 acc[KB];
#pragma unroll
    for (int j = 0; j < KB; ++j) acc[j] = d4{0., 0., 0., 0.};
#pragma unroll
    for (int s = 0; s < 4 * KB; ++s) {
      if (4 * s >= k) break;
      const int kr = 4 * s + lk;
      const bool ok = kr < k;
      const double p = ok ? (double)a.y[off + ro + kr] : 0.0, t = ok ? (double)T[ro + kr] : 0.0;
#pragma unroll
      for (int j = 0; j < KB; ++j) {
        acc[j] = mfma_f64(p, G[s][j], acc[j]);
        acc[j] = mfma_f64(t, Mt[s][j], acc[j]);
      }
    }
#pragma unroll
    for (int j = 0; j < KB; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = r0 + 4 * r + lk, c = 16 * j + li;
        if (i < rows && c < k) a.dy[off + (int64_t)i * k + c] = (float)(sc * acc[j][r]);
      }
  }
}

// Adam on all four tensors in one launch (blockIdx.y): 28 bytes a parameter, HBM-bound
struct AdamArgs {
  float* p[4];
  const float* g[4];
  float* m1[4];
  float* m2[4];
  int64_t n[4];
  float lr, b1, b2, eps, bc1, bc2;
};
__global__ __launch_bounds__(GT) void k_adam(AdamArgs a) {
  const int y = blockIdx.y;
  float* __restrict__ p = a.p[y];
  const float* __restrict__ g = a.g[y];
  float* __restrict__ m1 = a.m1[y];
  float* __restrict__ m2 = a.m2[y];
  const int64_t n = a.n[y], n4 = n >> 2;
  auto one = [&](float gi, float& m, float& v, float& pi) {
    m = fmaf(a.b1, m, (1.f - a.b1) * gi);
    v = fmaf(a.b2, v, (1.f - a.b2) * gi * gi);
    const float mh = m / a.bc1, vh = v / a.bc2;
    pi -= a.lr * mh / (sqrtf(vh) + a.eps);
  };
  const int64_t t0 = (int64_t)blockIdx.x * GT + threadIdx.x, stride = (int64_t)gridDim.x * GT;
  for (int64_t i = t0; i < n4; i += stride) {
    const f4 gi = reinterpret_cast<const f4*>(g)[i];
    f4 m = reinterpret_cast<f4*>(m1)[i], v = reinterpret_cast<f4*>(m2)[i], q = reinterpret_cast<f4*>(p)[i];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float me = m[e], ve = v[e], qe = q[e];
      one(gi[e], me, ve, qe);
      m[e] = me;
      v[e] = ve;
      q[e] = qe;
    }
    reinterpret_cast<f4*>(m1)[i] = m;
    reinterpret_cast<f4*>(m2)[i] = v;
    reinterpret_cast<f4*>(p)[i] = q;
  }
  for (int64_t i = 4 * n4 + t0; i < n; i += stride) one(g[i], m1[i], m2[i], p[i]);
}

// ---------------------------------------------------------------------------
// Window statistics, one launch.  The first `nblk` workgroups take FB pooled blocks each:
// lane column = pooled block, FG frame groups take every FG-th frame, and the groups'
// FP64 sums of the pooled value and its square meet in LDS in group order (mean and
// population standard deviation).  The other workgroups take one frame's mean each.
// Bound by reading X twice, once from HBM: 10.8 us for 76,800 x 100 (30.7 MB); one thread
// per pooled block and one 256-thread workgroup per frame took 210 + 76 us.
// VEC: 4 x 4 pooling read as 16-byte rows (16-byte aligned X), else element loads.
constexpr int FT = 1024, FB = 32, FG = FT / FB;
template <bool VEC>
__global__ __launch_bounds__(FT) void k_features(const float* __restrict__ X, int64_t W, int64_t H, int frames, int f,
                                                 int64_t nblk, const float* shift, const float* scale, float* feat) {
  __shared__ double sh[2][FG][FB];
  const int64_t wl = W / f, mu = wl * (H / f), m = W * H;
  const int tid = threadIdx.x;
  if (blockIdx.x < nblk) {
    const int c = tid % FB, tg = tid / FB;
    const int64_t p = (int64_t)blockIdx.x * FB + c;
    double s1 = 0.0, s2 = 0.0;
    if (p < mu) {
      const float* base = X + (p / wl * f) * W + p % wl * f;
      const double inv = 1.0 / ((double)f * f);
#pragma unroll 2
      for (int t = tg; t < frames; t += FG) {
        const float* col = base + (int64_t)t * m;
        double v = 0.0;
        if (VEC) {
          f4 x[4];
#pragma unroll
          for (int dy = 0; dy < 4; ++dy) x[dy] = *reinterpret_cast<const f4*>(col + dy * W);
#pragma unroll
          for (int dy = 0; dy < 4; ++dy)
#pragma unroll
            for (int dx = 0; dx < 4; ++dx) v += (double)x[dy][dx];
        } else {
          for (int dy = 0; dy < f; ++dy)
            for (int dx = 0; dx < f; ++dx) v += (double)col[dy * W + dx];
        }
        v *= inv;
        s1 += v;
        s2 += v * v;
      }
    }
    sh[0][tg][c] = s1;
    sh[1][tg][c] = s2;
    __syncthreads();
    if (tid < FB && p < mu) {
      s1 = 0.0;
      s2 = 0.0;
      for (int q = 0; q < FG; ++q) {
        s1 += sh[0][q][c];
        s2 += sh[1][q][c];
      }
      const double mean = s1 / frames;
      double var = s2 / frames - mean * mean;
      if (var < 0.0) var = 0.0;
      float a = (float)mean, b = (float)sqrt(var);
      if (shift) {
        a = (a - shift[p]) * scale[p];
        b = (b - shift[mu + p]) * scale[mu + p];
      }
      feat[p] = a;
      feat[mu + p] = b;
    }
    return;
  }
  const int64_t t = blockIdx.x - nblk;
  const float* col = X + t * m;
  double s = 0.0;
  int64_t i0 = 0;
  if (VEC) {  // m is a multiple of 16
    const f4* c4 = reinterpret_cast<const f4*>(col);
#pragma unroll 4
    for (int64_t i = tid; i < m >> 2; i += FT) {
      const f4 x = c4[i];
      s += ((double)x[0] + (double)x[1]) + ((double)x[2] + (double)x[3]);
    }
    i0 = m;
  }
  for (int64_t i = i0 + tid; i < m; i += FT) s += (double)col[i];
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o, 64);
  double* sw = &sh[0][0][0];
  if ((tid & 63) == 0) sw[tid >> 6] = s;
  __syncthreads();
  if (tid == 0) {
    double r = 0.0;
    for (int w = 0; w < FT / 64; ++w) r += sw[w];
    float v = (float)(r / m);
    if (shift) v = (v - shift[2 * mu + t]) * scale[2 * mu + t];
    feat[2 * mu + t] = v;
  }
}

__global__ __launch_bounds__(GT) void k_pool_rows(const float* A, int64_t W, int64_t H, int f, int c,
                                                  float* out) {
  const int64_t wl = W / f, mu = wl * (H / f);
  const int64_t e = (int64_t)blockIdx.x * GT + threadIdx.x;
  if (e >= mu * c) return;
  const int64_t p = e / c;
  const int cc = (int)(e % c);
  const int64_t by = p / wl, bx = p % wl;
  double s = 0.0;
  for (int dy = 0; dy < f; ++dy)
    for (int dx = 0; dx < f; ++dx) s += (double)A[((by * f + dy) * W + bx * f + dx) * c + cc];
  out[e] = (float)(s / ((double)f * f));
}

__global__ __launch_bounds__(GT) void k_upsample_rows(const float* A, int64_t W, int64_t H, int f, int c,
                                                      float* out) {
  const int64_t wl = W / f;
  const int64_t e = (int64_t)blockIdx.x * GT + threadIdx.x;
  if (e >= W * H * c) return;
  const int64_t i = e / c;
  const int cc = (int)(e % c);
  const int64_t y = i / W, x = i % W;
  out[e] = A[((y / f) * wl + x / f) * c + cc];
}

inline int grid_for(int64_t n, int cap = 4096) {
  int64_t g = (n + GT - 1) / GT;
  if (g < 1) g = 1;
  return (int)(g < cap ? g : cap);
}

uint64_t mix64(uint64_t x) {
  x += 0x9E3779B97F4A7C15ull;
  x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
  x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
  return x ^ (x >> 31);
}

// Standard normal deviate number idx of stream `seed` (SplitMix64 + Box-Muller).
double gauss(uint64_t seed, uint64_t idx) {
  const uint64_t a = mix64(seed ^ mix64(2 * idx)), b = mix64(seed ^ mix64(2 * idx + 1));
  const double u1 = ((a >> 11) + 0.5) * (1.0 / 9007199254740992.0);
  const double u2 = ((b >> 11) + 0.5) * (1.0 / 9007199254740992.0);
  return sqrt(-2.0 * log(u1)) * cos(6.283185307179586 * u2);
}

}  // namespace

struct rpca_mlp {
  int d_in, d_h, mu, nv, k, max_batch;
  int64_t d_out;
  float* param[4];
  float* grad[4];
  float* mom1[4];
  float* mom2[4];
  int64_t count[4];
  float* h;       // max_batch x d_h: relu(x W1 + b1)
  float* y;       // max_batch x d_out
  float* dy;      // max_batch x d_out
  float* dz;      // max_batch x d_h
  float* part;    // split-K partials
  int64_t part_cap;
  double* grams;  // max_batch x 6 x k x k
  double* gpart;  // row chunks' Gram matrices (loss_chunks)
  double* lossb;  // max_batch
  int step;
};

namespace {

// Products of fewer tiles (times ranges) than this take a wave per 16 rows (k_gemm's ROWS): with
// a wave per tile some of the chip's 1,024 SIMDs would have none.  Forward, us, with the
// line at 0 / 256 / 512 / 1024: 2000-100-29856 at 33 rows 42.4 / 33.5 / 24.5 / 24.6, 9700-512-49000 at
// 128 rows 129.7 / 129.4 / 129.3 / 113.7.
constexpr int64_t ROWS_BELOW = 1024;

// The first layer's product of a training step, and of more than MV rows, through K in ranges and in an order that
// depend on the sizes alone and stay as they are: a hidden unit's gate in the backward pass
// is the sign of this sum, so another order of the same additions now and then turns a unit
// whose input is zero to rounding on or off (one in 32,768 moved grad W1 by 2e-3 relative).
// A prediction of at most MV rows has no gates to keep and streams W1 once (k_gemv).
hipError_t gemm_in_order(rpca_mlp* net, GemmArgs g, hipStream_t s) {
  const int64_t tm = (g.M + BM - 1) / BM, tn = (g.N + BN - 1) / BN, tiles = tm * tn;
  const int64_t kslices = (g.K + BK - 1) / BK;
  int64_t splits = 1;
  if (tiles < 512 && kslices >= 8) {
    splits = std::min((512 + tiles - 1) / tiles, kslices / 4);
    splits = std::max<int64_t>(1, std::min(splits, net->part_cap / (g.M * g.N)));
  }
  g.kchunk = (kslices + splits - 1) / splits * BK;
  splits = (g.K + g.kchunk - 1) / g.kchunk;
  g.part = splits > 1 ? net->part : nullptr;
  if (tm > 65535 || splits > 65535) return hipErrorInvalidValue;
  if (tiles * splits < ROWS_BELOW)
    hipLaunchKernelGGL((k_gemm<false, false, 0, true>), dim3((unsigned)tn, (unsigned)tm, (unsigned)splits), dim3(GT), 0, s, g);
  else
    hipLaunchKernelGGL((k_gemm<false, false, 0, false>), dim3((unsigned)tn, (unsigned)tm, (unsigned)((splits + 3) / 4)),
                       dim3(GT), 0, s, g);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || splits == 1) return e;
  hipLaunchKernelGGL(k_splitk_reduce, dim3(grid_for(g.M * g.N)), dim3(GT), 0, s, g, (int)splits);
  return hipGetLastError();
}

// Launch C = op(A) op(B) with the epilogue in `e` (A, B, C, sizes filled by the caller).
hipError_t gemm(rpca_mlp* net, GemmArgs g, bool ta, bool tb, hipStream_t s) {
  const int64_t cap = net->part_cap / (g.M * g.N);
  if (!ta && !tb && g.M <= MV && (g.K >= MV_G || g.M == 1)) {
    // matrix-vector (at most four rows: the predictions of single windows; the tile kernel
    // pads them to 64 rows and takes 3x as long; several rows with fewer values than the K
    // groups leave groups idle, 64-8-130048 at 4 rows 18.3 us for 13.9 on tiles): 128 (or 32) columns a workgroup, K split until some 512 workgroups are
    // in flight, at least four values a K group
    const bool vec = g.N % 4 == 0 && g.ldb % 4 == 0 && ((uintptr_t)g.B & 15) == 0;
    const int64_t tn = (g.N + MV_L * (vec ? 4 : 1) - 1) / (MV_L * (vec ? 4 : 1));
    int64_t splits = (512 + tn - 1) / tn;
    if (splits > g.K / (4 * MV_G)) splits = g.K / (4 * MV_G);
    if (splits > cap) splits = cap;
    if (splits < 1) splits = 1;
    g.kchunk = (g.K + splits - 1) / splits;
    splits = (g.K + g.kchunk - 1) / g.kchunk;
    g.part = splits > 1 ? net->part : nullptr;
    if (splits > 65535) return hipErrorInvalidValue;
    const dim3 grid((unsigned)tn, 1, (unsigned)splits);
    if (vec) hipLaunchKernelGGL((k_gemv<4>), grid, dim3(MV_T), 0, s, g);
    else hipLaunchKernelGGL((k_gemv<1>), grid, dim3(MV_T), 0, s, g);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || splits == 1) return e;
    hipLaunchKernelGGL(k_splitk_reduce, dim3(grid_for(g.M * g.N)), dim3(GT), 0, s, g, (int)splits);
    return hipGetLastError();
  }
  const int64_t tm = (g.M + BM - 1) / BM, tn = (g.N + BN - 1) / BN;
  const int64_t kslices = (g.K + BK - 1) / BK;
  if (tm > 65535) return hipErrorInvalidValue;
  if (kslices <= 8) {
    // short K (a weight gradient over a small batch): one wave per tile
    g.kchunk = kslices * BK;
    g.part = nullptr;
    const bool rows = tm * tn < ROWS_BELOW;
    const dim3 grid((unsigned)(rows ? tn : (tn + 3) / 4), (unsigned)tm, 1);
    auto go = [&](auto a, auto b) {
      if (rows) hipLaunchKernelGGL((k_gemm<a(), b(), 1, true>), grid, dim3(GT), 0, s, g);
      else hipLaunchKernelGGL((k_gemm<a(), b(), 1, false>), grid, dim3(GT), 0, s, g);
    };
    if (!ta && !tb) go(std::false_type{}, std::false_type{});
    else if (ta && !tb) go(std::true_type{}, std::false_type{});
    else if (!ta && tb) go(std::false_type{}, std::true_type{});
    else go(std::true_type{}, std::true_type{});
    return hipGetLastError();
  }
  // K over the four waves of a workgroup, then over workgroups until two are resident
  // on every compute unit (the LDS sum holds 64 KB), at least two blocks a wave
  const int64_t tiles = tm * tn;
  int64_t splits = tiles < 512 ? 512 / tiles : 1;
  if (splits > kslices / 8) splits = kslices / 8;
  if (splits > cap) splits = cap;
  if (splits < 1) splits = 1;
  const int64_t per = (kslices + 4 * splits - 1) / (4 * splits);
  g.kchunk = per * BK;
  splits = (g.K + 4 * g.kchunk - 1) / (4 * g.kchunk);
  if (splits < 1) splits = 1;
  g.part = splits > 1 ? net->part : nullptr;
  if (splits > 65535) return hipErrorInvalidValue;
  const dim3 grid((unsigned)tn, (unsigned)tm, (unsigned)splits);
  if (!ta && !tb) hipLaunchKernelGGL((k_gemm<false, false, 4, false>), grid, dim3(GT), 0, s, g);
  else if (ta && !tb) hipLaunchKernelGGL((k_gemm<true, false, 4, false>), grid, dim3(GT), 0, s, g);
  else if (!ta && tb) hipLaunchKernelGGL((k_gemm<false, true, 4, false>), grid, dim3(GT), 0, s, g);
  else hipLaunchKernelGGL((k_gemm<true, true, 4, false>), grid, dim3(GT), 0, s, g);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || splits == 1) return e;
  hipLaunchKernelGGL(k_splitk_reduce, dim3(grid_for(g.M * g.N)), dim3(GT), 0, s, g, (int)splits);
  return hipGetLastError();
}

// Row chunks of the loss's Gram matrices for a batch: some 1024 workgroups in all, at
// least 256 rows a chunk; batch (cu + cv) never exceeds loss_chunk_cap(max_batch).
void loss_chunks(const rpca_mlp* n, int batch, LossArgs* a) {
  int per = (int)(((int64_t)n->mu * batch + 1023) / 1024);
  if (per < 256) per = 256;
  if (per > n->mu) per = n->mu;
  a->per = per;
  a->cu = (n->mu + per - 1) / per;
  a->cv = (n->nv + per - 1) / per;
}
int64_t loss_chunk_cap(const rpca_mlp* n) {
  LossArgs a;
  int64_t cap = 0;
  for (int b = 1; b <= n->max_batch; ++b) {
    loss_chunks(n, b, &a);
    const int64_t c = (int64_t)b * (a.cu + a.cv);
    if (c > cap) cap = c;
  }
  return cap;
}

GemmArgs gemm_args(const float* A, int64_t lda, const float* B, int64_t ldb, float* C, int64_t ldc,
                   int64_t M, int64_t N, int64_t K) {
  GemmArgs g;
  memset(&g, 0, sizeof(g));
  g.A = A;
  g.B = B;
  g.C = C;
  g.M = M;
  g.N = N;
  g.K = K;
  g.lda = lda;
  g.ldb = ldb;
  g.ldc = ldc;
  return g;
}

hipError_t forward_into(rpca_mlp* n, const float* x, int batch, float* y, bool training, hipStream_t s) {
  GemmArgs g1 = gemm_args(x, n->d_in, n->param[0], n->d_h, n->h, n->d_h, batch, n->d_h, n->d_in);
  g1.bias = n->param[1];
  g1.relu = 1;
  hipError_t e = training || batch > MV ? gemm_in_order(n, g1, s) : gemm(n, g1, false, false, s);
  if (e != hipSuccess) return e;
  GemmArgs g2 = gemm_args(n->h, n->d_h, n->param[2], n->d_out, y, n->d_out, batch, n->d_out, n->d_h);
  g2.bias = n->param[3];
  return gemm(n, g2, false, false, s);
}

void free_net(rpca_mlp* n) {
  for (int t = 0; t < 4; ++t) {
    if (n->param[t]) (void)hipFree(n->param[t]);
    if (n->grad[t]) (void)hipFree(n->grad[t]);
    if (n->mom1[t]) (void)hipFree(n->mom1[t]);
    if (n->mom2[t]) (void)hipFree(n->mom2[t]);
  }
  if (n->h) (void)hipFree(n->h);
  if (n->y) (void)hipFree(n->y);
  if (n->dy) (void)hipFree(n->dy);
  if (n->dz) (void)hipFree(n->dz);
  if (n->part) (void)hipFree(n->part);
  if (n->grams) (void)hipFree(n->grams);
  if (n->gpart) (void)hipFree(n->gpart);
  if (n->lossb) (void)hipFree(n->lossb);
  delete n;
}

}  // namespace

extern "C" {

int rpca_mlp_create(int32_t d_in, int32_t d_h, int32_t mu, int32_t nv, int32_t k, int32_t max_batch,
                    uint64_t seed, rpca_mlp** out) {
  if (!out || d_in <= 0 || d_h <= 0 || mu <= 0 || nv <= 0 || k <= 0 || k > KMAX_LOSS ||
      max_batch < 1 || max_batch > 4096)
    return RPCA_EINVAL;
  *out = nullptr;
  rpca_mlp* n = new rpca_mlp;
  memset(n, 0, sizeof(*n));
  n->d_in = d_in;
  n->d_h = d_h;
  n->mu = mu;
  n->nv = nv;
  n->k = k;
  n->max_batch = max_batch;
  n->d_out = (int64_t)(mu + nv) * k;
  n->count[0] = (int64_t)d_in * d_h;
  n->count[1] = d_h;
  n->count[2] = (int64_t)d_h * n->d_out;
  n->count[3] = n->d_out;
  n->part_cap = (int64_t)64 * max_batch * (d_h > 512 ? d_h : 512);
  bool ok = true;
  for (int t = 0; t < 4 && ok; ++t) {
    const size_t bytes = (size_t)n->count[t] * 4;
    ok = hipMalloc(&n->param[t], bytes) == hipSuccess && hipMalloc(&n->grad[t], bytes) == hipSuccess &&
         hipMalloc(&n->mom1[t], bytes) == hipSuccess && hipMalloc(&n->mom2[t], bytes) == hipSuccess &&
         hipMemset(n->mom1[t], 0, bytes) == hipSuccess && hipMemset(n->mom2[t], 0, bytes) == hipSuccess &&
         hipMemset(n->grad[t], 0, bytes) == hipSuccess;
  }
  ok = ok && hipMalloc(&n->h, (size_t)max_batch * d_h * 4) == hipSuccess &&
       hipMalloc(&n->dz, (size_t)max_batch * d_h * 4) == hipSuccess &&
       hipMalloc(&n->y, (size_t)max_batch * n->d_out * 4) == hipSuccess &&
       hipMalloc(&n->dy, (size_t)max_batch * n->d_out * 4) == hipSuccess &&
       hipMalloc(&n->part, (size_t)n->part_cap * 4) == hipSuccess &&
       hipMalloc(&n->grams, (size_t)max_batch * 6 * k * k * 8) == hipSuccess &&
       hipMalloc(&n->gpart, (size_t)loss_chunk_cap(n) * 3 * k * k * 8) == hipSuccess &&
       hipMalloc(&n->lossb, (size_t)max_batch * 8) == hipSuccess;
  if (!ok) {
    free_net(n);
    return RPCA_ENOMEM;
  }
  // He initialisation of the weights, zero biases
  const int64_t fan[2] = {d_in, d_h};
  for (int l = 0; l < 2; ++l) {
    const int t = 2 * l;
    std::vector<float> w((size_t)n->count[t]);
    const double sd = sqrt(2.0 / (double)fan[l]);
    const uint64_t s = mix64(seed + 0x51ED2701ull * (l + 1));
    for (int64_t i = 0; i < n->count[t]; ++i) w[i] = (float)(sd * gauss(s, (uint64_t)i));
    std::vector<float> z((size_t)n->count[t + 1], 0.f);
    if (hipMemcpy(n->param[t], w.data(), w.size() * 4, hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(n->param[t + 1], z.data(), z.size() * 4, hipMemcpyHostToDevice) != hipSuccess) {
      free_net(n);
      return RPCA_EHIP;
    }
  }
  *out = n;
  return RPCA_OK;
}

int rpca_mlp_param(rpca_mlp* n, int32_t which, float** ptr, int64_t* count) {
  if (!n || which < 0 || which > 3 || !ptr) return RPCA_EINVAL;
  *ptr = n->param[which];
  if (count) *count = n->count[which];
  return RPCA_OK;
}

int rpca_mlp_grad(rpca_mlp* n, int32_t which, float** ptr, int64_t* count) {
  if (!n || which < 0 || which > 3 || !ptr) return RPCA_EINVAL;
  *ptr = n->grad[which];
  if (count) *count = n->count[which];
  return RPCA_OK;
}

int rpca_mlp_forward(rpca_mlp* n, const float* x, int32_t batch, float* y, void* stream) {
  if (!n || !x || !y || batch < 1 || batch > n->max_batch) return RPCA_EINVAL;
  return forward_into(n, x, batch, y, false, (hipStream_t)stream) == hipSuccess ? RPCA_OK : RPCA_EHIP;
}

int rpca_mlp_loss_grad(rpca_mlp* n, const float* x, const float* TU, const float* TV, int32_t batch,
                       double* loss, void* stream) {
  if (!n || !x || !TU || !TV || !loss || batch < 1 || batch > n->max_batch) return RPCA_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  if (forward_into(n, x, batch, n->y, true, s) != hipSuccess) return RPCA_EHIP;
  LossArgs l;
  memset(&l, 0, sizeof(l));
  l.y = n->y;
  l.TU = TU;
  l.TV = TV;
  l.mu = n->mu;
  l.nv = n->nv;
  l.k = n->k;
  l.batch = batch;
  l.d_out = n->d_out;
  l.gpart = n->gpart;
  l.grams = n->grams;
  l.lossb = n->lossb;
  l.loss = loss;
  l.dy = n->dy;
  loss_chunks(n, batch, &l);
  const dim3 gg((unsigned)(l.cu + l.cv), (unsigned)batch);
  const int nb16 = (n->mu + 15) / 16 + (n->nv + 15) / 16;
  const int dyb = (nb16 + 15) / 16;  // four 16-row blocks a wave
  const dim3 gd((unsigned)dyb, (unsigned)batch);
  if (n->k <= 16) hipLaunchKernelGGL((k_loss_grams<1>), gg, dim3(GT), 0, s, l);
  else hipLaunchKernelGGL((k_loss_grams<2>), gg, dim3(GT), 0, s, l);
  hipLaunchKernelGGL(k_loss_finish, dim3(batch), dim3(GT), 0, s, l);
  if (n->k <= 16) hipLaunchKernelGGL((k_loss_dy<1>), gd, dim3(GT), 0, s, l);
  else hipLaunchKernelGGL((k_loss_dy<2>), gd, dim3(GT), 0, s, l);
  if (hipGetLastError() != hipSuccess) return RPCA_EHIP;
  // dW2 = h^T dy
  GemmArgs a = gemm_args(n->h, n->d_h, n->dy, n->d_out, n->grad[2], n->d_out, n->d_h, n->d_out, batch);
  if (gemm(n, a, true, false, s) != hipSuccess) return RPCA_EHIP;
  // dz = (dy W2^T) .* (h > 0)
  GemmArgs b = gemm_args(n->dy, n->d_out, n->param[2], n->d_out, n->dz, n->d_h, batch, n->d_h, n->d_out);
  b.gate = n->h;
  b.ldg = n->d_h;
  if (gemm(n, b, false, true, s) != hipSuccess) return RPCA_EHIP;
  // dW1 = x^T dz
  GemmArgs c = gemm_args(x, n->d_in, n->dz, n->d_h, n->grad[0], n->d_h, n->d_in, n->d_h, batch);
  if (gemm(n, c, true, false, s) != hipSuccess) return RPCA_EHIP;
  // db2 = colsum(dy), db1 = colsum(dz)
  ColsumArgs cs;
  cs.A[0] = n->dy;
  cs.A[1] = n->dz;
  cs.rows = batch;
  cs.cols[0] = n->d_out;
  cs.cols[1] = n->d_h;
  cs.out[0] = n->grad[3];
  cs.out[1] = n->grad[1];
  const int64_t cmax = n->d_out > n->d_h ? n->d_out : n->d_h;
  hipLaunchKernelGGL(k_colsum, dim3(grid_for(cmax, 1 << 30), 2), dim3(GT), 0, s, cs);
  return hipGetLastError() == hipSuccess ? RPCA_OK : RPCA_EHIP;
}

int rpca_mlp_adam_step(rpca_mlp* n, float lr, float beta1, float beta2, float eps, void* stream) {
  if (!n || !(lr > 0.f) || !(beta1 >= 0.f && beta1 < 1.f) || !(beta2 >= 0.f && beta2 < 1.f) || !(eps > 0.f))
    return RPCA_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  n->step += 1;
  const float bc1 = (float)(1.0 - pow((double)beta1, n->step));
  const float bc2 = (float)(1.0 - pow((double)beta2, n->step));
  AdamArgs a;
  int64_t cmax = 0;
  for (int t = 0; t < 4; ++t) {
    a.p[t] = n->param[t];
    a.g[t] = n->grad[t];
    a.m1[t] = n->mom1[t];
    a.m2[t] = n->mom2[t];
    a.n[t] = n->count[t];
    if (n->count[t] > cmax) cmax = n->count[t];
  }
  a.lr = lr;
  a.b1 = beta1;
  a.b2 = beta2;
  a.eps = eps;
  a.bc1 = bc1;
  a.bc2 = bc2;
  hipLaunchKernelGGL(k_adam, dim3(grid_for((cmax + 3) / 4), 4), dim3(GT), 0, s, a);
  return hipGetLastError() == hipSuccess ? RPCA_OK : RPCA_EHIP;
}

int rpca_mlp_train_step(rpca_mlp* n, const float* x, const float* TU, const float* TV, int32_t batch,
                        float lr, double* loss, void* stream) {
  const int rc = rpca_mlp_loss_grad(n, x, TU, TV, batch, loss, stream);
  if (rc != RPCA_OK) return rc;
  return rpca_mlp_adam_step(n, lr, 0.9f, 0.999f, 1e-8f, stream);
}

void rpca_mlp_destroy(rpca_mlp* n) {
  if (n) free_net(n);
}

int rpca_window_features(const float* X, int64_t W, int64_t H, int32_t frames, int32_t f,
                         const float* shift, const float* scale, float* feat, void* stream) {
  if (!X || !feat || W <= 0 || H <= 0 || frames <= 0 || f <= 0 || W % f || H % f ||
      (!shift) != (!scale))
    return RPCA_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  const int64_t mu = (W / f) * (H / f);
  const int64_t nblk = (mu + FB - 1) / FB;
  const bool vec = f == 4 && ((uintptr_t)X & 15) == 0;
  const dim3 grid((unsigned)(nblk + frames));
  if (vec) hipLaunchKernelGGL((k_features<true>), grid, dim3(FT), 0, s, X, W, H, (int)frames, (int)f, nblk, shift, scale, feat);
  else hipLaunchKernelGGL((k_features<false>), grid, dim3(FT), 0, s, X, W, H, (int)frames, (int)f, nblk, shift, scale, feat);
  return hipGetLastError() == hipSuccess ? RPCA_OK : RPCA_EHIP;
}

int rpca_pool_rows(const float* A, int64_t W, int64_t H, int32_t f, int32_t c, float* out, void* stream) {
  if (!A || !out || W <= 0 || H <= 0 || f <= 0 || c <= 0 || W % f || H % f) return RPCA_EINVAL;
  const int64_t n = (W / f) * (H / f) * c;
  hipLaunchKernelGGL(k_pool_rows, dim3(grid_for(n, 1 << 30)), dim3(GT), 0, (hipStream_t)stream, A, W, H, f,
                     c, out);
  return hipGetLastError() == hipSuccess ? RPCA_OK : RPCA_EHIP;
}

int rpca_upsample_rows(const float* A, int64_t W, int64_t H, int32_t f, int32_t c, float* out, void* stream) {
  if (!A || !out || W <= 0 || H <= 0 || f <= 0 || c <= 0 || W % f || H % f) return RPCA_EINVAL;
  const int64_t n = W * H * c;
  hipLaunchKernelGGL(k_upsample_rows, dim3(grid_for(n, 1 << 30)), dim3(GT), 0, (hipStream_t)stream, A, W, H,
                     f, c, out);
  return hipGetLastError() == hipSuccess ? RPCA_OK : RPCA_EHIP;
}

}  // extern "C"
