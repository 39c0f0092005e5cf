// Fused thin Gram product Z = Op^T (Op W) in one pass over X, for rank k <= 16
// and n <= 256 columns (one chunk of at most 16 column tiles).
//
// Op is the certificate's gradient operator G = Omega .* rho'(U V^T - X) (the
// residual source; its power iteration on M^T M needs D^T D x = G^T G x / lam_L^2,
// Sec. 3.4) or the data Omega .* X (the randomized-SVD start's subspace iteration
// on A^T A, Sec. 4.2).  Separate left and right sweeps would read X twice and
// carry FP64 vectors; here each 16-row strip
//   1. forms its G tiles exactly as the objective sweep does (MFMA with the
//      accumulator seeded by X and the A operand -U, then the clip), keeps them
//      in registers and accumulates Y_s = G_s W (16 x 16, through a per-wave
//      transpose tile);
//   2. once the strip's Y_s is complete, adds G_s^T Y_s to the per-tile Z
//      accumulators: Y_s is already in the B-operand layout of that product
//      (rows 4g + r of column c in lane (g, c)) and the G tiles in its A layout.
// Products and the per-workgroup sums are FP32 (MFMA), the sums over workgroups
// FP64 in a fixed order.  With the residual source the kernel computes
// (-G)^T (-G W) = G^T G W, so no negation is needed.
//
// Work split: as the objective sweep's split by columns -- a workgroup of eight waves, CG
// column groups of at most four tiles times RQ = 8 / CG row lanes; the V and W operands and
// the Z sums of a wave's tiles stay in registers.  The column groups' Y sums of a strip meet
// in LDS, so step 2 of a strip runs beside step 1 of the next: one barrier per strip, with
// every wave's products of both steps between two barriers.  Two workgroups per compute unit:
// while one waits at its barrier the other's waves have products to issue.
//
// What bounds it: at 76800 x 200 X takes 13.5 us at the card's copy rate, the matrix pipes
// are busy for 10 us (11 products of 32 cycles per tile, 8 with the data source), and they
// do not overlap VALU work.  With whole strips per wave (13 tiles in one wave's registers,
// one wave per SIMD, operands from LDS) it took 33.0 us with the residual source and 20.0
// with the data; this split takes 25.7 and 19.8 (one
// workgroup per compute unit with twice the registers: 32 and 20).
#include "sweep_cols.h"

namespace {

using rpca_cols::BUF_DWORD3;
using rpca_cols::f4;
using rpca_cols::mfma_f32;
using rpca_cols::NT;
using rpca_cols::TS;
using rpca_cols::WAVES;

constexpr int GA_TMAX = 16;   // column tiles (n <= 256)
constexpr int GA_TW = 4;      // most tiles of a wave

// Column groups: the fewest that leave a wave at most four tiles.
__host__ __device__ constexpr int ga_groups(int ntiles) { return ntiles <= GA_TW ? 1 : ntiles <= 2 * GA_TW ? 2 : 4; }

template <bool RESID, bool ELASTIC, bool MASKED>
__global__ __launch_bounds__(NT, 4) void k_gram_apply(rpca::GramApplyArgs a) {
  __shared__ __align__(16) float sT[WAVES * 2 * 16 * TS];  // transpose tiles, two per wave
  __shared__ __align__(16) float sY[2 * WAVES * 256];      // Y sums of the waves, two strips; at the end Z
  if (a.skip && *a.skip != 0.0) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 15, g = lane >> 4;
  const int64_t m = a.m;
  const int n = (int)a.n, k = a.k;
  const float lam_s = a.lam_s, kappa = a.kappa;
  const int ntiles = (n + 15) >> 4;
  const int cgs = ga_groups(ntiles), lcg = cgs == 1 ? 0 : cgs == 2 ? 1 : 2, rqs = WAVES >> lcg;
  const int rq = w >> lcg, cg = (w + rq) & (cgs - 1);  // the waves of a SIMD take different groups
  const int t0 = (cg * ntiles) >> lcg, nt = (((cg + 1) * ntiles) >> lcg) - t0;  // this wave's tiles (1 .. 4)
  float* const myT = sT + w * 2 * 16 * TS;

  // this workgroup's strips: whole pairs (a pair shares its 128-byte lines of X), every
  // rqs-th strip this wave's
  const int64_t nstrips = (m + 15) >> 4, npairs = (nstrips + 1) >> 1;
  const int R = gridDim.x, rg = blockIdx.x;
  const int64_t s_lo = 2 * (rg * npairs / R), s_hi = 2 * ((rg + 1) * npairs / R);
  const int64_t nst = (s_hi < nstrips ? s_hi : nstrips) - s_lo;
  const int64_t its = (nst + rqs - 1) / rqs;
  const int64_t s_end = s_lo + nst;
  const int64_t s_full = nt * m < ((int64_t)1 << 26) ? (m >> 4) : 0;  // strips read through the buffer resource

  const int j0 = 16 * t0, vcols = (n - j0 < 16 * nt ? n - j0 : 16 * nt);
  const float* __restrict__ Xw = a.X + j0 * m;
  const __amdgpu_buffer_rsrc_t xrs = __builtin_amdgcn_make_buffer_rsrc(
      (void*)Xw, (short)0, s_full ? (int)((uint32_t)vcols * ((uint32_t)m * 4u)) : 0, BUF_DWORD3);
  const uint32_t lane_off = (uint32_t)c * ((uint32_t)m * 4u) + 16u * g;
  const uint32_t tile_step = 64u * (uint32_t)m;
  const uint32_t* __restrict__ Mw = MASKED ? a.mask + (int64_t)j0 * a.mw : nullptr;
  // X (and the mask words) of tile t of strip s; past the strips read through the resource
  // the first one's, not used
  auto load_tile = [&](int64_t s, int t, f4& x, uint32_t& mb) {
    const uint32_t at = s < s_full && s < s_end ? (uint32_t)s * 64u : 0u;
    x = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(xrs, lane_off + (at + t * tile_step), 0, 0));
    if (MASKED) {
      const int last = vcols > 16 * t ? vcols - 16 * t - 1 : 0;
      const int64_t sc = s < s_end ? s : s_lo;
      mb = Mw[(int64_t)((c < last ? c : last) + 16 * t) * a.mw + (sc >> 1)] >> (16 * (int)(sc & 1) + 4 * g);
    }
  };
  // residual A operand of strip s: -U[row c][4q + g] (rows past m and ranks past k: 0)
  auto load_ua = [&](int64_t s, float (&ua)[4]) {
    if (!RESID) return;
    const int64_t row = (s < s_end ? s : s_lo) * 16 + c;
    const float* __restrict__ Us = a.U + (row < m ? row : m - 1) * k;
#pragma unroll
    for (int q = 0; q < 4; ++q) ua[q] = Us[4 * q + g < k ? 4 * q + g : k - 1];
  };

  auto run = [&](auto nwc) {
    constexpr int NW = decltype(nwc)::value;
    float ua[4] = {0.f, 0.f, 0.f, 0.f};
    f4 x[NW];
    uint32_t mb[NW] = {};
    load_ua(s_lo + rq, ua);
    // residual operand V[16 t + c][4q + g], Y operand W[16 t + 4g + q][c]
    // (loads return in order: what the first products need is requested first)
    float vr[RESID ? NW : 1][4], wg[NW][4];
    if (RESID)
#pragma unroll
      for (int t = 0; t < NW; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int jv = j0 + 16 * t + c, kk = 4 * q + g;
          vr[t][q] = a.V[(int64_t)(jv < n ? jv : n - 1) * k + (kk < k ? kk : k - 1)];
        }
#pragma unroll
    for (int t = 0; t < NW; ++t) load_tile(s_lo + rq, t, x[t], mb[t]);
#pragma unroll
    for (int t = 0; t < NW; ++t)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int jv = j0 + 16 * t + c, jw = j0 + 16 * t + 4 * g + q;
        const float u = a.W[(int64_t)(jw < n ? jw : n - 1) * 16 + c];
        wg[t][q] = jw < n ? u : 0.f;
        if (RESID) vr[t][q] = jv < n && 4 * q + g < k ? vr[t][q] : 0.f;
      }
    f4 G[NW], za[NW];
#pragma unroll
    for (int t = 0; t < NW; ++t) G[t] = za[t] = f4{0.f, 0.f, 0.f, 0.f};

#pragma unroll 1
    for (int64_t it = 0; it <= its; ++it) {
      if (it > 0) {  // Z += G^T Y of the strip before
        f4 y = f4{0.f, 0.f, 0.f, 0.f};
        const float* ys = sY + (((int)(it - 1) & 1) * WAVES + (rq << lcg)) * 256 + lane * 4;
#pragma unroll 4
        for (int q = 0; q < cgs; ++q) y += *reinterpret_cast<const f4*>(ys + q * 256);
#pragma unroll
        for (int h = 0; h < NW; h += 2) {  // a strip's sums on their own, then added: short chains
          f4 z[2];
#pragma unroll
          for (int v = 0; v < 2; ++v) z[v] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int v = 0; v < 2; ++v)
              if (h + v < NW) z[v] = mfma_f32(G[h + v < NW ? h + v : 0][r], y[r], z[v]);
#pragma unroll
          for (int v = 0; v < 2; ++v)
            if (h + v < NW) za[h + v < NW ? h + v : 0] += z[v];
        }
      }
      if (it == its) break;
      const int64_t s = s_lo + rq + it * rqs;
      if (s >= s_full || s >= s_end) {
        // by address, through the transpose tile (the ragged last strip, very long columns,
        // a row lane without a strip: zeros); the lane index is hidden from the compiler so
        // that this rare path's addresses are not kept across the strips
        int co = c;
        asm volatile("" : "+v"(co));
#pragma unroll
        for (int t = 0; t < NW; ++t) {
#pragma unroll 1
          for (int q = 0; q < 4; ++q) {
            const int64_t row = s * 16 + 4 * g + q;
            myT[co * TS + 4 * g + q] = row < m && s < s_end && 16 * t + co < vcols ? Xw[(16 * t + co) * m + row] : 0.f;
          }
          x[t] = *reinterpret_cast<const f4*>(myT + co * TS + 4 * g);
        }
      }
      if (RESID) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if (q == 3 && k <= 12) continue;
          const float u = 4 * q + g < k && s * 16 + c < m && s < s_end ? -ua[q] : 0.f;
#pragma unroll
          for (int t = 0; t < NW; ++t) x[t] = mfma_f32(u, vr[t][q], x[t]);
        }
        load_ua(s + rqs, ua);
      }
      f4 y = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int h = 0; h < NW; h += 2) {
#pragma unroll
        for (int v = 0; v < 2; ++v) {
          const int t = h + v;
          if (t >= NW) continue;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            float gv = x[t][r];
            if (RESID) {
              // -rho'(R) from the negated residual (clip, elastic slope beyond it)
              const float cl = __builtin_amdgcn_fmed3f(gv, -lam_s, lam_s);
              gv = ELASTIC ? fmaf(kappa, gv - cl, cl) : cl;
            }
            if (MASKED && !((mb[t] >> r) & 1u)) gv = 0.f;
            G[t][r] = gv;
            myT[v * 16 * TS + (4 * g + r) * TS + c] = G[t][r];
          }
        }
#pragma unroll
        for (int v = 0; v < 2; ++v)
          if (h + v < NW) load_tile(s + rqs, h + v, x[h + v], mb[h + v]);
        __builtin_amdgcn_sched_barrier(0);
        f4 gt[2], yt[2];
#pragma unroll
        for (int v = 0; v < 2; ++v) {
          gt[v] = *reinterpret_cast<const f4*>(myT + v * 16 * TS + c * TS + 4 * g);
          yt[v] = f4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int v = 0; v < 2; ++v)
            if (h + v < NW) yt[v] = mfma_f32(gt[v][q], wg[h + v < NW ? h + v : 0][q], yt[v]);
#pragma unroll
        for (int v = 0; v < 2; ++v)
          if (h + v < NW) y += yt[v];
      }
      *reinterpret_cast<f4*>(sY + (((int)it & 1) * WAVES + (rq << lcg) + cg) * 256 + lane * 4) = y;
      __syncthreads();
    }

    // ---- the row lanes' Z sums to lane 0 through LDS, fixed order; as many tiles at a time
    // as fit (the same barriers in every wave)
    float* zp = a.part + (int64_t)rg * n * 16;
    const int per = cgs == 4 ? 4 : 2;
#pragma unroll
    for (int h = 0; h < GA_TW; h += 2) {
      if (h >= per || h == 0) __syncthreads();  // the sums before have been read
#pragma unroll
      for (int v = 0; v < 2; ++v)
        if (rq > 0 && h + v < NW)
          *reinterpret_cast<f4*>(sY + ((((rq - 1) << lcg) + cg) * per + ((h + v) & (per - 1))) * 256 + lane * 4) =
              za[h + v < NW ? h + v : 0];
      if (h + 2 < per) continue;
      __syncthreads();
#pragma unroll
      for (int t = 0; t < NW; ++t) {
        if (rq > 0 || t < h + 2 - per || t >= h + 2) continue;
        f4 z = za[t];
        for (int q = 0; q + 1 < rqs; ++q)
          z += *reinterpret_cast<const f4*>(sY + (((q << lcg) + cg) * per + (t & (per - 1))) * 256 + lane * 4);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int j = 16 * t + 4 * g + r;
          if (j < vcols) zp[(j0 + j) * 16 + c] = z[r];
        }
      }
    }
  };
  if (nt == 4) run(std::integral_constant<int, 4>{});
  else if (nt == 3) run(std::integral_constant<int, 3>{});
  else if (nt == 2) run(std::integral_constant<int, 2>{});
  else run(std::integral_constant<int, 1>{});
}

// Z[j * ldz + col0 + p] = scale * (sum over workgroups r of part[r][j * 16 + p]), p < b.
// One pass: a block takes GR_OUT consecutive outputs; its GR_SL row slices sum
// workgroups sl, sl + GR_SL, ... in FP64 (all loads of a slice in flight at
// once), then one thread per output adds the slices in slice order.  The order
// depends only on the number of workgroups.
constexpr int GR_OUT = 16, GR_SL = 16, GR_INF = 16;
__global__ __launch_bounds__(256) void k_ga_reduce(const float* __restrict__ part, int64_t n, int rows, int b,
                                                   double scale, double* __restrict__ Z, int ldz, int col0,
                                                   const double* __restrict__ skip) {
  if (skip && *skip != 0.0) return;
  __shared__ double sh[GR_SL][GR_OUT + 1];
  const int oo = threadIdx.x & (GR_OUT - 1), sl = threadIdx.x / GR_OUT;
  const int64_t outs = n * b;
  const int64_t o = (int64_t)blockIdx.x * GR_OUT + oo;
  const int64_t oc = o < outs ? o : outs - 1;
  const int64_t j = oc / b;
  const int64_t src = j * 16 + (oc - j * b);
  const int64_t stride = n * 16;
  double s = 0.0;
  for (int r0 = sl; r0 < rows; r0 += GR_SL * GR_INF) {
    float x[GR_INF];
#pragma unroll
    for (int e = 0; e < GR_INF; ++e) {  // clamped rows: every load issued before the first use
      const int r = r0 + e * GR_SL;
      x[e] = part[(int64_t)(r < rows ? r : rows - 1) * stride + src];
    }
#pragma unroll
    for (int e = 0; e < GR_INF; ++e) s += r0 + e * GR_SL < rows ? (double)x[e] : 0.0;
  }
  sh[sl][oo] = s;
  __syncthreads();
  if (sl == 0 && o < outs) {
    double t = 0.0;
#pragma unroll
    for (int q = 0; q < GR_SL; ++q) t += sh[q][oo];
    Z[j * ldz + col0 + (o - j * b)] = scale * t;
  }
}

}  // namespace

namespace rpca {

bool gram_apply_fits(int64_t n, int k) { return n >= 1 && n <= 16 * GA_TMAX && k >= 0 && k <= 16; }

hipError_t launch_gram_apply_pass(const GramApplyArgs& a, bool resid, hipStream_t s) {
  if (!gram_apply_fits(a.n, resid ? a.k : 0) || a.row_groups < 1) return hipErrorInvalidValue;
  const dim3 grid((unsigned)a.row_groups);
  const bool mk = a.mask != nullptr;
  auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(NT), 0, s, a); };
  if (!resid) {
    if (mk) go(k_gram_apply<false, false, true>);
    else go(k_gram_apply<false, false, false>);
  } else if (a.kappa != 0.f) {
    if (mk) go(k_gram_apply<true, true, true>);
    else go(k_gram_apply<true, true, false>);
  } else {
    if (mk) go(k_gram_apply<true, false, true>);
    else go(k_gram_apply<true, false, false>);
  }
  return hipGetLastError();
}

hipError_t launch_gram_apply_sum(const GramApplyArgs& a, double* Z, int ldz, int col0, int b, double scale,
                                 hipStream_t s) {
  if (a.n < 1 || b < 1 || b > 16 || a.row_groups < 1) return hipErrorInvalidValue;
  const int64_t outs = a.n * b;
  hipLaunchKernelGGL(k_ga_reduce, dim3((unsigned)((outs + GR_OUT - 1) / GR_OUT)), dim3(GR_OUT * GR_SL), 0, s,
                     (const float*)a.part, a.n, a.row_groups, b, scale, Z, ldz, col0, a.skip);
  return hipGetLastError();
}

hipError_t launch_gram_apply(const GramApplyArgs& a, bool resid, double* Z, int ldz, int col0, int b, double scale,
                             hipStream_t s) {
  if (b < 1 || b > 16) return hipErrorInvalidValue;
  const hipError_t e = launch_gram_apply_pass(a, resid, s);
  if (e != hipSuccess) return e;
  return launch_gram_apply_sum(a, Z, ldz, col0, b, scale, s);
}

}  // namespace rpca
