// Objective/gradient: launch of the fused sweep (sweep_cols.h, sweep_kernel.h) and the finishing
// reduction with the device-side line-search step.

#include <math.h>

#include <algorithm>
#include <mutex>

#include "linesearch.h"

#include "rpca_internal.h"
#include "sweep_cols.h"
#include "sweep_kernel.h"
#include "wave_sum.h"

namespace {

// ---------------------------------------------------------------------------
// Finishing reduction, one launch.  Blocks of 16 waves:
//   bx < gv_blocks: the G^T U partials of whole rows of V.  A wave sums 16 workgroup rows of
//     64 / k rows of V (lane = output, all 16 loads in flight), `slices` waves side by side;
//     the slices meet in LDS and are added in row order:
//     gV = sum + lam_l V_t, or its preconditioned form.
//   several chunks only: gU = sum over chunks + lam_l U_t, one output per thread.
//   last: the sweep's scalar partials.
// Each block publishes up to four scalars; the last one to arrive forms f and g^T d and, in
// solver mode, runs one step of the line search.
//
// Bound by latency: 2 MB of partials at 76,800 x 200, k = 10, and a chain of a few dependent
// round trips to memory the eight L2 caches share.  As two launches (sums of 16 rows each,
// then their sum and the rest, fenced by a write-back of the L2 in every block) it took 4.8
// and 7.2 us there, 4.9 and 43 us at 8192^2, k = 25; this takes 6.9 and 12.5.  The scalars
// are written through and read past the L2 (agent scope), so no block writes its cache back.
constexpr int FIN_WAVES = 16;
constexpr int FIN_THREADS = 64 * FIN_WAVES;
constexpr int FIN_ROWS = 16;  // workgroup rows per slice

// Waves that share a V row's partials: enough slices of 16 rows for all workgroup rows, a
// power of two (the block's other waves take further rows of V).
__host__ __device__ constexpr int finish_slices(int row_groups) {
  int s = 1;
  while (s < FIN_WAVES && s * FIN_ROWS < row_groups) s *= 2;
  return s;
}

// Block bx of the nblk blocks of one instance.
template <bool TRIAL>
__device__ __forceinline__ void finish_body(const FinishArgs& a, const int bx, const int nblk) {
  __shared__ double sSum[FIN_WAVES][64];
  __shared__ double sPart[FIN_WAVES][7];
  __shared__ int s_last;
  int outi = 0;
  SolverState* st = a.st;
  if (TRIAL) {
    const int phase = st->phase, cur = st->cur;
    LOADED(phase, cur);
    if (phase != PH_TRIAL) return;
    outi = 1 - cur;
  }
  const int k = a.k;
  const int64_t mk = a.m * k;
  const float lam_l = a.lam_l;
  const float* Vt = a.V[outi];
  const float* Ut = a.U[outi];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  double p[4] = {0.0, 0.0, 0.0, 0.0};  // this block's scalars (its type says which)
  if (bx < a.gv_blocks) {
    const int slices = finish_slices(a.row_groups), groups = FIN_WAVES / slices;
    const int sl = w & (slices - 1), grp = w / slices;
    const int rpw = 64 / k, jr = lane / k, c = lane - jr * k;
    const int64_t j = ((int64_t)bx * groups + grp) * rpw + jr, nk = a.n * k, o = j * k + c;
    const bool ok = jr < rpw && j < a.n;
    float v = 0.f, dv = 0.f;
    if (ok && sl == 0) {
      v = Vt[o];
      if (TRIAL) dv = a.dV[o];
    }
    double s = 0.0;
    for (int r0 = 0; r0 < a.row_groups; r0 += slices * FIN_ROWS) {
      const int rb = r0 + sl * FIN_ROWS, left = a.row_groups - rb;
      double t = 0.0;
      if (ok && left > 0) {
        const float* src = a.gvpart + (int64_t)rb * nk + o;
        float x[FIN_ROWS];
#pragma unroll
        for (int e = 0; e < FIN_ROWS; ++e) x[e] = src[(e < left ? e : 0) * nk];
#pragma unroll
        for (int e = 0; e < FIN_ROWS; ++e) t += e < left ? (double)x[e] : 0.0;
      }
      if (r0) __syncthreads();  // the slices of the pass before have been read
      sSum[w][lane] = t;
      __syncthreads();
      if (sl == 0)
        for (int q = 0; q < slices; ++q) s += sSum[w + q][lane];
    }
    if (!a.pc) {
      if (ok && sl == 0) {
        const float gvv = (float)(s + (double)lam_l * (double)v);
        a.gV[outi][o] = gvv;
        p[0] = (double)v * (double)v;
        if (TRIAL) p[1] = (double)gvv * (double)dv;
      }
    } else {
      // preconditioned variables: grad_B = (G^T A) W + lam_l B M_V, ||V||^2 = sum B M_V B^T
      __syncthreads();
      if (sl == 0) sSum[w][lane] = s;
      __syncthreads();
      if (ok && sl == 0) {
        const float* W = a.pc;
        const float* MV = a.pc + 2 * k * k;
        double t1 = 0.0, t2 = 0.0;
        for (int t = 0; t < k; ++t) {
          t1 += sSum[w][jr * k + t] * (double)W[t * k + c];
          t2 += (double)Vt[j * k + t] * (double)MV[t * k + c];
        }
        const float gvv = (float)(t1 + (double)lam_l * t2);
        a.gV[outi][o] = gvv;
        p[0] = (double)v * t2;
        if (TRIAL) p[1] = (double)gvv * (double)dv;
      }
    }
  } else if (bx < nblk - 1) {
    const float* MU = a.pc ? a.pc + k * k : nullptr;
    const int64_t stride = (int64_t)(nblk - 1 - a.gv_blocks) * FIN_THREADS;
    for (int64_t o = (int64_t)(bx - a.gv_blocks) * FIN_THREADS + tid; o < mk; o += stride) {
      double s = 0.0;
      int cc = 0;
      for (; cc + 7 < a.nchunks; cc += 8) {  // eight loads in flight, summed in chunk order
        float x[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = a.gupart[(int64_t)(cc + e) * mk + o];
#pragma unroll
        for (int e = 0; e < 8; ++e) s += (double)x[e];
      }
      for (; cc < a.nchunks; ++cc) s += (double)a.gupart[(int64_t)cc * mk + o];
      double reg = Ut[o];
      if (MU) {  // A M_U
        const int64_t i = o / k;
        const int c = (int)(o % k);
        reg = 0.0;
        for (int t = 0; t < k; ++t) reg += (double)Ut[i * k + t] * (double)MU[t * k + c];
      }
      const float gu = (float)(s + (double)lam_l * reg);
      a.gU[outi][o] = gu;
      if (TRIAL) p[0] += (double)gu * (double)a.dU[o];
    }
    if (!TRIAL) return;  // nothing to publish
  } else {
    for (int q = tid; q < a.sweep_wgs; q += FIN_THREADS)
#pragma unroll
      for (int e = 0; e < 4; ++e) p[e] += a.spart[(int64_t)q * RPCA_NSCAL + e];
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    p[e] = wave_sum63(p[e]);
    if (lane == 63) sPart[w][e] = p[e];
  }
  __syncthreads();
  if (w == 0) {
    if (lane < 4) {
      double t = 0.0;
#pragma unroll
      for (int q = 0; q < FIN_WAVES; ++q) t += sPart[q][lane];
      put_agent(a.fpart + (int64_t)bx * 4 + lane, t);
    }
    if (lane == 0) s_last = arrive(a.counter) == (unsigned)(TRIAL ? nblk : a.gv_blocks + 1) - 1u;
  }
  __syncthreads();
  if (!s_last) return;
  // ||V||^2, gV . dV and gU . dU over the blocks; the scalar block's four sums
  double v7[7] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  for (int b = tid; b < nblk - 1; b += FIN_THREADS) {
    if (b < a.gv_blocks) {
      v7[0] += get_agent(a.fpart + (int64_t)b * 4);
      if (TRIAL) v7[1] += get_agent(a.fpart + (int64_t)b * 4 + 1);
    } else if (TRIAL) {
      v7[2] += get_agent(a.fpart + (int64_t)b * 4);
    }
  }
  if (tid < 4) v7[3] = get_agent(a.fpart + (int64_t)(nblk - 1) * 4 + tid);
#pragma unroll
  for (int e = 0; e < 3; ++e) {
    v7[e] = wave_sum63(v7[e]);
    if (lane == 63) sPart[w][e] = v7[e];
  }
  if (tid < 4) sPart[0][3 + tid] = v7[3];
  __syncthreads();
  double p0 = 0.0, p1 = 0.0, p2 = 0.0;
  for (int q = 0; q < FIN_WAVES; ++q) {
    p0 += sPart[q][0];
    p1 += sPart[q][1];
    p2 += sPart[q][2];
  }
  const double fd = sPart[0][3], uu = sPart[0][4], gd1 = sPart[0][5], g2 = sPart[0][6];
  if (!TRIAL) {
    if (tid == 0) {
      if (a.f_out) *a.f_out = fd + 0.5 * (double)lam_l * (uu + p0);
      if (a.aux_out) {
        a.aux_out[0] = fd;  // phi(U V^T)
        a.aux_out[1] = uu;  // ||U||^2
        a.aux_out[2] = p0;  // ||V||^2
        a.aux_out[3] = g2;  // ||G||_F^2
      }
      *a.counter = 0u;
    }
    return;
  }
  // line-search step on an LDS copy of the state head (one thread), written back by the block
  __shared__ SolverState sst;
  copy_state_head(&sst, st);
  __syncthreads();
  if (tid == 0) {
    sst.dir_pending = 0;  // this trial's direction has been formed
    rpca_ls::line_search_step(&sst, fd + 0.5 * (double)lam_l * (uu + p0), gd1 + p1 + p2);
    *a.counter = 0u;
  }
  __syncthreads();
  copy_state_head(st, &sst);
}

template <bool TRIAL>
__global__ __launch_bounds__(FIN_THREADS) void k_finish(FinishArgs a) {
  finish_body<TRIAL>(a, blockIdx.x, gridDim.x);
}

// Batched form (one launch for every instance of a batch).  off: block offsets of each
// instance in the grid; re-arms the work queues of the batched sweep that preceded it.
template <bool TRIAL>
__global__ __launch_bounds__(FIN_THREADS) void k_finish_batch(const FinishArgs* fa, const int* off, int count,
                                                             unsigned* queue_heads, int nheads) {
  if (blockIdx.x == 0 && (int)threadIdx.x < nheads) queue_heads[threadIdx.x] = 0u;
  int lo = 0, hi = count;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (off[mid] <= (int)blockIdx.x) lo = mid;
    else hi = mid;
  }
  finish_body<TRIAL>(fa[lo], blockIdx.x - off[lo], off[lo + 1] - off[lo]);
}

}  // namespace

namespace rpca {

hipError_t launch_sweep_f32_plain(const SweepArgs&, bool, hipStream_t);
hipError_t launch_sweep_f32_trial(const SweepArgs&, bool, hipStream_t);
hipError_t launch_sweep_bf16_plain(const SweepArgs&, bool, hipStream_t);
hipError_t launch_sweep_bf16_trial(const SweepArgs&, bool, hipStream_t);
hipError_t launch_sweep_f32_elastic(const SweepArgs&, bool, bool, hipStream_t);
hipError_t launch_cols_f32(const SweepArgs&, bool, bool, hipStream_t);
hipError_t launch_cols_bf16(const SweepArgs&, bool, bool, hipStream_t);
hipError_t launch_cols_f32_elastic(const SweepArgs&, bool, bool, hipStream_t);

// Sweep decomposition table, keyed by (split, k bucket, n bucket): the number of
// waves the strips are spread over and the divisor of the widest chunk.
// Defaults are what measurements at the benchmark shapes favoured; rpca_autotune
// replaces entries by timing the candidates of each split on the device.
// The table is process-wide: reads and writes hold its mutex (contexts of a
// batch are set up from several host threads).
namespace {
struct TuneTable {
  std::mutex mu;
  SweepTune t[TUNE_SPLITS][TUNE_KB][TUNE_NB];
  TuneTable() {
    for (int s = 0; s < TUNE_SPLITS; ++s)
      for (int a = 0; a < TUNE_KB; ++a)
        for (int b = 0; b < TUNE_NB; ++b) t[s][a][b] = tune_default(s, a, b);
  }
};
TuneTable& tune_table() {
  static TuneTable tt;  // initialised once, thread-safely
  return tt;
}
}  // namespace

int tune_k_bucket(int k) { return k <= 8 ? 0 : k <= 16 ? 1 : k <= 24 ? 2 : 3; }
int tune_n_bucket(int64_t n) { return n <= 64 ? 0 : n <= 128 ? 1 : n <= 256 ? 2 : n <= 512 ? 3 : 4; }

// Columns: 256 workgroups of eight waves, one per compute unit: what its registers and LDS
// hold.  Strips: workgroups of four waves; k <= 16: two per compute unit; k > 16: one, and for
// more than 512 columns (many chunks, few rows each) four times as many row groups
// (8192 x 8192, k = 25, masked: 444 us at 1,024 waves, 369 at 4,096).
SweepTune tune_default(int split, int kbucket, int nbucket) {
  if (split == TUNE_COLS) return SweepTune{2048, 1};
  return SweepTune{kbucket < 2 ? 2048 : nbucket == TUNE_NB - 1 ? 4096 : 1024, 1};
}

SweepTune tune_get(int split, int k, int64_t n) {
  TuneTable& tt = tune_table();
  std::lock_guard<std::mutex> lock(tt.mu);
  return tt.t[split][tune_k_bucket(k)][tune_n_bucket(n)];
}

void tune_set(int split, int kbucket, int nbucket, SweepTune t) {
  TuneTable& tt = tune_table();
  std::lock_guard<std::mutex> lock(tt.mu);
  tt.t[split][kbucket][nbucket] = t;
}

// Column chunks (each fitting the sweep's LDS budget) and the wave/workgroup
// split of the rows of the split by strips.
int strip_blocks_for(int64_t m, int64_t n, int k, int* row_groups, int* strips_per_wave, int* chunk_w,
                     int* nchunks, SweepTune t) {
  const int kb = (k + 15) / 16;
  int cmax = rpca_sweep::max_chunk(kb, k);
  if (t.chunk_div > 1) cmax = ((cmax / t.chunk_div + 15) / 16) * 16;
  if (cmax < 16) cmax = 16;
  int nch = (int)((n + cmax - 1) / cmax);
  int cw = (int)(((n + nch - 1) / nch + 15) / 16) * 16;
  if (cw > cmax) cw = cmax;
  nch = (int)((n + cw - 1) / cw);
  const int64_t nstrips = (m + 15) / 16;
  // the waves of all chunks together make up the table's target
  int64_t target = (t.target_waves + nch - 1) / nch;
  if (target > nstrips) target = nstrips;
  if (target < 1) target = 1;
  // workgroup rows split the strips as evenly as integers allow (the kernel
  // gives row rg the strips [rg S / R, (rg + 1) S / R))
  int64_t wgs = (target + rpca_sweep::WAVES - 1) / rpca_sweep::WAVES;
  if (wgs > nstrips) wgs = nstrips;
  const int64_t per_wg = (nstrips + wgs - 1) / wgs;
  *row_groups = (int)wgs;
  *strips_per_wave = (int)((per_wg + rpca_sweep::WAVES - 1) / rpca_sweep::WAVES);
  *chunk_w = cw;
  *nchunks = nch;
  return (int)(wgs * nch);
}

int sweep_blocks_for(int64_t m, int64_t n, int k, int* row_groups, int* strips_per_wg, int* chunk_w,
                     int* nchunks, int target_waves) {
  if (target_waves <= 0)
    return col_blocks_for(m, n, k, row_groups, strips_per_wg, chunk_w, nchunks, tune_get(TUNE_COLS, k, n));
  const SweepTune t{target_waves, tune_get(TUNE_STRIPS, k, n).chunk_div};
  return strip_blocks_for(m, n, k, row_groups, strips_per_wg, chunk_w, nchunks, t);
}

// Column chunks (at most 512 columns, cut evenly) and the workgroup split of the rows of the
// split by columns: a workgroup has eight waves and, unless the rows run
// out, at least one strip per row lane.
int col_blocks_for(int64_t m, int64_t n, int k, int* row_groups, int* strips_per_lane, int* chunk_w,
                   int* nchunks, SweepTune t) {
  const int64_t nstrips = (m + 15) / 16;
  int cmax = 16 * rpca_cols::WAVES * rpca_cols::wave_tiles(nstrips);
  if (n < cmax) cmax = (int)((n + 15) / 16) * 16;
  if (t.chunk_div > 1) cmax = ((cmax / t.chunk_div + 15) / 16) * 16;
  int nch = (int)((n + cmax - 1) / cmax);
  int cw = (int)(((n + nch - 1) / nch + 15) / 16) * 16;
  if (cw > cmax) cw = cmax;
  nch = (int)((n + cw - 1) / cw);
  // k > 16, and fewer strips than workgroups side by side: narrower chunks, down to a tile
  // per wave: V and the G^T U sums of a wide chunk are most of a workgroup's time there.  A call
  // with wide and narrow chunks, us: 583 x 359, k = 26: 20.6, 16.5; 300 x 144, k = 20: 16.3, 15.6;
  // 1000 x 500, k = 24: 22.9, 17.3; 600 x 600, k = 32: 20.8, 17.5; 256 x 512, k = 18: 20.1, 15.3;
  // 128 x 2048, k = 25: 22.1, 16.8; 2000 x 300, k = 20: 19.3, 17.8.  For k <= 16 the chunks are as
  // they were: it gains there too, a little later (583 x 359, k = 16: 16.9, 14.8; 512 x 512, k = 8:
  // 15.6, 14.6; 256 x 200 and 300 x 144, k = 10: nothing)
  if (k > 16) {
    const int tiles = (int)((n + 15) / 16);
    while ((nch + 1) * nstrips <= t.target_waves / rpca_cols::WAVES && tiles > rpca_cols::WAVES * nch) ++nch;
    cw = ((tiles + nch - 1) / nch) * 16;
    nch = (int)((n + cw - 1) / cw);
  }
  const int rqs = rpca_cols::WAVES / rpca_cols::col_groups(cw, nch, nstrips);
  // the workgroups of all chunks together make up the table's target; they split the
  // strips as evenly as integers allow
  const int64_t target = (t.target_waves + nch - 1) / nch;
  int64_t wgs = (target + rpca_cols::WAVES - 1) / rpca_cols::WAVES;
  if (wgs > (nstrips + rqs - 1) / rqs) wgs = (nstrips + rqs - 1) / rqs;
  // the kernel counts a workgroup's elements of U in 32 bits
  if (wgs < (nstrips + (1 << 21) - 1) >> 21) wgs = (nstrips + (1 << 21) - 1) >> 21;
  const int64_t per_wg = (nstrips + wgs - 1) / wgs;
  *row_groups = (int)wgs;
  *strips_per_lane = (int)((per_wg + rqs - 1) / rqs);
  *chunk_w = cw;
  *nchunks = nch;
  return (int)(wgs * nch);
}

void sweep_split(SweepArgs* a) {
  a->by_cols = 1;
  const int64_t strips = (a->m + 15) / 16;
  a->sdiv = strips / a->row_groups;
  a->srem = (int32_t)(strips % a->row_groups);
  a->kinv = (uint32_t)(((1ull << 32) + a->k - 1) / (unsigned)a->k);
  const int64_t most = a->sdiv + (a->srem ? 1 : 0);
  const int nst = (int)(most < 4096 ? most : 4096);
  const int cgs = rpca_cols::col_groups(a->chunk_w, a->nchunks, strips);
  a->lcg = cgs == 1 ? 0 : cgs == 2 ? 1 : cgs == 4 ? 2 : 3;
  a->spr = rpca_cols::sweep_round(a->k, a->chunk_w, cgs, false, nst);
  a->spr_bf16 = rpca_cols::sweep_round(a->k, a->chunk_w, cgs, true, nst);
}

hipError_t launch_sweep(const SweepArgs& sa, bool trial, bool bf16, hipStream_t stream) {
  const bool masked = sa.mask != nullptr;
  if (sa.by_cols) {
    if (sa.kappa != 0.f)
      return bf16 ? hipErrorInvalidValue : launch_cols_f32_elastic(sa, trial, masked, stream);
    return bf16 ? launch_cols_bf16(sa, trial, masked, stream) : launch_cols_f32(sa, trial, masked, stream);
  }
  if (sa.kappa != 0.f) {  // elastic-net marginal: FP32 products only (callers reject BF16 first)
    if (bf16) return hipErrorInvalidValue;
    return launch_sweep_f32_elastic(sa, trial, masked, stream);
  }
  if (bf16)
    return trial ? launch_sweep_bf16_trial(sa, masked, stream) : launch_sweep_bf16_plain(sa, masked, stream);
  return trial ? launch_sweep_f32_trial(sa, masked, stream) : launch_sweep_f32_plain(sa, masked, stream);
}

int finish_blocks(int64_t m, int64_t n, int k, int nchunks, int row_groups, int* gv_blocks) {
  const int rows = FIN_WAVES / finish_slices(row_groups) * (64 / k);  // whole rows of V per block
  const int gvb = (int)((n + rows - 1) / rows);
  int gub = 0;
  if (nchunks > 1) {
    // one output per thread (all chunks' partials of it in flight eight at a time)
    gub = (int)std::min<int64_t>((m * k + FIN_THREADS - 1) / FIN_THREADS, 1024);
  }
  if (gv_blocks) *gv_blocks = gvb;
  return gvb + gub + 1;
}

hipError_t launch_finish(const FinishArgs& fa, bool trial, hipStream_t stream) {
  FinishArgs f2 = fa;
  const int blocks = finish_blocks(fa.m, fa.n, fa.k, fa.nchunks, fa.row_groups, &f2.gv_blocks);
  if (trial)
    hipLaunchKernelGGL((k_finish<true>), dim3(blocks), dim3(FIN_THREADS), 0, stream, f2);
  else
    hipLaunchKernelGGL((k_finish<false>), dim3(blocks), dim3(FIN_THREADS), 0, stream, f2);
  return hipGetLastError();
}

hipError_t launch_sweep_batch_f32(int, int, const SweepArgs*, const SweepItem*, int, unsigned*, int, int, bool, bool,
                                  hipStream_t);
hipError_t launch_sweep_batch_bf16(int, int, const SweepArgs*, const SweepItem*, int, unsigned*, int, int, bool,
                                   bool, hipStream_t);
int sweep_batch_grid_f32(int, int, int, bool, bool);
int sweep_batch_grid_bf16(int, int, int, bool, bool);

hipError_t launch_sweep_batch(int kb, int tmax, const SweepArgs* args, const SweepItem* items, int nitems,
                              unsigned* head, int grid, int lds_floats, bool masked, bool trial, bool bf16,
                              hipStream_t s) {
  return bf16 ? launch_sweep_batch_bf16(kb, tmax, args, items, nitems, head, grid, lds_floats, masked, trial, s)
              : launch_sweep_batch_f32(kb, tmax, args, items, nitems, head, grid, lds_floats, masked, trial, s);
}

int sweep_batch_grid(int kb, int tmax, int lds_floats, bool masked, bool trial, bool bf16) {
  return bf16 ? sweep_batch_grid_bf16(kb, tmax, lds_floats, masked, trial)
              : sweep_batch_grid_f32(kb, tmax, lds_floats, masked, trial);
}

int sweep_lds_floats(int kb, int k, int cwp) { return rpca_sweep::lds_floats(kb, k, cwp); }
int sweep_tmax_class(int kb, int ntiles) { return rpca_sweep::tmax_class(kb, ntiles); }

hipError_t launch_finish_batch(const FinishArgs* fa, const int* off, int total, int count, unsigned* queue_heads,
                               int nheads, bool trial, hipStream_t stream) {
  if (nheads > FIN_THREADS) return hipErrorInvalidValue;
  if (trial)
    hipLaunchKernelGGL((k_finish_batch<true>), dim3(total), dim3(FIN_THREADS), 0, stream, fa, off, count, queue_heads,
                       nheads);
  else
    hipLaunchKernelGGL((k_finish_batch<false>), dim3(total), dim3(FIN_THREADS), 0, stream, fa, off, count,
                       queue_heads, nheads);
  return hipGetLastError();
}

hipError_t launch_objgrad(const SweepArgs& sa, const FinishArgs& fa, bool trial, bool bf16,
                          hipStream_t stream) {
  const hipError_t e = launch_sweep(sa, trial, bf16, stream);
  if (e != hipSuccess) return e;
  return launch_finish(fa, trial, stream);
}

}  // namespace rpca
