// Fused Split-SPCP objective/gradient sweep for gfx950, columns split over the waves of a
// workgroup: the sweep of every context that leaves the decomposition to the library.
//
// One pass over X evaluates, tile by tile in registers,
//   R = U V^T - X                 (the residual inside the marginal phi, Sec. 5 eq. Thm5)
//   rho(R), G = Omega .* clip(R)  (Huber value and derivative, Sec. 1 eq. PhiDef, Sec. 3.2 eq. diff)
//   G^T U and G V                 (the two gradient products, chain rule on eq. smoothNC)
// so neither R nor G is ever written to memory.
//
// Work split.  The columns are cut into chunks (grid.y) of at most 512.  A workgroup
// has eight waves: CG column groups (the fewest that leave a wave at most four 16-column
// tiles) times RQ = 8 / CG row lanes.  A wave keeps everything that belongs to its
// columns in registers for the whole kernel -- both V operands of its tiles and the
// G^T U accumulators -- and walks the workgroup's 16-row strips, every RQ-th of them; the
// next strip's X is requested as the current one's registers fall free.  What belongs to
// the rows goes through LDS: the workgroup's U rows are staged once, ahead of X (loads
// return in order), and the column groups' G V sums of each strip meet there.  One
// barrier later the waves finish the rows (regulariser, gradient, scalars), a strip each.
// Rows that do not fit the 160 KB are taken in rounds.
//
// Why this split, and what bounds it.  Per 16 x 16 tile the FP32 products take 11 MFMAs at
// k = 10 (32 cycles each; FP32 MFMAs do not overlap VALU work on gfx950), so at 76800 x 200
// the matrix pipes alone are busy for about 9 us and X takes 13.5 us at the card's copy
// rate; the rest is the fixed cost of a launch (arguments, code, V and U before the first
// strip) and VALU work.  The earlier split (whole strips per wave, V operands read from LDS
// for every tile, all the chunk's G^T U accumulators in registers) took 32.8 us there at
// k = 10, 41.5 us as a solver's trial, 31.9 us in BF16, and 371 us at 8192^2, k = 25; this
// one 26.0, 29.4, 21.4 and 167.  256 x 200: 12.8 to 7.8 us.  Two waves per SIMD and one
// workgroup per compute unit: four waves in 128 registers spilled and took 34.5 to 37 us,
// with shorter rounds and a barrier each.
//
// Per tile:
//   * -R = X - U V^T on MFMA: the accumulator is seeded with X and the A operand holds
//     -U; the Huber step then yields Gn = -G.  In the MFMA output layout (column j =
//     lane%16, rows 4*(lane/16)+r) Gn is already the A operand of G^T U with K running
//     over rows; the B operand holds -U, so the accumulator is +G^T U.
//   * G V contracts over columns: Gn goes through a per-wave 16 x 16 LDS tile (row
//     stride 20 floats: conflict-free both ways) and is read back as the A operand of
//     four consecutive columns a lane.
// FP32 uses v_mfma_f32_16x16x4f32.  BF16, k <= 16: the residual comes from a hi/lo
// split of U and V (v_mfma_f32_16x16x32_bf16 per block of eight ranks: lane group 0
// supplies hi(U) hi(V), 1 hi(U) lo(V), 2 lo(U) hi(V), 3 zeros), close to FP32 accuracy,
// and G, U and V are rounded to bf16 for the two gradient products; k in 17..32: U, V
// and G rounded to bf16 throughout.  Every cross-wave and cross-workgroup sum runs in a
// fixed order: bitwise reproducible.
#pragma once

#include <math.h>

#include <type_traits>

#include "rpca_internal.h"
#include "wave_sum.h"

namespace rpca_cols {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef short s4 __attribute__((ext_vector_type(4)));
typedef uint32_t u4v __attribute__((ext_vector_type(4)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));

constexpr int WAVES = 8;
constexpr int NT = 64 * WAVES;
constexpr int TW = 4;                      // most 16-column tiles of a wave
constexpr int CHUNK_MAX = 16 * TW * WAVES;  // widest column chunk
constexpr int TS = 20;                     // row stride of a transpose tile (floats)
constexpr int TSB = 24;                    // the same for bf16 (shorts)
constexpr int NTT = 2;                     // transpose tiles per wave (two tiles in flight)
constexpr uint32_t BUF_DWORD3 = 0x00020000;  // raw buffer resource word 3 on gfx9 (32-bit data format)

__device__ __forceinline__ f4 mfma_f32(float a, float b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ f4 mfma_bf16(s4 a, s4 b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ f4 mfma_bf16x32(u4v a, u4v b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8, a), __builtin_bit_cast(bf8, b), c, 0, 0, 0);
}

// FP32 -> BF16, round to nearest even, two values per instruction (v_cvt_pk_bf16_f32).
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f2v __attribute__((ext_vector_type(2)));
typedef uint32_t u2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pk2(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f2v{a, b}, bf16x2));
}
__device__ __forceinline__ s4 pack_bf16(float a, float b, float c, float d) {
  return __builtin_bit_cast(s4, u2v{pk2(a, b), pk2(c, d)});
}
__device__ __forceinline__ uint16_t bf16_bits(float x) { return __builtin_bit_cast(uint16_t, (__bf16)x); }
__device__ __forceinline__ float bf16_val(uint16_t b) { return __builtin_bit_cast(float, (uint32_t)b << 16); }

// Most tiles of a wave.  Its X is addressed in 32 bits, 64 bytes a row and tile: four tiles
// below 2^24 rows, two below 2^25 (2^24 x 100, k = 10: 3,103 us; with four, X read by address as
// it is needed, 3,519).  Longer columns are better read by address, four tiles a wave, than a
// tile a wave through the resource (2^25 x 100, k = 4: 6,444 us for 7,818), unless one tile is
// all there is (2^24 x 16, k = 4: 817 us for 1,097).
__host__ __device__ constexpr int wave_tiles(int64_t nstrips) {
  return nstrips >= (1 << 20) && nstrips < (1 << 21) ? 2 : TW;
}

// Column groups of a chunk: the fewest, a power of two, that leave a wave at most that many tiles;
// twice as many while the strips' waves then still run side by side (2048: two per SIMD) --
// a wave's strip is shorter, and with one strip per wave nothing else fills the chip.
__host__ __device__ constexpr int col_groups(int chunk_w, int nchunks, int64_t nstrips) {
  const int tiles = (chunk_w + 15) / 16, tw = wave_tiles(nstrips);
  int cgs = tiles <= tw ? 1 : tiles <= 2 * tw ? 2 : tiles <= 4 * tw ? 4 : 8;
  while (cgs < WAVES && cgs < tiles && 2 * cgs * nchunks * nstrips <= 2048) cgs *= 2;
  return cgs;
}

// LDS layout (floats), for rounds of `spr` strips and ub buffers of U rows (one if the
// workgroup has a single round, else two):
//   sV [cwp][ks]: V rows, row stride ks = k | 1 (odd: spreads the operand reads over the banks)
//   sU [ub][spr][16][ks]: -U'
//   sUb (BF16) [ub][spr][UB]: row r at 20 r: k <= 16: hi and lo bf16 of each block of eight
//      ranks, k > 16: 32 bf16; then [kb][g][c][4] bf16 of rows 4 g .. 4 g + 3 at
//      kk = 16 kb + c (the G^T U operand)
//   sGU [spr][CG][KB][lane][4]: the column groups' G V sums
//   sT [wave][NTT][16 TS]: transpose tiles; at the end the row lanes' G^T U accumulators
constexpr int LDS_LIMIT_FLOATS = 40960 - 128;  // 160 KB per workgroup, less the static part
struct SweepLds {
  int u_at, ub_at, gu_at, t_at, total;
};
__host__ __device__ constexpr SweepLds sweep_lds(int k, int chunk_w, int cgs, bool bf16, int spr, int ubuf) {
  const int kb = (k + 15) / 16, ks = k | 1, rqs = WAVES / cgs;
  const int pad = 16 * kb;  // operand reads run up to a padded rank past the last row
  const int e = (rqs - 1) * cgs * TW * kb * 256, t = WAVES * NTT * 16 * TS;
  SweepLds l{};
  l.u_at = (chunk_w * ks + pad + 3) & ~3;
  l.ub_at = l.u_at + ((ubuf * spr * 16 * ks + pad + 3) & ~3);
  l.gu_at = l.ub_at + (bf16 ? ubuf * spr * (16 * 20 + kb * 128) : 0);
  l.t_at = l.gu_at + spr * cgs * kb * 256;
  l.total = l.t_at + (t > e ? t : e);
  return l;
}
// Strips per round of a workgroup of at most nst strips: all of them if they fit a
// compute unit's LDS, else the most that do beside a second
// buffer of U rows; a multiple of the row lanes.
__host__ __device__ constexpr int sweep_round(int k, int chunk_w, int cgs, bool bf16, int nst) {
  const int rqs = WAVES / cgs, lim = LDS_LIMIT_FLOATS;
  int spr = (nst + rqs - 1) / rqs * rqs;
  if (spr < rqs) spr = rqs;
  if (sweep_lds(k, chunk_w, cgs, bf16, spr, 1).total <= lim) return spr;
  if (spr > 64) spr = 64 / rqs * rqs;
  while (spr > rqs && sweep_lds(k, chunk_w, cgs, bf16, spr, 2).total > lim) spr -= rqs;
  return spr;
}

// Huber value and derivative at one entry of the negated residual Rn = -R (the
// tiles compute X - U V^T): returns Gn = clip(Rn, +-lam_s) = -G.  l1: rho = c R - c^2 / 2
// with c = clip(R), accumulated as the two sums c R (f) and c^2 (g2).  ELASTIC (the
// elastic-net marginal, kappa = mu / (1 + mu)): the derivative continues with slope
// kappa beyond the threshold, Gn = c + kappa (Rn - c), and rho gains kappa (Rn - c)^2 / 2;
// f is rho itself, g2 the squared derivative.  An unobserved entry contributes nothing,
// whatever X holds there (even a NaN).
template <bool ELASTIC, bool MASKED>
__device__ __forceinline__ float huber(float Rn, float lam_s, float kappa, bool observed, float& f, float& g2) {
  float c = __builtin_amdgcn_fmed3f(Rn, -lam_s, lam_s);
  if (!ELASTIC) {
    if (MASKED) {
      c = observed ? c : 0.f;
      Rn = observed ? Rn : 0.f;
    }
    f = fmaf(c, Rn, f);
    g2 = fmaf(c, c, g2);
    return c;
  }
  float h = fmaf(-0.5f, c, Rn), d = Rn - c;
  if (MASKED) {
    c = observed ? c : 0.f;
    h = observed ? h : 0.f;
    d = observed ? d : 0.f;
  }
  f = fmaf(c, h, f);
  f = fmaf(0.5f * kappa * d, d, f);
  const float gn = fmaf(kappa, d, c);
  g2 = fmaf(gn, gn, g2);
  return gn;
}

// KQ = residual steps of four ranks (k <= 4 KQ): 3 or 4 for k <= 16, 6 to 8 above.
template <int KQ, bool MASKED, bool TRIAL, bool BF16, bool ELASTIC>
__device__ __forceinline__ void sweep_item(const SweepArgs& a, const int rg, const int ch, float* lds, double* sRed) {
  constexpr int KB = (KQ + 3) / 4;
  constexpr int UB = 16 * 20 + KB * 128;
  static_assert(!(BF16 && ELASTIC), "the elastic net uses FP32 products");

  if (a.arm && rg == 0 && ch == 0 && threadIdx.x == 0) *a.arm = 0u;
  int cur = 0, outi = 0;
  float alpha = 0.f;
  if (TRIAL) {
    const SolverState* st = a.st;
    const int phase = st->phase;
    const double al = st->alpha;
    cur = st->cur;
    LOADED(phase, cur);
    asm volatile("" ::"s"(al));
    if (phase != PH_TRIAL) return;
    alpha = (float)al;
    outi = 1 - cur;
  }
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform: strip control stays scalar
  const int c = lane & 15, g = lane >> 4;
  const int64_t m = a.m;
  const int k = a.k;
  const float lam_s = a.lam_s, lam_l = a.lam_l, kappa = a.kappa;
  const float* __restrict__ dU = a.dU;
  const float* __restrict__ pc = a.pc;

  const int64_t j_begin = (int64_t)ch * a.chunk_w;
  const int ncols = (int)((a.n - j_begin) < a.chunk_w ? (a.n - j_begin) : a.chunk_w);
  const int ntiles = (ncols + 15) >> 4;
  const int lcg = a.lcg, cgs = 1 << lcg;
  const int rqs = WAVES >> lcg;
  const int spr = BF16 ? a.spr_bf16 : a.spr;  // strips per round
  const int rq = w >> lcg, cg = (w + rq + 2 * (rg >> 8)) & (cgs - 1);
  const int t0 = (cg * ntiles) >> lcg, nt = (((cg + 1) * ntiles) >> lcg) - t0;  // this wave's tiles (0 .. TW)
  const int ks = k | 1;
  const uint32_t kinv = a.kinv;  // idx / k = mulhi(idx, kinv) (k > 1)
  auto row_of = [&](int idx) -> int { return k > 1 ? (int)__umulhi((uint32_t)idx, kinv) : idx; };

  // this workgroup's strips: srem workgroup rows own sdiv + 1, the others sdiv
  const int64_t s_lo = rg * a.sdiv + (rg < a.srem ? rg : a.srem);
  const int nst = (int)(a.sdiv + (rg < a.srem ? 1 : 0));
  const int64_t row0 = s_lo * 16;
  const int nrows = (int)(m - row0 < nst * 16 ? m - row0 : nst * 16);
  const int ubuf = a.sdiv + (a.srem ? 1 : 0) > spr ? 2 : 1;
  const SweepLds lay = sweep_lds(k, a.chunk_w, cgs, BF16, spr, ubuf);
  float* const sV = lds;
  float* const sU = lds + lay.u_at;
  uint16_t* const sUb = reinterpret_cast<uint16_t*>(lds + lay.ub_at);
  float* const sGU = lds + lay.gu_at;
  float* const sT = lds + lay.t_at;
  float* const myT = sT + w * NTT * 16 * TS;

  // ---- V rows and the first round's U rows (the trial point's) to LDS: short, mostly
  // cached, and requested ahead of X, whose first strips take the longest
  const float* __restrict__ U0 = a.U[cur] + row0 * k;
  const float* __restrict__ dU0 = TRIAL ? dU + row0 * k : nullptr;
  auto put_u = [&](int buf, int idx, float u) {  // -U' of element idx of a round
    const int lr = row_of(idx), kk = idx - lr * k;
    const float v = -u;
    sU[(buf * spr * 16 + lr) * ks + kk] = v;
    if constexpr (BF16) {
      uint16_t* su = sUb + (buf * spr + (lr >> 4)) * (2 * UB);
      const int rr = lr & 15;
      const uint16_t hi = bf16_bits(v);
      if (KB == 1) {
        su[rr * 40 + (kk >> 3) * 16 + (kk & 7)] = hi;
        su[rr * 40 + (kk >> 3) * 16 + 8 + (kk & 7)] = bf16_bits(v - bf16_val(hi));
      } else {
        su[rr * 40 + kk] = hi;
      }
      su[640 + (kk >> 4) * 256 + ((rr >> 2) * 16 + (kk & 15)) * 4 + (rr & 3)] = hi;
    }
  };
  constexpr int SB = 8;  // loads in flight per thread
  auto stage_u = [&](int r) {
    const int base = r * spr * 16 * k, have = nrows * k - base, all = spr * 16 * k;  // elements; zero past the rows
#pragma unroll 1
    for (int i0 = tid; i0 < all; i0 += SB * NT) {
      float u[SB], d[SB];
#pragma unroll
      for (int e = 0; e < SB; ++e) {
        const int idx = i0 + e * NT;
        u[e] = d[e] = 0.f;
        if (idx < have && idx < all) {
          u[e] = U0[base + idx];
          if (TRIAL) d[e] = dU0[base + idx];
        }
      }
#pragma unroll
      for (int e = 0; e < SB; ++e) {
        const int idx = i0 + e * NT;
        if (idx < all) {
          if (TRIAL) {
            u[e] = fmaf(alpha, d[e], u[e]);
            if (ch == 0 && idx < have) a.Ut[outi][row0 * k + base + idx] = u[e];
          }
          put_u(r & (ubuf - 1), idx, u[e]);
        }
      }
    }
  };
  {
    const float* __restrict__ Vc = a.V[cur] + j_begin * k;
    const float* __restrict__ dVc = TRIAL ? a.dV + j_begin * k : nullptr;
    const int have = ncols * k, all = ntiles * 16 * k;
#pragma unroll 1
    for (int i0 = tid; i0 < all; i0 += SB * NT) {
      float v[SB], d[SB];
#pragma unroll
      for (int e = 0; e < SB; ++e) {
        const int idx = i0 + e * NT;
        v[e] = d[e] = 0.f;
        if (idx < have) {
          v[e] = Vc[idx];
          if (TRIAL) d[e] = dVc[idx];
        }
      }
#pragma unroll
      for (int e = 0; e < SB; ++e) {
        const int idx = i0 + e * NT;
        if (idx < all) {
          if (TRIAL) {
            v[e] = fmaf(alpha, d[e], v[e]);
            if (rg == 0 && idx < have) a.Vt[outi][j_begin * k + idx] = v[e];
          }
          const int jl = row_of(idx);
          sV[jl * ks + (idx - jl * k)] = v[e];
        }
      }
    }
  }
  stage_u(0);

  // ---- X.  Strips whose 16 rows are all inside X read 16-byte pieces through a buffer
  // resource over the wave's columns (columns past the chunk are out of range and read
  // zero; any 4-byte alignment); the ragged last strip, and columns so long that the wave's
  // pass 32-bit offsets, are read by address
  const int nfull = nt * m < ((int64_t)1 << 26) ? (nrows >> 4) : 0;
  int vcols = ncols - 16 * t0;
  vcols = vcols < 0 ? 0 : vcols > 16 * nt ? 16 * nt : vcols;
  const int64_t jw = j_begin + 16 * t0;  // first column of the wave
  const float* __restrict__ Xw = a.X + jw * m;
  const __amdgpu_buffer_rsrc_t xrs = __builtin_amdgcn_make_buffer_rsrc(
      (void*)Xw, (short)0, nfull ? (int)((uint32_t)vcols * ((uint32_t)m * 4u)) : 0, BUF_DWORD3);
  const uint32_t lane_off = (uint32_t)c * ((uint32_t)m * 4u) + 16u * g + (uint32_t)s_lo * 64u;
  const uint32_t tile_step = 64u * (uint32_t)m;
  const uint32_t* __restrict__ Mw = MASKED ? a.mask + jw * a.mw + (s_lo >> 1) : nullptr;
  // X (and the mask words) of tile t of the workgroup's strip i (past the full strips the
  // first one's, not used: gone from the L2 by then, they are 51,200 of the 574,800 128-byte
  // lines fetched at 76800 x 200.  An offset past the resource fetches none of them and takes
  // the same time there, 30.5 us a call for 30.3, but costs k = 25 a register: 57.7 us for 56.2)
  auto load_tile = [&](int i, int t, f4& x, uint32_t& mb) {
    const uint32_t at = i < nfull ? (uint32_t)i * 64u : 0u;
    x = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(xrs, lane_off + (at + t * tile_step), 0, 0));
    if (MASKED) {
      const int last = vcols > 16 * t ? vcols - 16 * t - 1 : 0;  // clamp: a column past the chunk has X = V = 0
      const int ic = i < nst ? i : nst - 1;
      mb = Mw[(int64_t)((c < last ? c : last) + 16 * t) * a.mw + (ic + (int)(s_lo & 1)) / 2];
    }
  };
  f4 x[TW];
  uint32_t mw[TW] = {};
#pragma unroll
  for (int t = 0; t < TW; ++t) {
    x[t] = f4{0.f, 0.f, 0.f, 0.f};
    if (t < nt) load_tile(rq, t, x[t], mw[t]);
  }
  // preconditioned variables: this lane's operands of V' = B W^T (W = pc[0 .. k k))
  float wt[KQ][KB];
#pragma unroll
  for (int q = 0; q < KQ; ++q)
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
      const int t = 4 * q + g, kk = 16 * kb + c;
      wt[q][kb] = 0.f;
      if (pc && kk < k && t < k) wt[q][kb] = pc[kk * k + t];
    }
  __syncthreads();

  double f_acc = 0.0, uu_acc = 0.0, gud_acc = 0.0, gg_acc = 0.0;

  // Everything that holds the wave's tiles in registers, for a wave of NW tiles (nt, or one
  // that is never used if it has none): the tile loops carry no branches; the waves of a workgroup
  // run different instantiations and meet at the same barriers.
  auto run = [&](auto nwc) {
    constexpr int NW = decltype(nwc)::value;
    // ---- V' of this wave's tiles to registers
    // FP32: vr[t][q] = V'[16 t + c][4 q + g], vg[t][kb][q] = V'[16 t + 4 g + q][16 kb + c]
    // (ranks past k: vr is zero; vg's only reach output columns that are dropped)
    float vr[BF16 ? 1 : NW][KQ], vg[BF16 ? 1 : NW][KB][4];
    u4v vrb[BF16 && KB == 1 ? NW : 1][2];   // BF16, k <= 16: hi/lo blocks of eight ranks
    s4 vrs[BF16 && KB == 2 ? NW : 1][KB];   // BF16, k > 16
    s4 vgb[BF16 ? NW : 1][KB];
    const bool have = nt > 0;
#pragma unroll
    for (int t = 0; t < NW; ++t) {
      const float* vt = sV + (have ? 16 * (t0 + t) * ks : 0);  // this tile's rows
      int vst = ks;
      if (pc) {
        // B W^T on MFMA, then through a transpose tile to the operand layouts
        f4 vo[KB];
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) vo[kb] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q < KQ; ++q) {
          const float b = 4 * q + g < k ? vt[c * ks + 4 * q + g] : 0.f;
#pragma unroll
          for (int kb = 0; kb < KB; ++kb) vo[kb] = mfma_f32(b, wt[q][kb], vo[kb]);
        }
        static_assert(NTT * 16 * TS >= 16 * (16 * KB + 1), "a tile of V' fits the transpose tiles");
        vst = 16 * KB + 1;
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
          for (int r = 0; r < 4; ++r) myT[(4 * g + r) * vst + 16 * kb + c] = vo[kb][r];
        vt = myT;
      }
      if constexpr (!BF16) {
#pragma unroll
        for (int q = 0; q < KQ; ++q) {
          const float v = vt[c * vst + 4 * q + g];
          vr[t][q] = have && 4 * q + g < k ? v : 0.f;
        }
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
          for (int q = 0; q < 4; ++q) vg[t][kb][q] = vt[(4 * g + q) * vst + 16 * kb + c];
      } else {
        if constexpr (KB == 1) {
#pragma unroll
          for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int h = 0; h < 4; ++h) {
              const int kk = 8 * j + 2 * h;
              float v0 = vt[c * vst + kk], v1 = vt[c * vst + kk + 1];
              v0 = have && kk < k ? v0 : 0.f;
              v1 = have && kk + 1 < k ? v1 : 0.f;
              const uint32_t hi = pk2(v0, v1);
              const float h0 = __builtin_bit_cast(float, hi << 16), h1 = __builtin_bit_cast(float, hi & 0xFFFF0000u);
              const uint32_t lo = pk2(v0 - h0, v1 - h1);
              vrb[t][j][h] = g == 3 ? 0u : (g == 1 ? lo : hi);
            }
        } else {
#pragma unroll
          for (int kb = 0; kb < KB; ++kb) {
            const int kk = 16 * kb + 4 * g;
            float q4[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float v = vt[c * vst + kk + e];
              q4[e] = have && kk + e < k ? v : 0.f;
            }
            vrs[t][kb] = pack_bf16(q4[0], q4[1], q4[2], q4[3]);
          }
        }
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
          const float* q4 = vt + 4 * g * vst + 16 * kb + c;
          vgb[t][kb] = pack_bf16(q4[0], q4[vst], q4[2 * vst], q4[3 * vst]);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    // BF16: the U rows' ranks past k (never written) are masked off
    uint32_t umask[BF16 ? 4 : 1];
    if constexpr (BF16) {
#pragma unroll
      for (int h = 0; h < 4; ++h) {
        const int kk = KB == 1 ? 8 + 2 * h : 16 + 4 * g + 2 * (h & 1);
        umask[h] = (kk < k ? 0xFFFFu : 0u) | (kk + 1 < k ? 0xFFFF0000u : 0u);
      }
    }
    // G^T U over the strips so far, a strip's products summed by themselves first: in one
    // chain over the strips saturated entries add the same value again and again and round
    // alike.  28 video starts, gV against 64 bits: 5.9e-8 rms (8.8e-8 with groups of three
    // strips, 6.7e-8 in the split by strips), at the same speed (8192 x 8192, k = 25,
    // masked: 165 us for 174 when it was chosen); carrying the additions' rounding along as well gave 5.6e-8 for
    // 8 % more time there
    f4 gvs[NW][KB];
#pragma unroll
    for (int t = 0; t < NW; ++t)
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) gvs[t][kb] = f4{0.f, 0.f, 0.f, 0.f};

    // strip i of the workgroup (strip li of the round in U buffer ubf) against the wave's
    // tiles; strip inx is requested as the registers fall free
    auto strip = [&](int i, int li, int ubf, int inx) {
      if (NW == 1 && nt == 0) {  // no tile: zero sums (zeros times an infinite U or V would not be)
        float* dst = sGU + ((li * cgs + cg) * KB) * 256 + lane * 4;
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) *reinterpret_cast<f4*>(dst + kb * 256) = f4{0.f, 0.f, 0.f, 0.f};
        return;
      }
      if (i >= nfull) {
        // by address: 16 bytes at a time if the strip's rows are all there, else single
        // elements through the transpose tile; the lane index is hidden from the compiler so
        // that this rare path's addresses are not kept across the strips
        int co = c;
        asm volatile("" : "+v"(co));
        const int64_t row0s = (s_lo + i) * 16 + 4 * g;
        if ((s_lo + i + 1) * 16 <= m) {
#pragma unroll
          for (int t = 0; t < NW; ++t) {
            const bool in = 16 * t + co < vcols;
            struct __attribute__((packed, aligned(4))) F4 {
              f4 v;
            };
            const f4 v = reinterpret_cast<const F4*>(Xw + (in ? 16 * t + co : 0) * m + row0s)->v;
            x[t] = in ? v : f4{0.f, 0.f, 0.f, 0.f};
          }
        } else {
#pragma unroll
          for (int t = 0; t < NW; ++t) {
#pragma unroll 1
            for (int q = 0; q < 4; ++q)
              myT[co * TS + 4 * g + q] =
                  row0s + q < m && 16 * t + co < vcols ? Xw[(16 * t + co) * m + row0s + q] : 0.f;
            x[t] = *reinterpret_cast<const f4*>(myT + co * TS + 4 * g);
          }
        }
      }
      const float* us = sU + (ubf * spr + li) * 16 * ks;
      const uint16_t* usb = sUb + (ubf * spr + li) * (2 * UB);
      float ub[KB][4];
      s4 ubb[KB];
      if constexpr (!BF16) {
        float ua[KQ];
#pragma unroll
        for (int q = 0; q < KQ; ++q) ua[q] = us[c * ks + 4 * q + g];
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
          for (int q = 0; q < 4; ++q) ub[kb][q] = us[(4 * g + q) * ks + 16 * kb + c];
#pragma unroll
        for (int q = 0; q < KQ; ++q) {
          ua[q] = 4 * q + g < k ? ua[q] : 0.f;
#pragma unroll
          for (int t = 0; t < NW; ++t) x[t] = mfma_f32(ua[q], vr[t][q], x[t]);
        }
      } else {
        if constexpr (KB == 1) {
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            u4v ua = *reinterpret_cast<const u4v*>(usb + c * 40 + j * 16 + (g == 2 ? 8 : 0));
            if (j == 1)
#pragma unroll
              for (int h = 0; h < 4; ++h) ua[h] &= umask[h];
            else if (k < 8)
#pragma unroll
              for (int h = 0; h < 4; ++h) ua[h] &= (2 * h < k ? 0xFFFFu : 0u) | (2 * h + 1 < k ? 0xFFFF0000u : 0u);
#pragma unroll
            for (int t = 0; t < NW; ++t) x[t] = mfma_bf16x32(ua, vrb[t][j], x[t]);
          }
        } else {
#pragma unroll
          for (int kb = 0; kb < KB; ++kb) {
            u2v ua = *reinterpret_cast<const u2v*>(usb + c * 40 + 16 * kb + 4 * g);
            if (kb == 1) {
              ua[0] &= umask[0];
              ua[1] &= umask[1];
            }
#pragma unroll
            for (int t = 0; t < NW; ++t) x[t] = mfma_bf16(__builtin_bit_cast(s4, ua), vrs[t][kb], x[t]);
          }
        }
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) ubb[kb] = *reinterpret_cast<const s4*>(usb + 640 + kb * 256 + lane * 4);
      }
      f4 gv[NW][KB], gu[KB];
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) {
        gu[kb] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < NW; ++t) gv[t][kb] = f4{0.f, 0.f, 0.f, 0.f};
      }
      float ftile = 0.f, gtile = 0.f;
      const int bsh = 16 * (int)((s_lo + i) & 1) + 4 * g;  // this lane's rows in the mask word
#pragma unroll
      for (int h = 0; h < NW; h += NTT) {
        s4 Gp[NTT];
#pragma unroll
        for (int v = 0; v < NTT; ++v) {
          const int t = h + v;
          if (t >= NW) continue;
          const uint32_t bits = MASKED ? mw[t] >> bsh : 0u;
#pragma unroll
          for (int q = 0; q < 4; ++q)
            x[t][q] = huber<ELASTIC, MASKED>(x[t][q], lam_s, kappa, !MASKED || ((bits >> q) & 1u), ftile, gtile);
          if constexpr (!BF16) {
            float* tT = myT + v * 16 * TS;
#pragma unroll
            for (int q = 0; q < 4; ++q) tT[(4 * g + q) * TS + c] = x[t][q];
          } else {
            const uint32_t p0 = pk2(x[t][0], x[t][1]), p1 = pk2(x[t][2], x[t][3]);
            Gp[v] = __builtin_bit_cast(s4, u2v{p0, p1});
            uint16_t* tT = reinterpret_cast<uint16_t*>(myT + v * 16 * TS);
            tT[(4 * g + 0) * TSB + c] = (uint16_t)p0;
            tT[(4 * g + 1) * TSB + c] = (uint16_t)(p0 >> 16);
            tT[(4 * g + 2) * TSB + c] = (uint16_t)p1;
            tT[(4 * g + 3) * TSB + c] = (uint16_t)(p1 >> 16);
          }
        }
#pragma unroll
        for (int v = 0; v < NTT; ++v) {
          const int t = h + v;
          if (t >= NW) continue;
          if constexpr (!BF16) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
              for (int kb = 0; kb < KB; ++kb) gv[t][kb] = mfma_f32(x[t][q], ub[kb][q], gv[t][kb]);
          } else {
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) gv[t][kb] = mfma_bf16(Gp[v], ubb[kb], gv[t][kb]);
          }
        }
#pragma unroll
        for (int v = 0; v < NTT; ++v)
          if (h + v < NW) load_tile(inx, h + v, x[h + v], mw[h + v]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int v = 0; v < NTT; ++v) {
          const int t = h + v;
          if (t >= NW) continue;
          if constexpr (!BF16) {
            const f4 gt = *reinterpret_cast<const f4*>(myT + v * 16 * TS + c * TS + 4 * g);
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
              for (int kb = 0; kb < KB; ++kb) gu[kb] = mfma_f32(gt[q], vg[t][kb][q], gu[kb]);
          } else {
            const s4 gt = *reinterpret_cast<const s4*>(reinterpret_cast<const uint16_t*>(myT + v * 16 * TS) + c * TSB + 4 * g);
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) gu[kb] = mfma_bf16(gt, vgb[t][kb], gu[kb]);
          }
        }
      }
#pragma unroll
      for (int t = 0; t < NW; ++t)
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) gvs[t][kb] += gv[t][kb];
      // (past the range of FP32 both sums are infinite, and so is the value: not their difference)
      f_acc += ELASTIC || gtile == INFINITY ? (double)ftile : (double)ftile - 0.5 * (double)gtile;
      gg_acc += (double)gtile;
      float* dst = sGU + ((li * cgs + cg) * KB) * 256 + lane * 4;
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) *reinterpret_cast<f4*>(dst + kb * 256) = gu[kb];
    };

    // the rows of a round: G V + lam_L U (or its preconditioned form) and the scalars, a
    // strip per wave in the products' output layout (rows 4 g + q, rank 16 kb + c).  The column
    // groups' sums of a chunk and lam_L U are added in FP32, also where the split by strips has
    // two chunks or more (n > 256; n > 128 above k = 16) and adds those in 64 bits: its chains
    // within a chunk are longer, and gU is closer to 64 bits here -- rms of six inputs, there and
    // here: 5003 x 333, k = 13: 8.6e-8, 5.9e-8; 2000 x 512, k = 10: 1.2e-7, 6.6e-8; 3000 x 300,
    // k = 24: 8.0e-8, 7.9e-8; 4096 x 2048, k = 25: 5.77e-8, 5.75e-8.  In 64 bits it would be 5.3,
    // 6.1, 7.2 and 5.5e-8 for 2 to 10 % more time
    auto finish_round = [&](int i0, int ubf) {
      // (lane indices hidden from the compiler: its addresses are not kept across the strips)
      int c = lane & 15, g = lane >> 4;
      asm volatile("" : "+v"(c), "+v"(g));
      float mt[KQ][KB];  // M_U = pc[k k ..)
#pragma unroll
      for (int q = 0; q < KQ; ++q)
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
          const int t = 4 * q + g, kk = 16 * kb + c;
          mt[q][kb] = pc && kk < k && t < k ? pc[k * k + t * k + kk] : 0.f;
        }
      const int left = nst - i0 < spr ? nst - i0 : spr;
#pragma unroll 1
      for (int li = w; li < left; li += WAVES) {
        const float* us = sU + (ubf * spr + li) * 16 * ks;
        const int64_t r0 = row0 + (i0 + li) * 16;
        const int rows = m - r0 < 16 ? (int)(m - r0) : 16;
        f4 reg[KB];
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) reg[kb] = f4{0.f, 0.f, 0.f, 0.f};
        if (pc) {  // -(A M_U)
#pragma unroll
          for (int q = 0; q < KQ; ++q) {
            float ua = us[c * ks + 4 * q + g];
            ua = 4 * q + g < k ? ua : 0.f;
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) reg[kb] = mfma_f32(ua, mt[q][kb], reg[kb]);
          }
        }
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
          f4 gu = f4{0.f, 0.f, 0.f, 0.f};  // -(G V)
#pragma unroll 4
          for (int q = 0; q < cgs; ++q) gu += *reinterpret_cast<const f4*>(sGU + ((li * cgs + q) * KB + kb) * 256 + lane * 4);
          const int kk = 16 * kb + c;
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int rr = 4 * g + q;
            if (kk >= k || rr >= rows) continue;
            const float u = -us[rr * ks + kk];
            const float rg1 = pc ? -reg[kb][q] : u;
            const int64_t o = (r0 + rr) * k + kk;
            if (a.nchunks == 1) {
              const float gval = fmaf(lam_l, rg1, -gu[q]);
              a.gU[outi][o] = gval;
              if (TRIAL) gud_acc += (double)gval * (double)dU[o];
            } else {
              a.gupart[(int64_t)ch * m * k + o] = -gu[q];
            }
            if (ch == 0) uu_acc += (double)u * (double)rg1;
          }
        }
      }
    };

    // ---- rounds (one, if the strips' sums fit the LDS): strips, barrier, rows
#pragma unroll 1
    for (int i0 = 0, r = 0;; ++r) {
      const int ubf = r & (ubuf - 1);
      const int i1 = i0 + spr;
#pragma unroll 1
      for (int li = rq; li < spr && i0 + li < nst; li += rqs) {
        const int i = i0 + li, nx = li + rqs < spr ? i + rqs : i1 + rq;
        strip(i, li, ubf, nx);
      }
      __syncthreads();
      const bool last = i1 >= nst;
      if (last) {
        if (rq > 0) {  // the row lanes' accumulators: to lane 0 through LDS
#pragma unroll
          for (int t = 0; t < NW; ++t)
#pragma unroll
            for (int kb = 0; kb < KB; ++kb)
              *reinterpret_cast<f4*>(sT + ((((rq - 1) * cgs + cg) * TW + t) * KB + kb) * 256 + lane * 4) = gvs[t][kb];
        }
      }
      finish_round(i0, ubf);
      if (last) break;
      stage_u(r + 1);
      __syncthreads();
      i0 = i1;
    }
    f_acc = wave_sum63(f_acc);
    uu_acc = wave_sum63(uu_acc);
    gud_acc = wave_sum63(gud_acc);
    gg_acc = wave_sum63(gg_acc);
    if (lane == 63) {
      sRed[w] = f_acc;
      sRed[WAVES + w] = uu_acc;
      sRed[2 * WAVES + w] = gud_acc;
      sRed[3 * WAVES + w] = gg_acc;
    }
    __syncthreads();
    if (rq == 0) {  // G^T U of the workgroup's rows, in row lane order
      float* gvp = a.gvpart + (rg * a.n + j_begin + 16 * t0) * k;
#pragma unroll
      for (int t = 0; t < NW; ++t)
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
          f4 s = gvs[t][kb];
          for (int q = 1; q < rqs; ++q)
            s += *reinterpret_cast<const f4*>(sT + ((((q - 1) * cgs + cg) * TW + t) * KB + kb) * 256 + lane * 4);
          const int kk = 16 * kb + c;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int j = 16 * t + 4 * g + r;
            if (kk < k && j < vcols) gvp[j * k + kk] = s[r];
          }
        }
    }
  };
  if (nt == 4) run(std::integral_constant<int, 4>{});
  else if (nt == 3) run(std::integral_constant<int, 3>{});
  else if (nt == 2) run(std::integral_constant<int, 2>{});
  else run(std::integral_constant<int, 1>{});
  if (tid < 4) {
    double v = 0.0;
#pragma unroll
    for (int q = 0; q < WAVES; ++q) v += sRed[tid * WAVES + q];
    a.spart[((int64_t)rg * a.nchunks + ch) * RPCA_NSCAL + tid] = v;
  }
}

// Two waves per SIMD, one workgroup per compute unit: up to 256 registers per wave.
template <int KQ, bool MASKED, bool TRIAL, bool BF16, bool ELASTIC>
__global__ __launch_bounds__(NT, 2) void k_sweep_cols(SweepArgs a) {
  extern __shared__ __align__(16) float lds[];
  __shared__ double sRed[4 * WAVES];
  sweep_item<KQ, MASKED, TRIAL, BF16, ELASTIC>(a, blockIdx.x, blockIdx.y, lds, sRed);
}

// Dynamic LDS of an instance's sweep.
inline int lds_floats(const SweepArgs& a, bool bf16) {
  const int spr = bf16 ? a.spr_bf16 : a.spr;
  return sweep_lds(a.k, a.chunk_w, 1 << a.lcg, bf16, spr, a.sdiv + (a.srem ? 1 : 0) > spr ? 2 : 1).total;
}

// Residual steps of a rank class: k <= 12, 16, 24, 28, 32.  (Classes of two and five steps,
// k <= 8 and k <= 20, would take 3 to 5 % off their FP32 evaluations -- 76800 x 200, k = 8: 29.6
// us a call to 28.4, k = 20: 47.5 to 46.1; BF16 the same -- for two more kernels to each three.)
__host__ __device__ constexpr int kq_class(int k) { return k <= 12 ? 3 : k <= 16 ? 4 : k <= 24 ? 6 : k <= 28 ? 7 : 8; }

template <bool MASKED, bool TRIAL, bool BF16, bool ELASTIC = false>
hipError_t launch_cols(const SweepArgs& sa, hipStream_t s) {
  if (sa.k < 1 || sa.k > 32 || sa.chunk_w < 16 || sa.chunk_w % 16 || sa.chunk_w > CHUNK_MAX) return hipErrorInvalidValue;
  const int lds = lds_floats(sa, BF16);
  if (lds > LDS_LIMIT_FLOATS) return hipErrorInvalidValue;
  const dim3 grid(sa.row_groups, sa.nchunks), block(NT);
  const size_t bytes = lds * sizeof(float);
  switch (kq_class(sa.k)) {
    case 3: hipLaunchKernelGGL((k_sweep_cols<3, MASKED, TRIAL, BF16, ELASTIC>), grid, block, bytes, s, sa); break;
    case 4: hipLaunchKernelGGL((k_sweep_cols<4, MASKED, TRIAL, BF16, ELASTIC>), grid, block, bytes, s, sa); break;
    case 6: hipLaunchKernelGGL((k_sweep_cols<6, MASKED, TRIAL, BF16, ELASTIC>), grid, block, bytes, s, sa); break;
    case 7: hipLaunchKernelGGL((k_sweep_cols<7, MASKED, TRIAL, BF16, ELASTIC>), grid, block, bytes, s, sa); break;
    default: hipLaunchKernelGGL((k_sweep_cols<8, MASKED, TRIAL, BF16, ELASTIC>), grid, block, bytes, s, sa); break;
  }
  return hipGetLastError();
}

}  // namespace rpca_cols
