// Objective/gradient without any allocation: rpca_objgrad_noalloc runs the
// same fused sweep and finishing reduction as rpca_objgrad, with every partial
// sum in one library-owned device array instead of a context's workspace.
//
// The array below lives in the device code object, so each GPU the library runs
// on holds its own copy until the process ends.  Its name is only a host-side
// stand-in: host code resolves the device address once per device with
// hipGetSymbolAddress and passes that address to the kernels.
#include <math.h>
#include <string.h>

#include <algorithm>
#include <mutex>

#include "rpca_internal.h"

namespace {

constexpr size_t SCRATCH_BYTES = (size_t)RPCA_NOALLOC_SCRATCH_MB << 20;
constexpr int MAX_DEVICES = 64;

static __device__ __align__(256) unsigned char scratch[SCRATCH_BYTES];

std::mutex g_mu;
void* g_addr[MAX_DEVICES] = {nullptr};

// Device address of this GPU's copy of the array (resolved on first use).
hipError_t scratch_address(void** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= MAX_DEVICES) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_mu);
  if (!g_addr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_addr[dev] = p;
  }
  *out = g_addr[dev];
  return hipSuccess;
}

size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

// Scratch layout of one call (byte offsets; every region 256-byte aligned).
struct Layout {
  size_t counters, spart, fpart, gvpart, gupart, total;
};

Layout layout_for(int64_t m, int64_t n, int k, int row_groups, int nchunks, int sweep_wgs) {
  Layout L;
  size_t o = 0;
  L.counters = o;
  o += align256(16 * sizeof(unsigned));
  L.spart = o;
  o += align256((size_t)sweep_wgs * RPCA_NSCAL * sizeof(double));
  L.fpart = o;
  o += align256((size_t)rpca::finish_blocks(m, n, k, nchunks, row_groups, nullptr) * 4 * sizeof(double));
  L.gvpart = o;
  o += align256((size_t)row_groups * n * k * sizeof(float));
  L.gupart = o;
  if (nchunks > 1) o += align256((size_t)nchunks * m * k * sizeof(float));
  L.total = o;
  return L;
}

// Whether an instance's size is accepted: the documented limit, which counts the partials
// of the split by strips at its default entries, sums of
// 16 of them in 64 bits, and the scalars of their reduction in blocks of 256 threads.  The
// split in use has wider chunks and needs less; the limit stays where callers rely on it,
// whatever the tuning table holds.
bool within_limit(int64_t m, int64_t n, int k) {
  int rows = 0, spw = 0, cw = 0, nch = 0;
  const rpca::SweepTune t = rpca::tune_default(rpca::TUNE_STRIPS, rpca::tune_k_bucket(k), rpca::tune_n_bucket(n));
  const int wgs = rpca::strip_blocks_for(m, n, k, &rows, &spw, &cw, &nch, t);
  const int64_t vrows = 256 / k, ublocks = nch > 1 ? std::min<int64_t>((m * k + 255) / 256, 4096) : 0;
  const size_t blocks = (size_t)((n + vrows - 1) / vrows + ublocks);
  size_t o = align256(16 * sizeof(unsigned)) + align256((size_t)wgs * RPCA_NSCAL * sizeof(double)) +
             align256((blocks * 3 + 16) * sizeof(double)) + align256((size_t)((rows + 15) / 16) * n * k * sizeof(double)) +
             align256((size_t)rows * n * k * sizeof(float));
  if (nch > 1) o += align256((size_t)nch * m * k * sizeof(float));
  return o <= SCRATCH_BYTES;
}

}  // namespace

extern "C" int rpca_objgrad_noalloc(int64_t m, int64_t n, int32_t k, double lam_s, double lam_l,
                                    const uint32_t* mask_bits, const float* X, const float* U, const float* V,
                                    double* f, float* gU, float* gV, void* stream) {
  // the same argument rules as rpca_create + rpca_objgrad
  if (m < 1 || n < 1 || k < 1 || k > 32 || k > m || k > n) return RPCA_EINVAL;
  if (!(lam_s > 0) || !(lam_l > 0) || !isfinite(lam_s) || !isfinite(lam_l)) return RPCA_EINVAL;
  if (m > (int64_t)1 << 31 || n > (int64_t)1 << 24) return RPCA_EINVAL;
  if (!X || !U || !V || !f || !gU || !gV) return RPCA_EINVAL;
  if (!within_limit(m, n, k)) return RPCA_ETOOBIG;
  // the decomposition rpca_create would choose for this instance, or the default one if the
  // tuning table's takes more than the array
  int row_groups = 0, spw = 0, chunk_w = 0, nchunks = 0;
  int sweep_wgs = rpca::sweep_blocks_for(m, n, k, &row_groups, &spw, &chunk_w, &nchunks, 0);
  Layout L = layout_for(m, n, k, row_groups, nchunks, sweep_wgs);
  if (L.total > SCRATCH_BYTES) {
    const rpca::SweepTune t = rpca::tune_default(rpca::TUNE_COLS, rpca::tune_k_bucket(k), rpca::tune_n_bucket(n));
    sweep_wgs = rpca::col_blocks_for(m, n, k, &row_groups, &spw, &chunk_w, &nchunks, t);
    L = layout_for(m, n, k, row_groups, nchunks, sweep_wgs);
    if (L.total > SCRATCH_BYTES) return RPCA_ETOOBIG;
  }

  void* base = nullptr;
  if (scratch_address(&base) != hipSuccess) return RPCA_EHIP;
  unsigned char* b = static_cast<unsigned char*>(base);

  SweepArgs sa;
  memset(&sa, 0, sizeof(sa));
  sa.X = X;
  sa.mask = mask_bits;
  sa.m = m;
  sa.n = n;
  sa.k = k;
  sa.mw = mask_bits ? (int)((m + 31) / 32) : 0;
  sa.lam_s = (float)lam_s;
  sa.lam_l = (float)lam_l;
  sa.kappa = 0.f;
  sa.U[0] = sa.U[1] = U;
  sa.V[0] = sa.V[1] = V;
  sa.gU[0] = sa.gU[1] = gU;
  sa.gupart = nchunks > 1 ? reinterpret_cast<float*>(b + L.gupart) : nullptr;
  sa.gvpart = reinterpret_cast<float*>(b + L.gvpart);
  sa.spart = reinterpret_cast<double*>(b + L.spart);
  sa.chunk_w = chunk_w;
  sa.nchunks = nchunks;
  sa.row_groups = row_groups;
  rpca::sweep_split(&sa);
  // the array is shared: the sweep zeroes the counter, whatever an earlier call left there
  sa.arm = reinterpret_cast<unsigned*>(b + L.counters);

  FinishArgs fa;
  memset(&fa, 0, sizeof(fa));
  fa.m = m;
  fa.n = n;
  fa.k = k;
  fa.lam_l = (float)lam_l;
  fa.U[0] = fa.U[1] = U;
  fa.V[0] = fa.V[1] = V;
  fa.gU[0] = fa.gU[1] = gU;
  fa.gV[0] = fa.gV[1] = gV;
  fa.gupart = sa.gupart;
  fa.gvpart = sa.gvpart;
  fa.spart = sa.spart;
  fa.fpart = reinterpret_cast<double*>(b + L.fpart);
  fa.counter = reinterpret_cast<unsigned*>(b + L.counters);
  fa.f_out = f;
  fa.nchunks = nchunks;
  fa.row_groups = row_groups;
  fa.sweep_wgs = sweep_wgs;
  if (rpca::launch_objgrad(sa, fa, false, false, (hipStream_t)stream) != hipSuccess) return RPCA_EHIP;
  return RPCA_OK;
}
