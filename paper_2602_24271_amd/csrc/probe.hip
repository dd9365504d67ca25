// Measurement kernels (not on the evaluation path): the chip-wide ceiling of
// the exact FP64 modular product, FP64 FMAs on the VALU and the matrix cores
// at once, and one residue-base conversion (17 -> 18 or 18 -> 17 primes)
// computed two ways, split-FMA rows on the VALU (conv_row) and the library's
// integer matrix-core form (conv_pack, conv_tile, conv_value), timed and
// compared residue for residue.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstring>
#include <string>
#include <vector>

#include "../../include/nshe_probe.h"
#include "conv.h"

namespace nshe {

// ------------------------------------------------------ modular ceiling ---

// Eight independent chains of dependent lazy modular products per thread.
__global__ void __launch_bounds__(256) k_probe_modmul(double* out, int iters, double p,
                                                      double pinv, double w) {
  const size_t gid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  double x[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) x[c] = (double)((gid * 8 + c) % 1000003) + 1.0;
  for (int it = 0; it < iters; ++it) {
#pragma unroll
    for (int c = 0; c < 8; ++c) x[c] = mul_lazy(x[c], w, p, pinv);
  }
  double s = 0.0;
#pragma unroll
  for (int c = 0; c < 8; ++c) s += x[c];
  out[gid] = s;
}

// -------------------------------------------------- FP64 MFMA overlap ---

typedef double v4d __attribute__((ext_vector_type(4)));

// MODE 0: 64 FP64 FMAs per lane and iteration (eight chains); 1: four
// independent 16x16x4 FP64 MFMAs per wave and iteration (4096 FMAs per
// wave, 64 per lane); 2: both.
template <int MODE>
__global__ void __launch_bounds__(256) k_probe_overlap(double* out, int iters, double seed) {
  const size_t gid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const double a = seed + (double)threadIdx.x, b = 1.0 + 1e-9 * (double)threadIdx.x;
  double v[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) v[c] = a + c;
  v4d acc[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) acc[c] = v4d{0.0, 0.0, 0.0, 0.0};
  for (int it = 0; it < iters; ++it) {
    if constexpr (MODE != 0) {
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc[c], 0, 0, 0);
    }
    if constexpr (MODE != 1) {
#pragma unroll
      for (int r = 0; r < 8; ++r)
#pragma unroll
        for (int c = 0; c < 8; ++c) v[c] = __builtin_fma(v[c], b, 1e-300);
    }
  }
  double s = 0.0;
#pragma unroll
  for (int c = 0; c < 8; ++c) s += v[c];
#pragma unroll
  for (int c = 0; c < 4; ++c) s += acc[c][0] + acc[c][1] + acc[c][2] + acc[c][3];
  out[gid] = s;
}

// ------------------------------------------------------- conversion ---

// Balanced pseudo-random residues: v[r][c] for row r (prime m[r]).
__global__ void __launch_bounds__(256) k_probe_fill(double* v, size_t n, int rows,
                                                    const double* m, uint64_t seed) {
  const size_t gid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= n * rows) return;
  uint64_t z = seed + gid * 0x9e3779b97f4a7c15ull;
  z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
  z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
  z ^= z >> 31;
  const double p = m[gid / n];
  const double u = (double)(z >> 15);        // < 2^49
  const double r = u - p * __builtin_floor(u / p);
  v[gid] = r > 0.5 * p ? r - p : r;
}

// The split-FMA row on the FP64 VALU: sum_j y_j M_j (mod m) over NT <= 25 terms with four
// FMAs per term instead of a modular product.  Each input (a reduced
// residue, |y| <= 2^48) is split once as y = yh 2^24 + yl (|yh| <= 2^24,
// |yl| <= 2^23) and each constant is stored split the same way, M = c1 2^24
// + c0 (|c1| <= 2^24, |c0| <= 2^23).  Then
//   y M = yh c1 2^48 + (yh c0 + yl c1) 2^24 + yl c0,
// so the row is W48 [2^48]_m + W24 [2^24]_m + W0 (mod m) with W48 = sum yh
// c1, W24 = sum yh c0 + yl c1 and W0 = sum yl c0.  Every product is an
// integer of at most 2^48, so exact, and so is every partial sum (|W48|,
// |W24| <= NT 2^48 < 2^53, |W0| <= NT 2^46).  Every prime lies in
// (2^48, 2^49), so [2^24]_m = 2^24 and [2^48]_m = 2^48: T48 = W48 2^48 and
// T24 = W24 2^24 are exact doubles (exponent shifts), and each is reduced
// exactly by one FMA, T - q m with q = rint(T fl(1/m)): the true difference
// is an integer below 1.5 m for NT <= 16 (below 2.5 m for NT <= 25: the
// quotient estimate is within 2 of T / m <= 2^53), so exactly
// representable, and the FMA returns it.  The result is returned
// unreduced, |result| <= (NT / 4 + 7.2) 2^48.
constexpr int CONV_SPLIT_MAX = 25;
constexpr int CONV_CHUNK = 9;

// sp: the row's constants {c1, c0} per term; m in (2^48, 2^49), minv =
// fl(1/m).
template <int NT>
__device__ __forceinline__ double conv_row(const double (&yh)[NT], const double (&yl)[NT],
                                           const double* sp, double m, double minv) {
  static_assert(NT <= CONV_SPLIT_MAX, "partial sums must stay below 2^53");
  double w48 = 0.0, w24a = 0.0, w24b = 0.0, w0 = 0.0;
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    // constants are fetched CONV_CHUNK terms at a time: the row pointer is
    // made to depend on the running sums, so later terms' scalar loads are
    // not all hoisted to the row's start (which spills scalar registers)
    if (j && j % CONV_CHUNK == 0) asm volatile("" : "+s"(sp) : "v"(w0));
    const double c1 = cld(sp, 2 * j), c0 = cld(sp, 2 * j + 1);
    w48 = __builtin_fma(yh[j], c1, w48);
    w24a = __builtin_fma(yh[j], c0, w24a);
    w24b = __builtin_fma(yl[j], c1, w24b);
    w0 = __builtin_fma(yl[j], c0, w0);
  }
  // (ldexp: exponents 48 and 24 are inline operands; a 2^48 multiplier
  // would hold a register pair through the row loops)
  const double t48 = __builtin_ldexp(w48, 48), t24 = __builtin_ldexp(w24a + w24b, 24);
  const double r48 = __builtin_fma(-__builtin_rint(t48 * minv), m, t48);
  const double r24 = __builtin_fma(-__builtin_rint(t24 * minv), m, t24);
  return r48 + r24 + w0;
}

template <int NT, int NO>
__global__ void __launch_bounds__(256) k_conv_fma(size_t n, const double* __restrict__ y,
                                                  double* __restrict__ out,
                                                  const double* sp, const double* m,
                                                  const double* minv) {
  const size_t c = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= n) return;
  double yh[NT], yl[NT];
#pragma unroll
  for (int i = 0; i < NT; ++i) split24(y[(size_t)i * n + c], yh[i], yl[i]);
#pragma unroll
  for (int k = 0; k < NO; ++k) {
    const int kq = opaque_idx(k);
    const double mk = cld(m, kq), mi = cld(minv, kq);
    const double* row = opaque_row(sp, kq * NT * 2);
    const double a = conv_row<NT>(yh, yl, row, mk, mi);
    out[(size_t)k * n + c] = reduce_bal(a, mk, mi);
  }
}

// One coefficient per lane, as the library's per-coefficient kernels.
template <int NT, int NO>
__global__ void __launch_bounds__(256) k_conv_mfma(size_t n, const double* __restrict__ y,
                                                   double* __restrict__ out, const double* tab,
                                                   const double* m, const double* minv) {
  __shared__ v4i lt[conv_entries(NT, NO)];
  conv_table<conv_entries(NT, NO)>(lt, tab);
  __syncthreads();
  const size_t nb = (n + blockDim.x - 1) / blockDim.x;
  for (size_t bk = blockIdx.x; bk < nb; bk += gridDim.x) {
    const size_t gid = bk * blockDim.x + threadIdx.x;
    const bool ok = gid < n;
    const size_t c = ok ? gid : 0;
    double in[conv_steps(NT) * 4];
#pragma unroll
    for (int i = 0; i < conv_steps(NT) * 4; ++i) in[i] = i < NT ? y[(size_t)i * n + c] : 0.0;
    loads_issued();
    v4i g0[conv_steps(NT)], g1[conv_steps(NT)];
#pragma unroll
    for (int s = 0; s < conv_steps(NT); ++s) {
      const double q[4] = {in[4 * s], in[4 * s + 1], in[4 * s + 2], in[4 * s + 3]};
      conv_pack(q, NT - 4 * s, g0[s], g1[s]);
    }
#pragma unroll
    for (int t = 0; t < conv_tiles(NO); ++t) {
      ConvSum cs[4];
      conv_tile<NT>(lt + t * conv_steps(NT) * 64, g0, g1, cs);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int k = 4 * t + j;
        if (k >= NO) continue;
        const int kq = opaque_idx(k);
        const double mk = cld(m, kq), mi = cld(minv, kq);
        const double r = reduce_bal(conv_value<NT>(cs[j], mk, mi), mk, mi);
        if (ok) out[(size_t)k * n + c] = r;
      }
    }
  }
}

// Residues of a and b (balanced or within p/2 + 4) that differ mod m[row].
__global__ void __launch_bounds__(256) k_probe_compare(const double* a, const double* b,
                                                       size_t n, int rows, const double* m,
                                                       unsigned long long* bad) {
  const size_t gid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= n * rows) return;
  const double p = m[gid / n];
  if (to_canonical(a[gid], p) != to_canonical(b[gid], p)) atomicAdd(bad, 1ull);
}

}  // namespace nshe

using namespace nshe;

namespace {

thread_local std::string g_probe_err;

int probe_fail(const std::string& msg) {
  g_probe_err = msg;
  return -4;
}

#define PCHK(expr)                                                                   \
  do {                                                                               \
    hipError_t e_ = (expr);                                                          \
    if (e_ != hipSuccess) return probe_fail(std::string(#expr ": ") + hipGetErrorString(e_)); \
  } while (0)

double bal(uint64_t x, uint64_t m) { return x > m / 2 ? (double)x - (double)m : (double)x; }

struct DevBuf {
  void* p = nullptr;
  ~DevBuf() { if (p) (void)hipFree(p); }
};

template <int NT, int NO>
int run_conversion(const uint64_t* qin, const uint64_t* qout, size_t n, int reps,
                   nshe_conv_probe* res) {
  // constants: M_ik uniform-looking, canonical mod qout[k]
  std::vector<uint64_t> M((size_t)NT * NO);
  uint64_t z = 0x1234567ull;
  for (int i = 0; i < NT; ++i)
    for (int k = 0; k < NO; ++k) {
      z = z * 6364136223846793005ull + 1442695040888963407ull;
      const uint64_t mk = qout[k];
      M[(size_t)i * NO + k] = (z >> 11) % mk;
    }
  std::vector<double> sp((size_t)NO * NT * 2), mo(NO), mi(NO), mq(NT);
  for (int k = 0; k < NO; ++k) {
    const uint64_t mk = qout[k];
    mo[k] = (double)mk;
    mi[k] = 1.0 / (double)mk;
    for (int i = 0; i < NT; ++i) {
      const double cb = bal(M[(size_t)i * NO + k], mk);
      const double c1 = __builtin_nearbyint(cb * 0x1p-24);
      sp[((size_t)k * NT + i) * 2] = c1;
      sp[((size_t)k * NT + i) * 2 + 1] = cb - c1 * 0x1p24;
    }
  }
  for (int i = 0; i < NT; ++i) mq[i] = (double)qin[i];
  const std::vector<int32_t> at = conv_matrix(M, NT, std::vector<uint64_t>(qout, qout + NO));
  DevBuf dy, dof, dom, dtab, dbad;
  const size_t tab_doubles = sp.size() + 2 * (size_t)NO + NT;
  PCHK(hipMalloc(&dy.p, (size_t)NT * n * 8));
  PCHK(hipMalloc(&dof.p, (size_t)NO * n * 8));
  PCHK(hipMalloc(&dom.p, (size_t)NO * n * 8));
  PCHK(hipMalloc(&dtab.p, tab_doubles * 8 + at.size() * 4 + 256));
  PCHK(hipMalloc(&dbad.p, 8));
  double* tb = static_cast<double*>(dtab.p);
  double *d_sp = tb, *d_m = d_sp + sp.size(), *d_mi = d_m + NO, *d_mq = d_mi + NO;
  double* d_at = reinterpret_cast<double*>(reinterpret_cast<char*>(dtab.p) +
                                           ((tab_doubles * 8 + 255) & ~(size_t)255));
  PCHK(hipMemcpy(d_sp, sp.data(), sp.size() * 8, hipMemcpyHostToDevice));
  PCHK(hipMemcpy(d_m, mo.data(), NO * 8, hipMemcpyHostToDevice));
  PCHK(hipMemcpy(d_mi, mi.data(), NO * 8, hipMemcpyHostToDevice));
  PCHK(hipMemcpy(d_mq, mq.data(), NT * 8, hipMemcpyHostToDevice));
  PCHK(hipMemcpy(d_at, at.data(), at.size() * 4, hipMemcpyHostToDevice));
  PCHK(hipMemset(dbad.p, 0, 8));
  double* y = static_cast<double*>(dy.p);
  double* of = static_cast<double*>(dof.p);
  double* om = static_cast<double*>(dom.p);
  const dim3 blk(256);
  hipLaunchKernelGGL(k_probe_fill, dim3((unsigned)((NT * n + 255) / 256)), blk, 0, 0, y, n, NT,
                     d_mq, 42ull);
  PCHK(hipGetLastError());
  const size_t nb = (n + 255) / 256;
  const dim3 gf((unsigned)nb), gm((unsigned)(nb < 4096 ? nb : 4096));
  hipEvent_t e0, e1;
  PCHK(hipEventCreate(&e0));
  PCHK(hipEventCreate(&e1));
  float ms_f = 0.f, ms_m = 0.f;
  for (int pass = 0; pass < 2; ++pass) {   // pass 0 warms up
    PCHK(hipEventRecord(e0, 0));
    for (int r = 0; r < reps; ++r)
      hipLaunchKernelGGL((k_conv_fma<NT, NO>), gf, blk, 0, 0, n, y, of, d_sp, d_m, d_mi);
    PCHK(hipEventRecord(e1, 0));
    PCHK(hipEventSynchronize(e1));
    PCHK(hipEventElapsedTime(&ms_f, e0, e1));
    PCHK(hipEventRecord(e0, 0));
    for (int r = 0; r < reps; ++r)
      hipLaunchKernelGGL((k_conv_mfma<NT, NO>), gm, blk, 0, 0, n, y, om, d_at, d_m, d_mi);
    PCHK(hipEventRecord(e1, 0));
    PCHK(hipEventSynchronize(e1));
    PCHK(hipEventElapsedTime(&ms_m, e0, e1));
  }
  hipLaunchKernelGGL(k_probe_compare, dim3((unsigned)((NO * n + 255) / 256)), blk, 0, 0, of, om, n,
                     NO, d_m, static_cast<unsigned long long*>(dbad.p));
  PCHK(hipGetLastError());
  unsigned long long bad = 0;
  PCHK(hipMemcpy(&bad, dbad.p, 8, hipMemcpyDeviceToHost));
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  res->coefficients = n;
  res->ms_fma = ms_f / reps;
  res->ms_mfma = ms_m / reps;
  res->mismatches = bad;
  return 0;
}

}  // namespace

extern "C" {

const char* nshe_probe_last_error(void) { return g_probe_err.c_str(); }

int nshe_probe_modmul(int hip_device, int iters, nshe_modmul_probe* out) {
  if (!out || iters < 1) return probe_fail("bad argument");
  PCHK(hipSetDevice(hip_device));
  const uint64_t p = 562949953421231ull;  // any odd p < 2^49 (rounding-quotient product)
  const int blocks = 256 * 16, threads = 256;
  DevBuf buf;
  PCHK(hipMalloc(&buf.p, (size_t)blocks * threads * 8));
  double* o = static_cast<double*>(buf.p);
  const double pd = (double)p, pinv = 1.0 / pd, w = bal(0x123456789abull % p, p);
  hipEvent_t e0, e1;
  PCHK(hipEventCreate(&e0));
  PCHK(hipEventCreate(&e1));
  float ms = 0.f;
  for (int pass = 0; pass < 2; ++pass) {
    PCHK(hipEventRecord(e0, 0));
    hipLaunchKernelGGL(k_probe_modmul, dim3(blocks), dim3(threads), 0, 0, o, iters, pd, pinv, w);
    PCHK(hipEventRecord(e1, 0));
    PCHK(hipEventSynchronize(e1));
    PCHK(hipEventElapsedTime(&ms, e0, e1));
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  const double products = (double)blocks * threads * 8 * iters;
  out->ms = ms;
  out->products_per_s = products / (ms * 1e-3);
  out->fp64_ops_per_s = out->products_per_s * 6.0;
  return 0;
}

int nshe_probe_fp64_overlap(int hip_device, int iters, nshe_overlap_probe* out) {
  if (!out || iters < 1) return probe_fail("bad argument");
  PCHK(hipSetDevice(hip_device));
  const int blocks = 256 * 16, threads = 256;
  DevBuf buf;
  PCHK(hipMalloc(&buf.p, (size_t)blocks * threads * 8));
  double* o = static_cast<double*>(buf.p);
  hipEvent_t e0, e1;
  PCHK(hipEventCreate(&e0));
  PCHK(hipEventCreate(&e1));
  float ms[3] = {0.f, 0.f, 0.f};
  for (int mode = 0; mode < 3; ++mode) {
    for (int pass = 0; pass < 2; ++pass) {
      PCHK(hipEventRecord(e0, 0));
      if (mode == 0)
        hipLaunchKernelGGL(k_probe_overlap<0>, dim3(blocks), dim3(threads), 0, 0, o, iters, 1.0);
      else if (mode == 1)
        hipLaunchKernelGGL(k_probe_overlap<1>, dim3(blocks), dim3(threads), 0, 0, o, iters, 1.0);
      else
        hipLaunchKernelGGL(k_probe_overlap<2>, dim3(blocks), dim3(threads), 0, 0, o, iters, 1.0);
      PCHK(hipGetLastError());
      PCHK(hipEventRecord(e1, 0));
      PCHK(hipEventSynchronize(e1));
      PCHK(hipEventElapsedTime(&ms[mode], e0, e1));
    }
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  const double fmas = (double)blocks * threads * 64 * iters;
  out->ms_valu = ms[0];
  out->ms_mfma = ms[1];
  out->ms_both = ms[2];
  out->fma_per_s_valu = fmas / (ms[0] * 1e-3);
  out->fma_per_s_mfma = fmas / (ms[1] * 1e-3);
  return 0;
}

int nshe_probe_conversion(int hip_device, const uint64_t* in_primes, int n_in,
                          const uint64_t* out_primes, int n_out, size_t n_coef, int reps,
                          nshe_conv_probe* out) {
  if (!in_primes || !out_primes || !out || n_coef == 0 || reps < 1)
    return probe_fail("bad argument");
  PCHK(hipSetDevice(hip_device));
  if (n_in == 17 && n_out == 18) return run_conversion<17, 18>(in_primes, out_primes, n_coef, reps, out);
  if (n_in == 18 && n_out == 17) return run_conversion<18, 17>(in_primes, out_primes, n_coef, reps, out);
  return probe_fail("supported shapes: 17 -> 18 and 18 -> 17 primes");
}

}  // extern "C"
