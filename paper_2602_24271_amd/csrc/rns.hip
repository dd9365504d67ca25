// Per-coefficient residue-number-system kernels: exact centred lifts between
// the data basis Q = {q_i} and the extension basis B = {b_k}, the BFV
// scale-and-round, key-switch accumulation and mod-down, and the
// conversions at the library boundary.
//
// Exact centred lift (used by the product's operand lift and by the
// scale-and-round): for residues x_i of X in [0, Q), let
// y_i = [x_i (Q/q_i)^-1]_{q_i} (balanced) and S = sum_i y_i / q_i.  Then
// sum_i y_i (Q/q_i) = X + kQ with k = S - X/Q an integer, so the centred
// representative of X is sum_i y_i (Q/q_i) - rint(S) Q.  S is evaluated in
// double precision with absolute error below 2^-45 (L <= 24 terms of
// magnitude < 1/2); when S lies within 2^-40 of a half-integer the rounding
// decision is taken exactly instead: floor(S) = k, and X > (Q-1)/2 is
// decided by comparing mixed-radix digits of X with those of (Q-1)/2
// (Garner's algorithm).  Each such event is counted, per call site
// (MarginSite).  The window is a context setting (tb.lift_edge = 1/2 - 2^-40
// by default); a debug setting widens it to 1/4, which leaves floor(S)
// exact (S is then at least 1/4 from an integer) and sends about half of
// all coefficients through the exact path.
//
// Scale and round (BFV multiply): for d in Q u B (|d| < QB/2), the exact
// r = [t d]_Q (centred) gives y = (t d - r) / Q = round(t d / Q) exactly.
// In base B: [y]_{b_k} = [t Q^-1 d_k - sum_i y_i q_i^-1 + v]_{b_k} where
// y_i, v are the lift quantities of r; then y is lifted from B to Q (|y| <
// t N Q / 2 < B / 32, so that lift's estimate is never near a half-integer;
// a violation would be counted in `fault`).
//
// The sums over the other basis (sum_i y_i [Q/q_i]_{b_k} and the like) are
// matrix products mod b_k; they run on the integer matrix cores over signed
// bytes (conv_pack, conv_tile) with one modular reduction per output.
#include <algorithm>
#include <type_traits>

#include "conv.h"
#include "kernels.h"

namespace nshe {


// Whether the lift takes its exact decision: S within 2^-40 of a
// half-integer, or within 1/4 under the debug switch (tb.lift_edge < 1/2 -
// 2^-40, a uniform flag: the default window stays a literal, which keeps the
// kernels' register counts).
__device__ __forceinline__ bool lift_near_half(double S, double v, const Tables& tb) {
  const double d = __builtin_fabs(S - v);
  return d > 0.5 - 0x1p-40 || (tb.lift_edge < 0.5 - 0x1p-40 && d > tb.lift_edge);
}

// Garner mixed-radix digits of X (canonical residues r, basis q_0..q_{L-1})
// compared with those of (Q-1)/2: returns X > (Q-1)/2.
// (Arguments by value: taking the address of the kernel's Tables argument
// would copy it to scratch memory in every thread.  A rare fallback: its
// loops stay rolled and its digits in private memory, so that it does not
// raise the register count - and lower the occupancy - of its callers.)
template <int L>
__device__ __noinline__ bool mrc_greater_than_half(const double* r, const double* __restrict__ P,
                                                   const double* __restrict__ Pinv,
                                                   const double* __restrict__ inv,
                                                   const double* __restrict__ half) {
  double a[L];
#pragma unroll 1
  for (int i = 0; i < L; ++i) {
    const double p = P[i], pinv = Pinv[i];
    double t = r[i];
#pragma unroll 1
    for (int j = 0; j < i; ++j) {
      t = mul_bal(t - a[j], inv[j * L + i], p, pinv);
      t = to_canonical(t, p);
    }
    a[i] = t;
  }
#pragma unroll 1
  for (int i = L - 1; i >= 0; --i) {
    const double h = half[i];
    if (a[i] != h) return a[i] > h;
  }
  return false;
}

// Per-poly block mapping of the per-coefficient kernels: block b covers
// coefficients [(b mod bpp) blockDim, ...) of poly b / bpp, so the poly and
// its base address are uniform (scalar registers): limb accesses are buffer
// loads with one per-lane offset and a scalar limb offset.  A workgroup takes
// blocks b, b + gridDim, ... (the conversion constants it holds in LDS serve
// them all).  Every lane of a wave takes part in the conversions (matrix
// instructions and lane swaps), also those past the last coefficient of a
// ring smaller than the block: they repeat coefficient 0 and store nothing
// (ok).
struct PolyBlock {
  size_t pc;
  int c;
  bool ok;
};

__device__ __forceinline__ unsigned poly_blocks(int n, size_t n_poly) {
  return (unsigned)(n_poly * (size_t)((n + (int)blockDim.x - 1) / (int)blockDim.x));
}

__device__ __forceinline__ PolyBlock poly_block(int n, unsigned b) {
  const unsigned bpp = (unsigned)((n + (int)blockDim.x - 1) / (int)blockDim.x);
  const size_t pc = b / bpp;
  const int c = (int)(b - pc * bpp) * (int)blockDim.x + (int)threadIdx.x;
  return PolyBlock{pc, c < n ? c : 0, c < n};
}

// ------------------------------------------------------------------ lift ---

// A store of a lane that has a coefficient; the others' offset is past every
// buffer, where stores are dropped.
__device__ __forceinline__ unsigned store_off(bool ok, unsigned off) {
  return ok ? off : 0x7ffffff8u;
}

// The constants of primes 4s..4s+3 of a basis, four doubles each (kq, kb): a
// few wide scalar loads, fenced per step so that no later step's are held
// through it.  (Steps past the last prime read the table's padding.)
__device__ __forceinline__ const double* step_consts(const double* tab, int s) {
  return opaque_row(tab, 16 * s);
}

// Touches every cache line of a table of n doubles, together: a kernel's
// scalar caches start cold, and the steps' loads would otherwise miss one after
// the other (about half a microsecond each).
template <int N>
__device__ __forceinline__ void touch_lines(const double* tab) {
  constexpr int LINES = (N + 7) / 8;
  int v[(LINES + 7) / 8 * 8];
#pragma unroll
  for (int i = 0; i < (LINES + 7) / 8 * 8; ++i)
    v[i] = cldi(reinterpret_cast<const int*>(tab), i < LINES ? 16 * i : 0);
#pragma unroll
  for (int i = 0; i < LINES; i += 8)
    asm volatile("" ::"s"(v[i]), "s"(v[i + 1]), "s"(v[i + 2]), "s"(v[i + 3]), "s"(v[i + 4]),
                 "s"(v[i + 5]), "s"(v[i + 6]), "s"(v[i + 7]));
}

// A lift kernel's LDS copy of the conversion constants, made behind the first
// block's loads (mod-down + lift of eight ciphertexts 52 us, 56 before them;
// the scale-and-round, with twice the limbs and constants, fills its tables
// first: behind the loads its barrier holds every wave until all of the
// workgroup's limbs are in, 83 us against 66).
template <int L>
__device__ __forceinline__ void lift_setup(v4i* tab, const Tables& tb, bool& first) {
  if (!first) return;
  conv_table<conv_entries(L, L + 1)>(tab, tb.mx_lift);
  touch_lines<conv_steps(L) * 16>(tb.kq);
  touch_lines<conv_steps(L + 1) * 16>(tb.kb);
  __syncthreads();
  first = false;
}

// Inputs 4s..4s+3 of a conversion (zero past L).
template <int L>
__device__ __forceinline__ void pack_step(const double (&y)[L], int s, v4i& g0, v4i& g1) {
  double q[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) q[j] = 4 * s + j < L ? y[4 * s + j < L ? 4 * s + j : 0] : 0.0;
  conv_pack(q, L - 4 * s, g0, g1);
}

// The rest of a lift whose L residues o (balanced) and y_i = [o_i
// (Q/q_i)^-1]_{q_i} (packed in g0, g1), S = sum_i y_i / q_i are already in
// registers: the overflow count v (exact decision near a half-integer), then
// limbs L..2L of rs at vo.  tab: the conversion's constants in LDS.
// |conv_value| < 0.98 2^49 (m / 2 + 2^47.7), |v Q_b| <= (L / 2 + 1) 2^48: sums
// below 2^53.
// The matrix cores take the contraction off the FP64 VALU (15 -> 16 primes: 32
// matrix instructions and about 380 VALU issue slots per 64 coefficients
// against 1170 as split FMAs): the int64 lift 18 -> 12 us at one ciphertext,
// the lift of 2^12-point rings with 17 primes 20 -> 12.5 us.
template <int L, int SITE>
__device__ __forceinline__ void lift_tail(const double (&o)[L], const v4i (&g0)[conv_steps(L)],
                                          const v4i (&g1)[conv_steps(L)], double S,
                                          __amdgpu_buffer_rsrc_t rs, unsigned vo, unsigned ls,
                                          bool ok, const v4i* tab, const Tables& tb) {
  constexpr int LB = L + 1;
  double v = __builtin_rint(S);
  if (ok && lift_near_half(S, v, tb)) {
    double r[L];
#pragma unroll
    for (int i = 0; i < L; ++i) r[i] = to_canonical(o[i], cld(tb.p, i));
    v = __builtin_floor(S) + (mrc_greater_than_half<L>(r, tb.p, tb.pinv, tb.mrc_inv, tb.mrc_half) ? 1.0 : 0.0);
    atomicAdd(tb.margin + SITE, 1ull);
  }
  const unsigned so = store_off(ok, vo);
#pragma unroll
  for (int t = 0; t < conv_tiles(LB); ++t) {
    const double* kb = step_consts(tb.kb, t);
    ConvSum cs[4];
    conv_tile<L>(tab + t * conv_steps(L) * 64, g0, g1, cs);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int k = 4 * t + j;
      if (k >= LB) continue;
      const double b = cld(kb, 4 * j), binv = cld(kb, 4 * j + 1);
      const double a = __builtin_fma(-v, cld(kb, 4 * j + 3), conv_value<L>(cs[j], b, binv));
      buf_store(reduce_bal(a, b, binv), rs, so, (L + k) * ls);
    }
  }
}

// ------------------------------------------------- inverse-transform output ---

// Where a per-coefficient kernel reads coefficient c of a limb written by an
// inverse transform.  Plain: at c.  After the split inverse of a 2^15-point
// limb (FUSED) the coefficient is the inverse's last stage applied to the two
// half outputs U and V of its pair: U + V for the lower half of the
// coefficients, (U - V) w for the upper, w = the full inverse's last-stage
// twiddle of the limb's prime.  Every such value is only ever multiplied by a
// constant, so w is folded into that constant (the tables' second rows) and
// the kernels form U + V or U - V (|.| <= p + 8, as |U|, |V| <= p/2 + 4).
// Lanes l and l + 32 of a wave hold the two coefficients of a pair: each loads
// one of U and V and they trade (pair_combine).

// U + sg V for a pair whose U is in lane l and V in lane l + 32 (sg = +1
// in the lower lanes, -1 in the upper): a lower lane gets U + V, an upper
// lane U - V.  v_permlane32_swap exchanges the upper half of one
// register's lanes with the lower half of another's (a VALU operation, no
// LDS round trip); swapping a register with itself leaves U in every
// lane's first result and V in every lane's second, so no lane selects.
__device__ __forceinline__ double pair_combine(double x, double sg) {
  const unsigned long long b = __double_as_longlong(x);
  const unsigned lo = (unsigned)b, hi = (unsigned)(b >> 32);
  const auto l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
  const auto h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
  const double u = __longlong_as_double(((unsigned long long)h[0] << 32) | l[0]);
  const double v = __longlong_as_double(((unsigned long long)h[1] << 32) | l[1]);
  return __builtin_fma(sg, v, u);
}

// ----------------------------------------------------------------- scale ---

// The scale-and-round's second conversion and outputs (THIRD: the product's
// third component, the relinearization digit source).  rw: the destination,
// at lane offset wo.
template <int L, int A, bool THIRD>
__device__ __forceinline__ void scale_out(const v4i (&h0)[conv_steps(L + 1)],
                                          const v4i (&h1)[conv_steps(L + 1)], double v2,
                                          __amdgpu_buffer_rsrc_t rw, unsigned wo, unsigned ls,
                                          const v4i* tab, const Tables& tb) {
  constexpr int LB = L + 1;
  double grp[A];   // the current digit group's canonical mixed-radix digits
#pragma unroll
  for (int t = 0; t < conv_tiles(L); ++t) {
    const double* kq = step_consts(tb.kq, t);
    ConvSum sm[4];
    conv_tile<LB>(tab + t * conv_steps(LB) * 64, h0, h1, sm);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int i = 4 * t + j;
      if (i >= L) continue;
      const double q = cld(kq, 4 * j), qinv = cld(kq, 4 * j + 1);
      double o = reduce_bal(__builtin_fma(-v2, cld(kq, 4 * j + 3), conv_value<LB>(sm[j], q, qinv)),
                            q, qinv);
      // the third component is only read as relinearization digits: its
      // canonical residues, or with A primes per digit each digit's canonical
      // mixed-radix digits (Garner: limb g + m of the group starting at g gets
      // v_m = t_m, t_0 = d_{g+m}, t_{k+1} = [(t_k - v_k) q_{g+k}^-1]_{q_{g+m}};
      // every difference is below 2^49 < 2 q)
      if constexpr (THIRD) {
        o = to_canonical(o, q);
        if constexpr (A > 1) {
          const int m = i % A;
          if (m > 0) {
            double tt = o;
#pragma unroll
            for (int k = 0; k < m; ++k)
              tt = mul_bal(tt - grp[k], cld(tb.mrc_inv, (i - m + k) * L + i), q, qinv);
            o = to_canonical(tt, q);
          }
          grp[m] = o;
        }
      }
      buf_store(o, rw, wo, i * ls);
    }
  }
}

// dt: [n_poly][L+LB][N] coefficient domain (balanced).  Writes
// [round(t d / Q)]_Q into limbs 0..L-1 of the same poly.
// FUSED: dt holds the split inverse's half outputs (see above); each
// wave takes 32 coefficient pairs (c, c + N/2), lanes 0-31 the lower
// coefficients and 32-63 the upper, and writes its outputs in place at the
// positions it alone reads.  A: data primes per key-switching digit (the
// third component's digit format).  tb.dig_src (not null, A = 3 only): the
// third component (the relinearization digit source) goes there instead,
// ciphertext ct at dig_src + ct 2 (L + A) N (the key-switch sums' stride),
// limb i at + i N, and coefficient c at position (c mod 2) N/2 + c/2
// (k_ntt_fwd_par's layout; in place, those positions are read by other
// waves).
// Bound by memory traffic at many ciphertexts: 31 limbs in and 15 out per
// polynomial (15 + 3 primes), 1.16 GB at 32 ciphertexts, in 239 us (4.9 TB/s);
// the same conversions as split FP64 FMAs (4 per term, on the VALU) took 380.
// Every limb is loaded at the block's start: loaded as they were needed, the
// waits of the second half's limbs alone made it 310.  At one ciphertext 20 us
// (29): there it is latency, six waves per CU.  From 17 primes on the tables in
// LDS (52 KB and more a workgroup of four waves) leave three waves per SIMD or
// fewer, and the registers of the fourth hold the limbs: bounded to four, 17
// primes spilled 3 of them and 20 primes 12 (24 ciphertexts 225 us, now 212,
// and 325, now 276).
template <int L, bool FUSED, int A>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(L > 17 ? 2 : L > 16 ? 3 : 4)))
k_scale(int n, size_t n_poly, double* dt, Tables tb) {
  constexpr int LB = L + 1, W = L + LB;
  __shared__ v4i tab1[conv_entries(L, LB)];
  __shared__ v4i tab2[conv_entries(LB, L)];
  // a lane's constants depend on the coefficient's half: both rows of t_qhinv
  // and c1 in LDS, limb i's at 2 i
  __shared__ double kl[2 * W];
  conv_table<conv_entries(L, LB)>(tab1, tb.mx_c2);
  conv_table<conv_entries(LB, L)>(tab2, tb.mx_back);
  for (int t = (int)threadIdx.x; t < 2 * W; t += (int)blockDim.x) {
    const int i = t >> 1, r = t & 1;
    kl[t] = i < L ? tb.t_qhinv[r * L + i] : tb.c1[r * LB + i - L];
  }
  touch_lines<conv_steps(L) * 16>(tb.kq);
  touch_lines<conv_steps(LB) * 16>(tb.kb);
  __syncthreads();
  const int lane = (int)threadIdx.x & 63;
  const bool hi = FUSED && lane >= 32;
  const double sg = hi ? -1.0 : 1.0;
  const double* kc = kl + (hi ? 1 : 0);
  const unsigned ls = (unsigned)n * 8;   // bytes per limb
  const unsigned nb = poly_blocks(n, n_poly);
  for (unsigned bk = blockIdx.x; bk < nb; bk += gridDim.x) {
    // FUSED: the launcher requires N to be a multiple of the block (pb.ok holds)
    const PolyBlock pb = poly_block(n, bk);
    const auto rs = make_rsrc(dt + pb.pc * (size_t)W * n, (unsigned)(W * n * 8));
    const int t0 = (int)threadIdx.x;
    const int cp = ((pb.c - t0) >> 1) + (t0 >> 6) * 32 + (lane & 31);
    const unsigned vo = FUSED ? (unsigned)(cp + (hi ? n >> 1 : 0)) * 8 : (unsigned)pb.c * 8;
    double x[W];
#pragma unroll
    for (int i = 0; i < W; ++i) x[i] = buf_load(rs, vo, i * ls);
    loads_issued();
    double S = 0.0;
    v4i g0[conv_steps(L)], g1[conv_steps(L)];
    {
      double y[L];
#pragma unroll
      for (int s = 0; s < conv_steps(L); ++s) {
        const double* kq = step_consts(tb.kq, s);
#pragma unroll
        for (int j = 0; j < 4 && 4 * s + j < L; ++j) {
          const int i = 4 * s + j;
          const double p = cld(kq, 4 * j), pinv = cld(kq, 4 * j + 1);
          y[i] = mul_bal(FUSED ? pair_combine(x[i], sg) : x[i], kc[2 * i], p, pinv);
          S += y[i] * pinv;
        }
        pack_step<L>(y, s, g0[s], g1[s]);
      }
    }
    double v = __builtin_rint(S);
    if (pb.ok && lift_near_half(S, v, tb)) {
      // (both of a pair's values read again: its other lane may not be here)
      double r[L];
      const unsigned vu = FUSED ? (unsigned)cp * 8 : vo;
#pragma unroll
      for (int i = 0; i < L; ++i) {
        const double p = cld(tb.p, i), pinv = cld(tb.pinv, i);
        const double u = buf_load(rs, vu, i * ls);
        const double d = FUSED ? __builtin_fma(sg, buf_load(rs, vu + (unsigned)n * 4, i * ls), u) : u;
        r[i] = to_canonical(mul_bal(d, tb.t_q[(hi ? L : 0) + i], p, pinv), p);
      }
      v = __builtin_floor(S) + (mrc_greater_than_half<L>(r, tb.p, tb.pinv, tb.mrc_inv, tb.mrc_half) ? 1.0 : 0.0);
      atomicAdd(tb.margin + (FUSED ? MARGIN_SCALE_SPLIT : MARGIN_SCALE), 1ull);
    }
    // The first conversion's outputs, four base-B residues w_k per tile, are
    // the second's inputs, four per step: each tile's are packed at once, so
    // only their bytes are kept.  Every sum before a reduction stays below
    // 2^53 (a lazy product, |v b_hat_inv| <= (L / 2 + 1) 2^48 and |conv_value|
    // < 0.98 2^49), where reduce_bal is exact with its result within p/2 + 4,
    // so |w_k| <= 2^48.
    double S2 = 0.0;
    v4i h0[conv_steps(LB)], h1[conv_steps(LB)];
    static_assert(conv_tiles(LB) == conv_steps(LB), "a tile's outputs are a step's inputs");
#pragma unroll
    for (int t = 0; t < conv_tiles(LB); ++t) {
      const double* kb = step_consts(tb.kb, t);
      ConvSum sm[4];
      conv_tile<L>(tab1 + t * conv_steps(L) * 64, g0, g1, sm);
      double w[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int k = 4 * t + j;
        w[j] = 0.0;
        if (k >= LB) continue;
        const double b = cld(kb, 4 * j), binv = cld(kb, 4 * j + 1);
        const double d = FUSED ? pair_combine(x[L + k], sg) : x[L + k];
        const double acc = __builtin_fma(v, cld(kb, 4 * j + 2),
                                         mul_lazy(d, kc[2 * (L + k)], b, binv)) -
                           conv_value<L>(sm[j], b, binv);
        w[j] = reduce_bal(acc, b, binv);
        S2 += w[j] * binv;
      }
      conv_pack(w, LB - 4 * t, h0[t], h1[t]);
    }
    const double v2 = __builtin_rint(S2);
    if (pb.ok && __builtin_fabs(S2 - v2) > 0.25) atomicAdd(tb.margin + MARGIN_FAULT, 1ull);
    // where the outputs go: in place, or the digit source's own buffer and
    // position (see above; every input has been read by now)
    if (pb.pc % 3 != 2) {
      scale_out<L, A, false>(h0, h1, v2, rs, store_off(pb.ok, vo), ls, tab2, tb);
    } else {
      const bool own = A == 3 && tb.dig_src;
      const auto rw = make_rsrc(own ? tb.dig_src + (pb.pc / 3) * (size_t)(2 * (L + A)) * n
                                    : dt + pb.pc * (size_t)W * n,
                                (unsigned)((own ? L : W) * n * 8));
      const unsigned wo = own ? (((vo >> 3) & 1u) * (unsigned)(n >> 1) + (vo >> 4)) * 8u : vo;
      scale_out<L, A, true>(h0, h1, v2, rw, store_off(pb.ok, wo), ls, tab2, tb);
    }
  }
}

// ---------------------------------------------------------- key switching ---

// Digits whose loads are in flight together in the key-switch product, for
// chunks of ch ciphertexts and `per` loads per digit: as many as keep the
// loaded values within about 80 registers.  One digit at a time costs one
// memory latency per digit, which is most of the time at one ciphertext (24 ->
// 16 us with three-prime digits); from eight ciphertexts on the chunk's own
// loads fill the pipeline, and one digit at a time, its loads free to move
// into the products before them, is the faster (2^12-point ring, 8
// ciphertexts, 17 digits: 22 us against 27 in batches).
constexpr int mac_batch(int dn, int ch, int per) {
  const int fit = ch >= 8 || 40 / per < 1 ? 1 : 40 / per;
  const int rounds = (dn + fit - 1) / fit;
  return (dn + rounds - 1) / rounds;
}

// acc[ct][b][i] = sum_j dig[ct][j][i] * evk[j][b][i] (NTT domain) over the
// L / A digits, limbs i = 0..L+A-1 (the last A mod the special primes).
// The key is read once per chunk of CH ciphertexts.
template <int L, int A, int CH>
__global__ void __launch_bounds__(256) k_ks_mac(int n, int n_ct, const double* dig,
                                                const double* evk, double* acc, Tables tb) {
  constexpr int K = L + A;
  constexpr int DN = L / A;
  constexpr int UJ = mac_batch(DN, CH, 2 + CH);
  const size_t gid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= (size_t)K * n) return;
  const int i = (int)(gid / n);
  const int c = (int)(gid - (size_t)i * n);
  const int prime = i < L ? i : L + 1 + i;
  const double p = cld(tb.p, prime), pinv = cld(tb.pinv, prime);
  for (int c0 = 0; c0 < n_ct; c0 += CH) {
    double a0[CH], a1[CH];
#pragma unroll
    for (int u = 0; u < CH; ++u) a0[u] = a1[u] = 0.0;
    auto batch = [&](int j0) {
      // every load of the chunk and batch is issued before the products: past
      // the last ciphertext or digit the index is clamped (a valid address)
      // and the value is not used
      double e0[UJ], e1[UJ], dv[UJ][CH];
#pragma unroll
      for (int jj = 0; jj < UJ; ++jj) {
        const int j = j0 + jj < DN ? j0 + jj : DN - 1;
        e0[jj] = evk[((size_t)(j * 2 + 0) * K + i) * n + c];
        e1[jj] = evk[((size_t)(j * 2 + 1) * K + i) * n + c];
#pragma unroll
        for (int u = 0; u < CH; ++u) {
          const int cu = c0 + u < n_ct ? c0 + u : n_ct - 1;
          dv[jj][u] = __builtin_nontemporal_load(&dig[((size_t)(cu * DN + j) * K + i) * n + c]);
        }
      }
      if constexpr (UJ > 1) loads_issued();
#pragma unroll
      for (int jj = 0; jj < UJ; ++jj) {
        const int j = j0 + jj;
        if (j >= DN) break;
#pragma unroll
        for (int u = 0; u < CH; ++u) {
          a0[u] += mul_lazy(dv[jj][u], e0[jj], p, pinv);
          a1[u] += mul_lazy(dv[jj][u], e1[jj], p, pinv);
        }
        // digit transforms are not reduced at their end: |dv| < 15.1 p (at
        // most ten unreduced stages from inputs below 2.61 p, the bound of a
        // two-prime digit's value; 13.5 p from one-prime digits below 2 p and
        // from three-prime digits, reduced to balanced form first;
        // 6.1 p at N = 2^15), so each product with a balanced key is below
        // (1/2 + 0.094 x 15.1) p = 1.92 p and eight of them plus a reduced sum
        // stay below 15.9 p < 2^53 / p (> 16.6 p for p < 2^48.95): reduce the
        // sums every 8 digits
        if ((j & 7) == 7) {
#pragma unroll
          for (int u = 0; u < CH; ++u) {
            a0[u] = reduce_bal(a0[u], p, pinv);
            a1[u] = reduce_bal(a1[u], p, pinv);
          }
        }
      }
    };
    if constexpr (UJ > 1) {
#pragma unroll 1
      for (int j0 = 0; j0 < DN; j0 += UJ) batch(j0);
    } else {
      for (int j0 = 0; j0 < DN; ++j0) batch(j0);
    }
#pragma unroll
    for (int u = 0; u < CH; ++u) {
      if (c0 + u < n_ct) {
        acc[((size_t)((c0 + u) * 2 + 0) * K + i) * n + c] = reduce_bal(a0[u], p, pinv);
        acc[((size_t)((c0 + u) * 2 + 1) * K + i) * n + c] = reduce_bal(a1[u], p, pinv);
      }
    }
  }
}

// k_ks_mac for digit transforms by coefficient parity (k_ntt_fwd_par,
// N = 2^15): half 0 of a digit's limb holds E, half 1 holds O, both in the
// 2^14 transform's order (standard index k at (k mod 32) 512 + k / 32).
// Thread (u, m), u < 16, m < 1024, takes k = 16 m + u, whose values in the
// full transform are X_0 = E_k + z O_k and X_1 = E_k - z O_k (z =
// psi^brv(2^14 + k), tw_last), at its standard positions 2k and 2k + 1:
// stored, as the key and the sums are, at 2u 1024 + m and (2u + 1) 1024 + m
// (consecutive threads, consecutive addresses); E_k and O_k sit at
// (16 (m mod 2) + u) 512 + m / 2.  The sums are those of k_ks_mac.
// Bounds: |E|, |O| < 5.9 p, so |X| < 7 p and each product with a balanced
// key is below 1.16 p: eight of them plus a reduced sum stay below 15.9 p.
template <int L, int A, int CH>
__global__ void __launch_bounds__(256) k_ks_mac_par(int n_ct, const double* dig,
                                                    const double* evk, double* acc, Tables tb) {
  constexpr int K = L + A;
  constexpr int DN = L / A;
  constexpr int UJ = mac_batch(DN, CH, 4 + 2 * CH);
  constexpr int NF = 1 << 15, NH = NF / 2;
  const int gid = blockIdx.x * 256 + threadIdx.x;
  if (gid >= K * NH) return;
  const int i = gid >> 14;
  const int t = gid & (NH - 1);
  const int u = t >> 10, m = t & 1023;
  const int prime = i < L ? i : L + 1 + i;
  const double p = cld(tb.p, prime), pinv = cld(tb.pinv, prime);
  const double z = tb.tw_last[(size_t)i * NH + t];
  const size_t pe = (size_t)(((m & 1) << 4) + u) * 512 + (m >> 1);
  const size_t p0 = (size_t)(2 * u) * 1024 + m;
  for (int c0 = 0; c0 < n_ct; c0 += CH) {
    // [key component][position] per ciphertext of the chunk
    double a00[CH], a01[CH], a10[CH], a11[CH];
#pragma unroll
    for (int v = 0; v < CH; ++v) a00[v] = a01[v] = a10[v] = a11[v] = 0.0;
    auto batch = [&](int j0) {
      // every load of the chunk and batch is issued before the products: past
      // the last ciphertext or digit the index is clamped (a valid address)
      // and the value is not used
      double e00[UJ], e01[UJ], e10[UJ], e11[UJ], ev[UJ][CH], od[UJ][CH];
#pragma unroll
      for (int jj = 0; jj < UJ; ++jj) {
        const int j = j0 + jj < DN ? j0 + jj : DN - 1;
        const double* kj = evk + ((size_t)(j * 2) * K + i) * NF + p0;
        e00[jj] = kj[0];
        e01[jj] = kj[1024];
        e10[jj] = kj[(size_t)K * NF];
        e11[jj] = kj[(size_t)K * NF + 1024];
#pragma unroll
        for (int v = 0; v < CH; ++v) {
          const int cv = c0 + v < n_ct ? c0 + v : n_ct - 1;
          const double* dp = dig + ((size_t)(cv * DN + j) * K + i) * NF + pe;
          ev[jj][v] = __builtin_nontemporal_load(dp);
          od[jj][v] = __builtin_nontemporal_load(dp + NH);
        }
      }
      if constexpr (UJ > 1) loads_issued();
#pragma unroll
      for (int jj = 0; jj < UJ; ++jj) {
        const int j = j0 + jj;
        if (j >= DN) break;
#pragma unroll
        for (int v = 0; v < CH; ++v) {
          const double w = mul_lazy(od[jj][v], z, p, pinv);
          const double x0 = ev[jj][v] + w, x1 = ev[jj][v] - w;
          a00[v] += mul_lazy(x0, e00[jj], p, pinv);
          a01[v] += mul_lazy(x1, e01[jj], p, pinv);
          a10[v] += mul_lazy(x0, e10[jj], p, pinv);
          a11[v] += mul_lazy(x1, e11[jj], p, pinv);
        }
        if ((j & 7) == 7) {
#pragma unroll
          for (int v = 0; v < CH; ++v) {
            a00[v] = reduce_bal(a00[v], p, pinv);
            a01[v] = reduce_bal(a01[v], p, pinv);
            a10[v] = reduce_bal(a10[v], p, pinv);
            a11[v] = reduce_bal(a11[v], p, pinv);
          }
        }
      }
    };
    if constexpr (UJ > 1) {
#pragma unroll 1
      for (int j0 = 0; j0 < DN; j0 += UJ) batch(j0);
    } else {
      for (int j0 = 0; j0 < DN; ++j0) batch(j0);
    }
#pragma unroll
    for (int v = 0; v < CH; ++v) {
      if (c0 + v < n_ct) {
        double* o0 = acc + ((size_t)((c0 + v) * 2 + 0) * K + i) * NF + p0;
        double* o1 = acc + ((size_t)((c0 + v) * 2 + 1) * K + i) * NF + p0;
        o0[0] = reduce_bal(a00[v], p, pinv);
        o0[1024] = reduce_bal(a01[v], p, pinv);
        o1[0] = reduce_bal(a10[v], p, pinv);
        o1[1024] = reduce_bal(a11[v], p, pinv);
      }
    }
  }
}

// The centred residue r = [x]_P of a key-switch sum, P = P_0 ... P_{A-1},
// in mixed radix r = k_0 + P_0 k_1 + P_0 P_1 k_2 from its balanced residues
// a_m mod P_m (Garner, every digit balanced): k_0 = a_0,
// k_1 = [(a_1 - a_0) P_0^-1]_{P_1}, k_2 = [((a_2 - a_0) P_0^-1 - k_1) P_1^-1]_{P_2}
// (each difference below 2 P_m: all primes lie in [2^48, 2^49)).  With
// balanced digits |r| <= sum_m (P_m - 1)/2 prod_{l<m} P_l = (P - 1)/2: r is
// exactly the centred residue, with no comparison.
template <int A>
__device__ __forceinline__ void special_digits(const double (&a)[A], double (&k)[A],
                                               const Tables& tb, int L) {
  k[0] = a[0];
  if constexpr (A >= 2) {
    const int ip1 = 2 * L + 2;
    k[1] = mul_bal(a[1] - a[0], tb.p_inv_p[0], cld(tb.p, ip1), cld(tb.pinv, ip1));
  }
  if constexpr (A >= 3) {
    const int ip2 = 2 * L + 3;
    const double p2 = cld(tb.p, ip2), p2inv = cld(tb.pinv, ip2);
    const double t = mul_bal(a[2] - a[0], tb.p_inv_p[1], p2, p2inv);
    k[2] = mul_bal(t - k[1], tb.p_inv_p[2], p2, p2inv);
  }
}

// Limb m of a group's digits from the canonical residues o (Garner, as the
// scale-and-round's), in rotation-digit form; v: the group's plain digits so far.
template <int A>
__device__ __forceinline__ double rotation_digit(double o, int m, double (&v)[A], const double* inv,
                                                 int stride, double q, double qinv) {
  bool low = true;
#pragma unroll
  for (int k = 0; k < A; ++k) {
    if (k >= m) continue;
    o = mul_bal(o - v[k], cld(inv, k * stride), q, qinv);
    low = low && v[k] == 0.0;
  }
  if (m > 0) o = to_canonical(o, q);
  v[m] = o;
  return m > 0 && low ? -1.0 - o : o;
}

// The mod-down: e_b + (acc_b - [acc_b]_P) P^-1 mod q_i for both components b
// of each ciphertext (poly = ct * 2 + b), [acc_b]_P the centred residue mod P
// of the special limbs in mixed-radix digits k_m: per limb, acc_b times
// [N^-1 P^-1]_{q_i} (an inverse transform returns N times the sum) minus
// k_m times [(P_0 ... P_{m-1}) P^-1]_{q_i}.  Each lazy product is below
// 0.9 q_i (operands below 2 q_i: P_k may exceed q_i, all lie below 2^49), so a
// sum stays below 4.2 q_i.  What becomes of the result z (OUT):
//   MD_SUM   a rotation's, in a running sum: stored in ext (limbs 0..L-1), and component
//            1's rotation digits (see rotated_digit) in its limbs L..2L-1.  e_0 holds the
//            sum's component 0 and its rotation already (k_automorph), e_1 is what
//            ext holds;
//   MD_LIFT  stored in ext and lifted (limbs L..2L) for the squaring that
//            follows: the next level of a chain lifts exactly this;
//   MD_I64   canonical residues in the int64 output, with finish the mask's
//            (Delta, 0) - z; wt (table not null): a batched wave's ciphertexts,
//            written through the table's out pointers;
//   MD_SUM_I64  MD_SUM's z in the int64 output.
// one_e: component 1's e is zero (a rotation's), not read; SUM kinds: read in ext.
// FUSED: acc holds the split inverse's in-place half outputs of a 2^15-point
// limb (U of pair c at (c / 512) 1024 + c mod 512, V 512 further; see
// k_ntt_inv_half): lanes l and l + 32 of a wave hold the two coefficients of a
// pair (c, c + N/2) and trade half outputs as the scale-and-round does, the
// last inverse stage's twiddle folded into the second rows of NP_inv_q and
// ninv_P.
// Bound by memory traffic: MD_LIFT moves 33 limbs in and 31 out per polynomial
// (15 + 3 primes), 1.07 GB at 32 ciphertexts in 204 us (5.3 TB/s; 206 with the
// lift as split FMAs on the VALU).  At one ciphertext it is latency: every
// limb is loaded up front and the constants' cache lines are touched together
// (MD_LIFT 21 -> 13 us, MD_I64 12.5 -> 10).
template <int L, int A, bool FUSED, int OUT>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(L > 20 ? 2 : 4)))
k_moddown(int n, size_t n_poly, const double* __restrict__ acc, const double* __restrict__ dt,
          double* __restrict__ ext, int64_t* __restrict__ out, int finish, int one_e, Tables tb,
          WaveTab wt) {
  constexpr int K = L + A;
  constexpr int W = 2 * L + 1;
  constexpr bool SUM = OUT == MD_SUM || OUT == MD_SUM_I64, I64 = OUT == MD_I64 || OUT == MD_SUM_I64;
  __shared__ v4i tab[OUT == MD_LIFT ? conv_entries(L, L + 1) : 1];
  __shared__ double kl[2 * K];   // NP_inv_q's and ninv_P's two rows, limb i's at 2 i
  const int t = (int)threadIdx.x, lane = t & 63;
  const bool hi = FUSED && lane >= 32;
  const double sg = hi ? -1.0 : 1.0;
  const double* kc = kl + (hi ? 1 : 0);
  const unsigned ls = (unsigned)n * 8;
  const unsigned nb = poly_blocks(n, n_poly);
  bool first = true;
  for (unsigned bk = blockIdx.x; bk < nb; bk += gridDim.x) {
    const PolyBlock pb = poly_block(n, bk);
    const int cp = ((pb.c - t) >> 1) + (t >> 6) * 32 + (lane & 31);
    const int ht = n >> 6;                         // 512: see k_ntt_inv_half
    const unsigned pos =
        FUSED ? (unsigned)((cp / ht) * 2 * ht + cp % ht + (hi ? ht : 0)) * 8 : (unsigned)pb.c * 8;
    const int c = FUSED ? cp + (hi ? n >> 1 : 0) : pb.c;
    const unsigned vo = (unsigned)c * 8;
    const size_t cb = pb.pc, ct = cb >> 1;
    const int b = (int)(cb & 1);
    const auto ra = make_rsrc(acc + cb * (size_t)K * n, (unsigned)(K * n * 8));
    // (an empty buffer reads as zeros)
    const double* eb = SUM && b ? ext + cb * (size_t)W * n : dt + (ct * 3 + b) * (size_t)W * n;
    const auto re = make_rsrc(eb, !SUM && one_e && b ? 0u : (unsigned)(L * n * 8));
    const auto rs = make_rsrc(ext + cb * (size_t)W * n, (unsigned)(W * n * 8));
    // every load is issued before the first use
    double xa[K], e[L];
#pragma unroll
    for (int m = 0; m < A; ++m) xa[L + m] = buf_load(ra, pos, (L + m) * ls);
#pragma unroll
    for (int i = 0; i < L; ++i) {
      xa[i] = buf_load(ra, pos, i * ls);
      e[i] = buf_load(re, vo, i * ls);
    }
    loads_issued();
    if (first) {
      if constexpr (OUT == MD_LIFT) conv_table<conv_entries(L, L + 1)>(tab, tb.mx_lift);
      for (int k = t; k < 2 * K; k += (int)blockDim.x)
        kl[k] = k < 2 * L ? tb.NP_inv_q[(k & 1) * L + (k >> 1)] : tb.ninv_P[k - 2 * L];
      touch_lines<conv_steps(L) * 16>(tb.kq);
      touch_lines<conv_steps(L) * 4 * A>(tb.km);
      if constexpr (OUT == MD_LIFT) touch_lines<conv_steps(L + 1) * 16>(tb.kb);
      __syncthreads();
      first = false;
    }
    // [N^-1 acc_Pk]_Pk of this coefficient (balanced), then the centred
    // residue's mixed-radix digits
    const int ip = 2 * L + 1;
    double as[A], kP[A];
#pragma unroll
    for (int m = 0; m < A; ++m)
      as[m] = mul_bal(FUSED ? pair_combine(xa[L + m], sg) : xa[L + m], kc[2 * (L + m)],
                      cld(tb.p, ip + m), cld(tb.pinv, ip + m));
    special_digits<A>(as, kP, tb, L);
    const unsigned so = store_off(pb.ok, vo);
    int64_t* o64 = nullptr;
    if constexpr (I64)
      o64 = (wt.table ? wt.table[(size_t)(*wt.wave) * wt.stride + ct].out + (size_t)b * L * n
                      : out + cb * (size_t)L * n) + c;
    double o[L], y[L], grp[A];
    double S = 0.0;
    v4i g0[conv_steps(L)], g1[conv_steps(L)];
#pragma unroll
    for (int s = 0; s < conv_steps(L); ++s) {
      const double* kq = step_consts(tb.kq, s);
      const double* km = opaque_row(tb.km, 4 * A * s);
#pragma unroll
      for (int j = 0; j < 4 && 4 * s + j < L; ++j) {
        const int i = 4 * s + j;
        const double q = cld(kq, 4 * j), qinv = cld(kq, 4 * j + 1);
        double r = mul_lazy(FUSED ? pair_combine(xa[i], sg) : xa[i], kc[2 * i], q, qinv);
#pragma unroll
        for (int m = 0; m < A; ++m) r -= mul_lazy(kP[m], cld(km, A * j + m), q, qinv);
        r += e[i];
        if constexpr (OUT == MD_I64) {
          // finish: -z, plus Delta at coefficient 0 of c0
          if (finish) r = b == 0 && c == 0 ? cld(tb.delta_q, i) - r : -r;
        }
        const double z = reduce_bal(r, q, qinv);
        if constexpr (I64) {
          if (pb.ok) o64[(size_t)i * n] = to_i64(z, q);
        } else {
          buf_store(z, rs, so, i * ls);
        }
        if constexpr (OUT == MD_SUM) {
          const int m = i % A;
          if (b)
            buf_store(rotation_digit<A>(to_canonical(z, q), m, grp, tb.mrc_inv + (i - m) * L + i, L,
                                        q, qinv),
                      rs, so, (L + i) * ls);
        }
        if constexpr (OUT == MD_LIFT) {
          o[i] = z;
          y[i] = mul_bal(z, cld(kq, 4 * j + 2), q, qinv);
          S += y[i] * qinv;
        }
      }
      if constexpr (OUT == MD_LIFT) pack_step<L>(y, s, g0[s], g1[s]);
    }
    if constexpr (OUT == MD_LIFT)
      lift_tail<L, FUSED ? MARGIN_MODDOWN_LIFT : MARGIN_LIFT>(o, g0, g1, S, rs, vo, ls, pb.ok, tab,
                                                              tb);
  }
}

// Subtraction z = [x - y]_Q of two ciphertexts (int64, canonical; y one
// ciphertext broadcast when y_bcast) into ext limbs 0..L-1, followed by the
// lift of z (limbs L..2L): the first level of the chain, one kernel.  One
// thread per coefficient of each (ct, b) polynomial, in blocks (PolyBlock).
// wt (table not null): a batched wave's ciphertexts, x and y read through
// the table (a broadcast y is every entry's y).
template <int L, int SITE>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4)))
k_sub_lift(int n, size_t n_poly, const int64_t* __restrict__ xs, const int64_t* __restrict__ ys,
           int y_bcast, double* __restrict__ ext, Tables tb, WaveTab wt) {
  constexpr int W = 2 * L + 1;
  __shared__ v4i tab[conv_entries(L, L + 1)];
  bool first = true;
  const unsigned nb = poly_blocks(n, n_poly);
  for (unsigned bk = blockIdx.x; bk < nb; bk += gridDim.x) {
    const PolyBlock pb = poly_block(n, bk);   // poly = ct * 2 + b
    const size_t cb = pb.pc;
    const int b = (int)(cb & 1);
    const int64_t* xp;
    const int64_t* yp;
    if (wt.table) {
      const CtPtrs e = wt.table[(size_t)(*wt.wave) * wt.stride + (cb >> 1)];
      xp = e.x + (size_t)b * L * n + pb.c;
      yp = e.y + (size_t)b * L * n + pb.c;
    } else {
      xp = xs + cb * (size_t)L * n + pb.c;
      yp = (y_bcast ? ys + (size_t)b * L * n : ys + cb * (size_t)L * n) + pb.c;
    }
    const auto rs = make_rsrc(ext + cb * (size_t)W * n, (unsigned)(W * n * 8));
    const unsigned vo = (unsigned)pb.c * 8, ls = (unsigned)n * 8;
    int64_t xv[L], yv[L];
#pragma unroll
    for (int i = 0; i < L; ++i) {
      xv[i] = xp[(size_t)i * n];
      yv[i] = yp[(size_t)i * n];
    }
    loads_issued();
    lift_setup<L>(tab, tb, first);
    double o[L], y[L];
    double S = 0.0;
    const unsigned so = store_off(pb.ok, vo);
    v4i g0[conv_steps(L)], g1[conv_steps(L)];
#pragma unroll
    for (int s = 0; s < conv_steps(L); ++s) {
      const double* kq = step_consts(tb.kq, s);
#pragma unroll
      for (int j = 0; j < 4 && 4 * s + j < L; ++j) {
        const int i = 4 * s + j;
        const double q = cld(kq, 4 * j), qinv = cld(kq, 4 * j + 1);
        o[i] = reduce_bal((double)xv[i] - (double)yv[i], q, qinv);
        y[i] = mul_bal(o[i], cld(kq, 4 * j + 2), q, qinv);
        S += y[i] * qinv;
        buf_store(o[i], rs, so, i * ls);
      }
      pack_step<L>(y, s, g0[s], g1[s]);
    }
    lift_tail<L, SITE>(o, g0, g1, S, rs, vo, ls, pb.ok, tab, tb);
  }
}

// Canonical int64 residues of n_poly polynomials ([n_poly][L][N]) into ext
// limbs 0..L-1 (balanced) and their lift into limbs L..2L: the conversion
// (k_i64_to_polys) and the lift in one pass.  The first
// n_first polynomials come from in, the others from in2 (a product's two
// operands in one launch).
template <int L>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4)))
k_i64_lift(int n, size_t n_poly, const int64_t* __restrict__ in,
           const int64_t* __restrict__ in2, size_t n_first, double* __restrict__ ext, Tables tb) {
  constexpr int W = 2 * L + 1;
  __shared__ v4i tab[conv_entries(L, L + 1)];
  bool first = true;
  const unsigned nb = poly_blocks(n, n_poly);
  for (unsigned bk = blockIdx.x; bk < nb; bk += gridDim.x) {
    const PolyBlock pb = poly_block(n, bk);
    const int64_t* ip =
        (pb.pc < n_first ? in + pb.pc * (size_t)L * n : in2 + (pb.pc - n_first) * (size_t)L * n) +
        pb.c;
    const auto rs = make_rsrc(ext + pb.pc * (size_t)W * n, (unsigned)(W * n * 8));
    const unsigned vo = (unsigned)pb.c * 8, ls = (unsigned)n * 8;
    int64_t xv[L];
#pragma unroll
    for (int i = 0; i < L; ++i) xv[i] = ip[(size_t)i * n];
    loads_issued();
    lift_setup<L>(tab, tb, first);
    double o[L], y[L];
    double S = 0.0;
    const unsigned so = store_off(pb.ok, vo);
    v4i g0[conv_steps(L)], g1[conv_steps(L)];
#pragma unroll
    for (int s = 0; s < conv_steps(L); ++s) {
      const double* kq = step_consts(tb.kq, s);
#pragma unroll
      for (int j = 0; j < 4 && 4 * s + j < L; ++j) {
        const int i = 4 * s + j;
        const double q = cld(kq, 4 * j), qinv = cld(kq, 4 * j + 1);
        o[i] = from_u64(xv[i], q);
        y[i] = mul_bal(o[i], cld(kq, 4 * j + 2), q, qinv);
        S += y[i] * qinv;
        buf_store(o[i], rs, so, i * ls);
      }
      pack_step<L>(y, s, g0[s], g1[s]);
    }
    lift_tail<L, MARGIN_I64_LIFT>(o, g0, g1, S, rs, vo, ls, pb.ok, tab, tb);
  }
}

// ------------------------------------------------------ plaintext products ---

// The basis plaintext of one slot: m_i = N^-1 zeta^-i mod t, zinv = zeta^-1
// for the slot's root zeta (t < 2^24, so products fit 64 bits).
__global__ void __launch_bounds__(256) k_basis_plain(int n, uint64_t t, uint64_t zinv,
                                                     uint64_t ninv_t, int64_t* out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  uint64_t r = 1, b = zinv;
  for (unsigned e = (unsigned)i; e; e >>= 1) {
    if (e & 1) r = r * b % t;
    b = b * b % t;
  }
  out[i] = (int64_t)(r * ninv_t % t);
}

// Plaintext polynomial (int64 [N] in [0, t)) -> its centred value times
// N^-1 in each data prime (limbs 0..L-1 at stride N): the operand of a
// pointwise product whose inverse transform returns N times the result.
__global__ void __launch_bounds__(256) k_plain_limbs(int n, int L, int64_t t, const int64_t* pt,
                                                     double* out, Tables tb) {
  const size_t gid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= (size_t)L * n) return;
  const int i = (int)(gid / n);
  const int c = (int)(gid - (size_t)i * n);
  const int64_t v = pt[c];
  const double x = (double)(v > t / 2 ? v - t : v);
  out[gid] = mul_bal(x, cld(tb.ninv, i), cld(tb.p, i), cld(tb.pinv, i));
}

// out[ct][b][i] = fx[ct][b][i] pt[i] (NTT domain, data limbs of [ct][2][W][N];
// out may be fx).
__global__ void __launch_bounds__(256) k_pointwise_plain(int n, int L, int n_ct, const double* fx,
                                                         double* out, const double* pt,
                                                         Tables tb) {
  const size_t gid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= (size_t)n_ct * 2 * L * n) return;
  const size_t row = gid / n;
  const int c = (int)(gid - row * n);
  const int i = (int)(row % L);
  const size_t cb = row / L;
  const size_t off = (cb * (2 * L + 1) + i) * n + c;
  out[off] = mul_bal(fx[off], pt[(size_t)i * n + c], cld(tb.p, i), cld(tb.pinv, i));
}

// ----------------------------------------------------------- comparisons ---

// acc += the tensors of k products of transformed operands (acc = their sum
// when first): per limb of the extended basis, pointwise in the NTT domain, d0
// = a0 b0, d1 = a0 b1 + a1 b0, d2 = a1 b1, each running sum kept as a balanced
// residue.  fa, fb: [k][n_ct][2][W][N] (balanced transform outputs); acc:
// [n_ct][3][W][N].  Summing products' tensors before one scale-and-round
// is exact while the sum stays inside the extended basis' range.
__global__ void __launch_bounds__(256) k_tensor_mac(int n, int W, size_t total, int k,
                                                    const double* __restrict__ fa,
                                                    const double* __restrict__ fb,
                                                    double* __restrict__ acc, int first,
                                                    Tables tb) {
  const size_t gid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= total) return;
  const size_t per = (size_t)W * n;
  const size_t ct = gid / per, r = gid - ct * per;
  const int l = (int)(r / n);                 // extended-basis limb = prime index
  const double p = cld(tb.p, l), pinv = cld(tb.pinv, l);
  const double* a = fa + ct * 2 * per + r;
  const double* b = fb + ct * 2 * per + r;
  double* o = acc + ct * 3 * per + r;
  double d0 = 0.0, d1 = 0.0, d2 = 0.0;
  if (!first) {
    d0 = o[0];
    d1 = o[per];
    d2 = o[2 * per];
  }
#pragma unroll 4
  for (int j = 0; j < k; ++j, a += 2 * total, b += 2 * total) {
    const double a0 = a[0], a1 = a[per], b0 = b[0], b1 = b[per];
    d0 = reduce_bal(d0 + mul_lazy(a0, b0, p, pinv), p, pinv);
    d1 = reduce_bal(d1 + (mul_lazy(a0, b1, p, pinv) + mul_lazy(a1, b0, p, pinv)), p, pinv);
    d2 = reduce_bal(d2 + mul_lazy(a1, b1, p, pinv), p, pinv);
  }
  o[0] = d0;
  o[per] = d1;
  o[2 * per] = d2;
}

// out[jj * out_stride + r] = [sum_t coef[jj * k + t] * b.p[t][r]]_q per
// residue r < per, jj < J <= 16 (int64 canonical in and out).
// Coefficients are small centred integers (|c| <= 2^15: the comparison
// polynomial's coefficients mod a Fermat prime t <= 65537), stored as
// doubles (exact) and uniform across the grid: scalar loads that the FMAs
// take as they are, with no conversion per use.  Each input v (balanced, |v| <= 2^48) is
// split once as v = vh 2^24 + vl (split24), so that every product is an
// exact FMA (|vh c| <= 2^39): two exact sums per output over k <= 256
// terms (below 2^47), combined once as Wh [2^24]_q + Wl.  For the small
// plaintext primes' matrices (16 x 8 at t = 257: one pass), rings below 32
// and the single top term; JT: J fixed at compile time (1), or 0 for any J (a branch
// per output and term).
template <int JT>
__global__ void __launch_bounds__(256) k_lincomb(int n, int L, size_t per, int k, BabyPtrs b,
                                                 const double* coef, int Jr, int64_t* out,
                                                 size_t out_stride, Tables tb) {
  const int J = JT ? JT : Jr;
  const size_t gid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= per) return;
  const int i = (int)((gid / n) % L);
  const double p = cld(tb.p, i), pinv = cld(tb.pinv, i);
  constexpr int JA = JT ? JT : 16;
  double ah[JA], al[JA];
#pragma unroll
  for (int jj = 0; jj < JA; ++jj) ah[jj] = al[jj] = 0.0;
  // babies in groups of G whose loads are all issued before their products
  // (one load per term would leave the loop waiting on memory latency)
  constexpr int G = 4;
  int t = 0;
  for (; t + G <= k; t += G) {
    double vh[G], vl[G];
#pragma unroll
    for (int u = 0; u < G; ++u) split24(from_u64(b.p[t + u][gid], p), vh[u], vl[u]);
#pragma unroll
    for (int jj = 0; jj < JA; ++jj) {
      if (jj < J) {
#pragma unroll
        for (int u = 0; u < G; ++u) {
          const double c = cld(coef, jj * k + t + u);
          ah[jj] = __builtin_fma(vh[u], c, ah[jj]);
          al[jj] = __builtin_fma(vl[u], c, al[jj]);
        }
      }
    }
  }
  for (; t < k; ++t) {
    double vh, vl;
    split24(from_u64(b.p[t][gid], p), vh, vl);
#pragma unroll
    for (int jj = 0; jj < JA; ++jj) {
      if (jj < J) {
        const double c = cld(coef, jj * k + t);
        ah[jj] = __builtin_fma(vh, c, ah[jj]);
        al[jj] = __builtin_fma(vl, c, al[jj]);
      }
    }
  }
  const double t24 = cld(tb.two24, i);
#pragma unroll
  for (int jj = 0; jj < JA; ++jj)
    if (jj < J)
      out[(size_t)jj * out_stride + gid] =
          to_i64(reduce_bal(mul_lazy(ah[jj], t24, p, pinv) + al[jj], p, pinv), p);
}

// Four values' words -> their bytes 0..3, one word per byte position.
__device__ __forceinline__ void bytes_across(const unsigned (&w)[4], int (&o)[4]) {
  const unsigned a = __builtin_amdgcn_perm(w[1], w[0], 0x05010400u);   // b0 b0' b1 b1'
  const unsigned b = __builtin_amdgcn_perm(w[1], w[0], 0x07030602u);   // b2 b2' b3 b3'
  const unsigned c = __builtin_amdgcn_perm(w[3], w[2], 0x05010400u);
  const unsigned e = __builtin_amdgcn_perm(w[3], w[2], 0x07030602u);
  o[0] = (int)__builtin_amdgcn_perm(c, a, 0x05040100u);
  o[1] = (int)__builtin_amdgcn_perm(c, a, 0x07060302u);
  o[2] = (int)__builtin_amdgcn_perm(e, b, 0x05040100u);
  o[3] = (int)__builtin_amdgcn_perm(e, b, 0x07060302u);
}

// The same combinations of 256 inputs to 128 outputs (t = 65537), all outputs
// of 32 residues in one block, on the integer matrix cores.  A canonical value
// v < 2^49 is seven signed bytes (v + 0x808080808080, bytes 0..5 XOR 0x80; byte
// 6 is at most 2), and a coefficient's c - LC_BIAS exactly two (the host checks
// their range; -32768 <= c <= 32766).  v_mfma_i32_32x32x32_i8 sums every
// byte product of equal weight 2^(8s), s < 8, in 32 bits (|A_s| <= 2 256 2^14 =
// 2^23), and
//   sum_t c_t v_t = sum_s 2^(8s) A_s + LC_BIAS sum_t v_t
// is exact in two doubles (below 2^41 and 2^49) whose high one times 2^24 is
// reduced by one exact FMA.
// out[j * out_stride + r] may lie on the inputs: a block has read all the
// values of its residues before it writes any.
// Bound by HBM (256 values in and 128 out per residue): four waves hold 32
// residues' bytes in LDS (56 KB, two blocks to a compute unit), each wave loads
// 64 inputs at once and forms all eight weights of 32 outputs, so one pass
// reads each input once.  2 ciphertexts of N = 2^15, L = 15 (6.0 GB): 1.57 ms,
// 3.8 TB/s; eight passes of 16 outputs on the FP64 VALU took 7.0 ms.
constexpr int LC_K = LINCOMB_K, LC_RES = 32, LC_BIAS = LINCOMB_BIAS;
__global__ void __launch_bounds__(256, 2) k_lincomb_mx(int n, int L, const int64_t* in,
                                                       size_t in_stride, const double* coef,
                                                       int64_t* out, size_t out_stride,
                                                       Tables tb) {
  constexpr int STEPS = LC_K / 32;
  __shared__ v4i dig[STEPS][7][64];
  __shared__ unsigned long long sums[8][LC_RES];
  const int lane = (int)threadIdx.x & 63, wave = (int)threadIdx.x >> 6;
  const int col = lane & 31, half = lane >> 5;
  const size_t r0 = (size_t)blockIdx.x * LC_RES;
  const int64_t* src = in + r0 + col + (size_t)(wave * (LC_K / 4) + half * 16) * in_stride;
  unsigned long long v[2][16], sum = 0;
#pragma unroll
  for (int q = 0; q < 2; ++q)
#pragma unroll
    for (int u = 0; u < 16; ++u)
      v[q][u] = (unsigned long long)src[(size_t)(q * 32 + u) * in_stride];
  loads_issued();
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    v4i o[7];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      unsigned lo[4], hi[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const unsigned long long x = v[q][4 * g + u];
        sum += x;
        const unsigned long long w = x + 0x808080808080ull;
        lo[u] = (unsigned)w;
        hi[u] = (unsigned)(w >> 32);
      }
      int l[4], h[4];
      bytes_across(lo, l);
      bytes_across(hi, h);
#pragma unroll
      for (int a = 0; a < 4; ++a) o[a][g] = l[a] ^ (int)0x80808080u;
      o[4][g] = h[0] ^ (int)0x80808080u;
      o[5][g] = h[1] ^ (int)0x80808080u;
      o[6][g] = h[2];
    }
#pragma unroll
    for (int a = 0; a < 7; ++a) dig[wave * 2 + q][a][lane] = o[a];
  }
  sums[wave * 2 + half][col] = sum;
  __syncthreads();

  // this wave's 32 outputs: row j of the coefficients' tile, bytes as written
  // by the host (step, byte, lane)
  const v4i* ct = reinterpret_cast<const v4i*>(coef) + (size_t)wave * STEPS * 2 * 64 + lane;
  v16i acc[8] = {};
#pragma unroll 2
  for (int s = 0; s < STEPS; ++s) {
    const v4i c0 = ct[(s * 2) * 64], c1 = ct[(s * 2 + 1) * 64];
    v4i d[7];
#pragma unroll
    for (int a = 0; a < 7; ++a) d[a] = dig[s][a][lane];
#pragma unroll
    for (int a = 0; a < 7; ++a)
      acc[a] = __builtin_amdgcn_mfma_i32_32x32x32_i8(c0, d[a], acc[a], 0, 0, 0);
#pragma unroll
    for (int a = 0; a < 7; ++a)
      acc[a + 1] = __builtin_amdgcn_mfma_i32_32x32x32_i8(c1, d[a], acc[a + 1], 0, 0, 0);
  }
  unsigned long long all = 0;
#pragma unroll
  for (int u = 0; u < 8; ++u) all += sums[u][col];
  const double bl = (double)((int)(all & 0xffffff) * LC_BIAS),
               bh = (double)(all >> 24) * (double)LC_BIAS;
  const int i = (int)((r0 / n) % L);
  const double p = cld(tb.p, i), pinv = cld(tb.pinv, i);
  int64_t* dst = out + r0 + col + (size_t)(wave * 32 + half * 4) * out_stride;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    double wl = __builtin_fma((double)acc[1][r], 0x1p8, (double)acc[0][r] + bl);
    wl = __builtin_fma((double)acc[2][r], 0x1p16, wl);
    double wh = __builtin_fma((double)acc[4][r], 0x1p8, (double)acc[3][r] + bh);
    wh = __builtin_fma((double)acc[5][r], 0x1p16, wh);
    wh = __builtin_fma((double)acc[6][r], 0x1p24, wh);
    wh = __builtin_fma((double)acc[7][r], 0x1p32, wh);
    const double t = wh * 0x1p24;
    const double x = __builtin_fma(-__builtin_rint(t * pinv), p, t) + wl;
    dst[(size_t)(8 * (r / 4) + r % 4) * out_stride] = to_i64(reduce_bal(x, p, pinv), p);
  }
}

// The trivial encryption (Delta, 0) of 1 in each of n_ct ciphertexts.
__global__ void __launch_bounds__(256) k_fill_one(int n, int L, size_t total, int64_t* out,
                                                  Tables tb) {
  const size_t gid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= total) return;
  const size_t row = gid / n;                 // (ct * 2 + b) * L + i
  const int c = (int)(gid - row * n);
  const int i = (int)(row % L);
  const int b = (int)((row / L) & 1);
  out[gid] = (b == 0 && c == 0) ? to_i64(cld(tb.delta_q, i), cld(tb.p, i)) : 0;
}

// out = [x - y]_Q or [y - x]_Q (negate), y broadcast over ct if y_bcast.
__global__ void __launch_bounds__(256) k_diff_i64(int n, int L, size_t total, const int64_t* x,
                                                  const int64_t* y, int y_bcast, int negate,
                                                  int64_t* out, Tables tb) {
  const size_t gid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= total) return;
  const size_t per_ct = (size_t)2 * L * n;
  const int i = (int)((gid / n) % L);
  const int64_t q = (int64_t)cld(tb.p, i);
  const int64_t a = x[gid], b = y[y_bcast ? gid % per_ct : gid];
  int64_t d = negate ? b - a : a - b;
  out[gid] = d < 0 ? d + q : d;
}

// ------------------------------------------------------------- rotations ---

// A rotation's input: c0 in ext's component 0 (limbs 0..L-1, balanced) and the
// digits of c1 in ext's component 1, limbs L..2L-1 (rotation digits, below).
// The automorphism a(X) -> a(X^g) takes output coefficient j from i = j g^-1
// mod 2N when i < N, else from i - N with its sign changed (X^N = -1).
//
// Rotation digits: each digit group's canonical mixed-radix digits v_0, v_1,
// v_2 of [c1]_{Q_j} (residues when a digit is one prime), v_m stored as -1 - v_m
// when every lower digit of the group is zero (m > 0).  The digits of the
// negated coefficient, Q_j - D, then follow digit by digit: the first nonzero
// one becomes q_m - v_m, those above it q_m - 1 - v_m, those below stay 0.  So the
// digits are formed once, before the permutation, by the kernel that makes c1
// (the mod-down of the previous rotation).
__device__ __forceinline__ double rotated_digit(double x, bool neg, bool lowest, double q) {
  const bool low = lowest || x < 0.0;      // no nonzero digit below this one
  const double v = x < 0.0 ? -1.0 - x : x;
  const double c = low ? (v == 0.0 ? 0.0 : q - v) : q - 1.0 - v;
  return neg ? c : v;
}

// The rotation digits of ext's component 1 (residues in limbs 0..L-1), one
// thread per (ciphertext, digit group, coefficient).
template <int A>
__global__ void __launch_bounds__(256) k_rotation_digits(int n, int L, int n_ct, double* ext,
                                                         Tables tb) {
  const int groups = L / A;
  const size_t gid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= (size_t)n_ct * groups * n) return;
  const size_t row = gid / n;               // ct * groups + j
  const int c = (int)(gid - row * n);
  const size_t ct = row / groups;
  const int g = (int)(row - ct * groups) * A;
  double* d = ext + ((ct * 2 + 1) * (size_t)(2 * L + 1) + g) * n + c;
  double r[A], v[A];
#pragma unroll
  for (int m = 0; m < A; ++m) r[m] = d[(size_t)m * n];
#pragma unroll
  for (int m = 0; m < A; ++m) {
    const int i = g + m;
    const double q = cld(tb.p, i), qinv = cld(tb.pinv, i);
    d[(size_t)(L + m) * n] =
        rotation_digit<A>(to_canonical(r[m], q), m, v, tb.mrc_inv + g * L + i, L, q, qinv);
  }
}

// One limb of a rotation: where it comes from and goes to.
struct RotLimb {
  const double* src;
  double* dst;
  bool digit;      // a digit limb (else c0's, balanced)
  bool lowest;     // its group's first
  bool split;      // stored by coefficient parity
  bool add;        // c0's limb itself is added (a running sum)
  double q;
};

__device__ __forceinline__ RotLimb rot_limb(size_t item, int n, int L, int alpha,
                                            const double* ext, double* dt, double* dsrc,
                                            size_t dsrc_stride, int split, int sum,
                                            const Tables& tb) {
  const size_t W = (size_t)2 * L + 1;
  const size_t ct = item / (2 * L);
  const int r = (int)(item - ct * 2 * L), i = r < L ? r : r - L;
  RotLimb l;
  l.digit = r >= L;
  l.src = ext + (l.digit ? (ct * 2 + 1) * W + L + i : ct * 2 * W + i) * n;
  l.dst = l.digit ? dsrc + ct * dsrc_stride + (size_t)i * n : dt + (ct * 3 * W + i) * n;
  l.lowest = i % alpha == 0;
  l.split = l.digit && split;
  l.add = !l.digit && sum;
  l.q = cld(tb.p, i);
  return l;
}

__device__ __forceinline__ double rot_value(const RotLimb& l, double x, bool neg) {
  return l.digit ? rotated_digit(x, neg, l.lowest, l.q) : (neg ? -x : x);
}

// The automorphism into the key-switching input layout: sigma(c0) into dt's
// component 0 (component 1 is zero and not written: the mod-down's one_e), the
// digits of sigma(c1) into the digit source.  sum: c0 + sigma(c0) (unreduced) in place of
// sigma(c0), so that the running sum's mod-down reads one addend per component.
// Each value is read where it lies.
__global__ void __launch_bounds__(256) k_automorph(int n, int L, int alpha, int n_ct,
                                                   unsigned ginv, const double* ext, double* dt,
                                                   double* dsrc, size_t dsrc_stride, int split,
                                                   int sum, Tables tb) {
  const size_t gid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= (size_t)n_ct * 2 * L * n) return;
  const size_t item = gid / n;
  const int j = (int)(gid - item * n);
  const RotLimb l = rot_limb(item, n, L, alpha, ext, dt, dsrc, dsrc_stride, split, sum, tb);
  const unsigned s = ((unsigned)j * ginv) & (2u * n - 1u);
  const double own = l.add ? l.src[j] : 0.0;
  l.dst[l.split ? (j & 1) * (n >> 1) + (j >> 1) : j] =
      rot_value(l, l.src[s & (unsigned)(n - 1)], s >= (unsigned)n) + own;
}

// The same, one workgroup of 1024 threads per limb (N = 1024 E), staged through
// LDS as two 32-bit halves: the limb is read and written in order, and the
// permutation's reads, a stride of g^-1 (odd) words apart, meet no bank twice.
// Reading each value where it lies touches a cache line per value: 220 us for
// the column's 32 ciphertexts (15 + 3 primes) and 40 more for the digits, which
// followed the permutation; staged, with the digits formed before, 119 us
// (0.5 GB, bound by memory traffic).  Used from 90 limbs on: below that too few
// CUs hold a workgroup.  The sum costs it nothing (a limb's own values stay in
// registers and LDS; read again they cost what the mod-down saves) and takes 15
// limbs per ciphertext off the mod-down, 203 -> 172 us: the column's SUM 14.14 ->
// 13.90 ms, of three ciphertexts 1.95 -> 1.88.
template <int E>
__global__ void __launch_bounds__(1024) k_automorph_lds(int L, int alpha, unsigned ginv,
                                                        const double* ext, double* dt,
                                                        double* dsrc, size_t dsrc_stride,
                                                        int split, int sum, Tables tb) {
  constexpr int n = 1024 * E;
  __shared__ uint32_t lds[n];
  const RotLimb l = rot_limb(blockIdx.x, n, L, alpha, ext, dt, dsrc, dsrc_stride, split, sum, tb);
  const int tid = threadIdx.x;
  // (opaque per pass: no element's addresses stay in registers between passes)
  unsigned s0 = (unsigned)tid * ginv;
  const unsigned step = 1024u * ginv;
  const auto rs = make_rsrc(l.src, n * 8), rd = make_rsrc(l.dst, n * 8);
  const unsigned vo = (l.split ? (tid & 1) * (n >> 1) + (tid >> 1) : tid) * 8;
  const unsigned eo = l.split ? 4096 : 8192;   // bytes between a thread's elements
  const uint32_t mask = l.add ? ~0u : 0u;
  uint32_t lo[E], hi[E], own[E];   // own: the low half in order, for the sum
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const unsigned long long v = __double_as_longlong(buf_load(rs, tid * 8, e * 8192));
    lo[e] = (uint32_t)v;
    hi[e] = (uint32_t)(v >> 32);
  }
  loads_issued();
#pragma unroll
  for (int e = 0; e < E; ++e) {
    // (own registers: as halves of the loaded pairs they spill 42)
    asm volatile("v_mov_b32 %0, %1" : "=v"(lo[e]) : "v"(lo[e]));
    asm volatile("v_mov_b32 %0, %1" : "=v"(hi[e]) : "v"(hi[e]));
  }
#pragma unroll
  for (int e = 0; e < E; ++e) lds[e * 1024 + tid] = lo[e];
  __syncthreads();
#pragma unroll
  for (int e = 0; e < E; ++e) {
    own[e] = lo[e] & mask;
    lo[e] = lds[(s0 + e * step) & (n - 1)];
    if (e % 8 == 7) loads_issued();
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < E; ++e) lds[e * 1024 + tid] = hi[e];
  __syncthreads();
  loads_issued();
  asm volatile("" : "+v"(s0));
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const unsigned s = (s0 + e * step) & (2 * n - 1);
    const unsigned long long v = ((unsigned long long)lds[s & (n - 1)] << 32) | lo[e];
    double x = rot_value(l, __longlong_as_double(v), s >= (unsigned)n);
    x += __longlong_as_double(((unsigned long long)(lds[e * 1024 + tid] & mask) << 32) | own[e]);
    buf_store(x, rd, vo, e * eo);
    if (e % 4 == 3) loads_issued();
  }
}

// The third component of dt (limbs 0..L-1) into the digit source's own
// buffer: ciphertext ct at src + ct src_stride, coefficient c at position
// (c mod 2) N/2 + c/2 (see k_scale).
__global__ void __launch_bounds__(256) k_digit_split(int n, int L, int n_ct, const double* dt,
                                                     double* src, size_t src_stride) {
  const size_t gid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= (size_t)n_ct * L * n) return;
  const size_t row = gid / n;               // ct * L + i
  const int c = (int)(gid - row * n);
  const size_t ct = row / L;
  const int i = (int)(row - ct * L);
  const size_t W = (size_t)2 * L + 1;
  src[ct * src_stride + (size_t)i * n + (c & 1) * (n >> 1) + (c >> 1)] =
      dt[(ct * 3 * W + 2 * W + i) * n + c];
}

// A primes per key-switching digit (A = 2, 3): the digit source (limbs
// 0..L-1 of ciphertext ct at src + ct src_stride, canonical residues d_i, in
// any coefficient order) into each digit's
// canonical mixed-radix digits, in place (as k_scale writes them): limb
// g + m of the group starting at g = j A gets v_m = t_m, t_0 = d_{g+m},
// t_{k+1} = [(t_k - v_k) q_{g+k}^-1]_{q_{g+m}}, so that digit j,
// D_j = v_0 + q_g v_1 + q_g q_{g+1} v_2 in [0, Q_j), is [c]_{Q_j}.  One
// thread per (ciphertext, digit, coefficient).
template <int A>
__global__ void __launch_bounds__(256) k_digit_mrc(int n, int L, int n_ct, double* src,
                                                   size_t src_stride, Tables tb) {
  const int groups = L / A;
  const size_t gid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= (size_t)n_ct * groups * n) return;
  const size_t row = gid / n;               // ct * groups + j
  const int c = (int)(gid - row * n);
  const int j = (int)(row % groups);
  const size_t ct = row / groups;
  const int g = j * A;
  double* d = src + ct * src_stride + (size_t)g * n + c;
  double v[A];
  v[0] = d[0];
#pragma unroll
  for (int m = 1; m < A; ++m) {
    const int ib = g + m;
    const double q = cld(tb.p, ib), qinv = cld(tb.pinv, ib);
    double t = d[(size_t)m * n];
#pragma unroll
    for (int k = 0; k < m; ++k) t = mul_bal(t - v[k], cld(tb.mrc_inv, (g + k) * L + ib), q, qinv);
    v[m] = to_canonical(t, q);
    d[(size_t)m * n] = v[m];
  }
}

// ------------------------------------------------------------ boundary ---

// out = [a + sum_{j < k} b[j * stride]]_q per residue (BFV addition of
// canonical residues; each partial sum is kept in [0, q) by one
// conditional subtraction, so any k is exact).
__global__ void __launch_bounds__(256) k_sum_i64(int n, int L, size_t total, const int64_t* a,
                                                 const int64_t* b, size_t stride, int k,
                                                 int64_t* out, Tables tb) {
  const size_t gid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= total) return;
  const int i = (int)((gid / n) % L);
  const int64_t q = (int64_t)cld(tb.p, i);
  int64_t s = a[gid];
  for (int j = 0; j < k; ++j) {
    s += b[(size_t)j * stride + gid];
    s = s >= q ? s - q : s;
  }
  out[gid] = s;
}

__global__ void k_fill_table(TableChunk ch, CtPtrs* table) {
  const int i = threadIdx.x;
  if (i < ch.n) table[ch.first + i] = ch.e[i];
}

__global__ void k_set_counter(int* counter, int v) {
  if (threadIdx.x == 0 && blockIdx.x == 0) counter[0] = v;
}

__global__ void k_bump_counter(int* counter, int step) {
  if (threadIdx.x == 0 && blockIdx.x == 0) counter[0] += step;
}

__global__ void __launch_bounds__(256) k_sub_i64(int n, int L, size_t total, const int64_t* x,
                                                 const int64_t* y, int64_t* out, Tables tb) {
  const size_t gid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= total) return;
  const int i = (int)((gid / n) % L);
  const double p = cld(tb.p, i);
  double z = (double)x[gid] - (double)y[gid];
  out[gid] = (int64_t)(z < 0.0 ? z + p : z);
}

// int64 [n_ct][npoly][L][N] canonical -> balanced doubles at
// out + ct * ct_stride + poly * poly_stride + i * N.
__global__ void __launch_bounds__(256) k_i64_to_polys(int n, int L, int npoly, size_t total,
                                                      const int64_t* in, double* out,
                                                      size_t ct_stride, size_t poly_stride,
                                                      int canon_from, Tables tb) {
  const size_t gid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= total) return;
  const size_t row = gid / n;               // (ct * npoly + poly) * L + i
  const int c = (int)(gid - row * n);
  const int i = (int)(row % L);
  const size_t cp = row / L;
  const size_t ct = cp / npoly;
  const int poly = (int)(cp - ct * npoly);
  // polys from canon_from on keep the canonical residue (digit sources)
  out[ct * ct_stride + poly * poly_stride + (size_t)i * n + c] =
      poly >= canon_from ? (double)in[gid] : from_u64(in[gid], cld(tb.p, i));
}

// balanced doubles -> canonical int64 [n_ct][npoly][L][N].
__global__ void __launch_bounds__(256) k_polys_to_i64(int n, int L, int npoly, size_t total,
                                                      const double* in, size_t ct_stride,
                                                      size_t poly_stride, int64_t* out,
                                                      Tables tb) {
  const size_t gid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= total) return;
  const size_t row = gid / n;
  const int c = (int)(gid - row * n);
  const int i = (int)(row % L);
  const size_t cp = row / L;
  const size_t ct = cp / npoly;
  const int poly = (int)(cp - ct * npoly);
  out[gid] = to_i64(in[ct * ct_stride + poly * poly_stride + (size_t)i * n + c], cld(tb.p, i));
}

// rows of int64 residues -> balanced doubles; row r uses prime
// row_prime[r % nprime_rows].
__global__ void __launch_bounds__(256) k_i64_rows(size_t total, int n, const int64_t* in,
                                                  double* out, const int* row_prime,
                                                  int nprime_rows, Tables tb) {
  const size_t gid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= total) return;
  const size_t row = gid / n;
  const int prime = row_prime[row % nprime_rows];
  out[gid] = from_u64(in[gid], cld(tb.p, prime));
}

__device__ __forceinline__ int brv(int x, int bits) {
  return (int)(__builtin_bitreverse32((unsigned)x) >> (32 - bits));
}

// NTT-domain rows between the internal order and natural evaluation order:
// natural j holds a(psi^(2j+1)), i.e. standard position brv(j), stored at
// internal position (i mod E) * T + i / E.
__global__ void __launch_bounds__(256) k_ntt_order(size_t total, int log2n, int loge,
                                                   const double* in, int64_t* out,
                                                   const int* row_prime, int nprime_rows,
                                                   Tables tb) {
  const size_t gid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= total) return;
  const int n = 1 << log2n;
  const size_t row = gid / n;
  const int j = (int)(gid - row * n);
  const int prime = row_prime[row % nprime_rows];
  const int i = brv(j, log2n);
  const int E = 1 << loge;
  const int T = n >> loge;
  const int pos = (i & (E - 1)) * T + (i >> loge);
  out[gid] = to_i64(in[row * (size_t)n + pos], cld(tb.p, prime));
}

// p[0..words) = v (a fill kernel rather than hipMemsetAsync, so that calls
// a caller captures into a graph record no memset node).
__global__ void __launch_bounds__(256) k_fill_u64(uint64_t* p, size_t words, uint64_t v) {
  const size_t gid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid < words) p[gid] = v;
}

// Input check of the debug switch: *bad = 1 if a residue of the int64
// polynomials [n_poly][L][N] lies outside [0, q_i).
__global__ void __launch_bounds__(256) k_check_residues(int n, int L, size_t total,
                                                        const int64_t* in, Tables tb) {
  const size_t gid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= total) return;
  const int i = (int)((gid / (size_t)n) % (size_t)L);
  const int64_t v = in[gid];
  if (v < 0 || v >= (int64_t)tb.p[i]) atomicOr(tb.bad_input, 1);
}

// ---------------------------------------------------------------- host ---

// Workgroup and grid of the kernels that hold conversion constants in LDS
// (see poly_block): twice the tuned block, so that more waves share a copy,
// and at most POLY_GRID workgroups, which then take several blocks each.
constexpr size_t POLY_GRID = 4096;

static inline int poly_threads(const Dims& d) { return 2 * d.block; }

static inline dim3 poly_grid(const Dims& d, size_t n_poly) {
  const size_t nb = n_poly * (size_t)((d.n + poly_threads(d) - 1) / poly_threads(d));
  return dim3((unsigned)std::min(nb, POLY_GRID));
}

static inline dim3 grid_for(size_t total, int block = 256) {
  return dim3((unsigned)((total + block - 1) / block));
}

#define NSHE_L_CASES(X) X(2) X(3) X(4) X(8) X(12) X(15) X(16) X(17) X(20) X(24)
// data-prime counts built for two and three primes per key-switching digit
#define NSHE_L2_CASES(X) X(2) X(4) X(8) X(16)
#define NSHE_L3_CASES(X) X(3) X(12) X(15)

// f(L, alpha) as integral constants, for the decompositions built.
template <class F>
static hipError_t for_digits(int L, int alpha, F f) {
  using std::integral_constant;
#define C_(L_, A_) \
  if (L == L_) return f(integral_constant<int, L_>{}, integral_constant<int, A_>{});
#define C1_(L_) C_(L_, 1)
#define C2_(L_) C_(L_, 2)
#define C3_(L_) C_(L_, 3)
  if (alpha == 1) { NSHE_L_CASES(C1_) }
  if (alpha == 2) { NSHE_L2_CASES(C2_) }
  if (alpha == 3) { NSHE_L3_CASES(C3_) }
#undef C1_
#undef C2_
#undef C3_
#undef C_
  return hipErrorInvalidValue;
}

template <int OUT>
static hipError_t launch_moddown(const Dims& d, const double* acc, const double* dt, double* ext,
                                 int64_t* out, int finish, int one_e, const Tables& tb,
                                 hipStream_t st) {
  const size_t np = (size_t)d.n_ct * 2;
  // the split inverse's pairs need whole blocks (see k_moddown)
  if (d.fused && d.n % poly_threads(d)) return hipErrorInvalidValue;
  return for_digits(d.L, d.alpha, [&](auto l, auto a) {
    constexpr int L = decltype(l)::value, A = decltype(a)::value;
    if (d.fused)
      hipLaunchKernelGGL((k_moddown<L, A, true, OUT>), poly_grid(d, np), dim3(poly_threads(d)), 0,
                         st, d.n, np, acc, dt, ext, out, finish, one_e, tb, d.tab);
    else
      hipLaunchKernelGGL((k_moddown<L, A, false, OUT>), poly_grid(d, np), dim3(poly_threads(d)), 0,
                         st, d.n, np, acc, dt, ext, out, finish, one_e, tb, d.tab);
    return hipGetLastError();
  });
}

hipError_t run_moddown(const Dims& d, const double* acc, const double* dt, const ModDownOut& o,
                       const Tables& tb, hipStream_t st) {
  switch (o.kind) {
    case MD_SUM: return launch_moddown<MD_SUM>(d, acc, dt, o.ext, nullptr, 0, o.one_e, tb, st);
    case MD_LIFT: return launch_moddown<MD_LIFT>(d, acc, dt, o.ext, nullptr, 0, o.one_e, tb, st);
    case MD_I64:
      return launch_moddown<MD_I64>(d, acc, dt, o.ext, o.out, o.finish, o.one_e, tb, st);
    case MD_SUM_I64:
      return launch_moddown<MD_SUM_I64>(d, acc, dt, o.ext, o.out, 0, o.one_e, tb, st);
  }
  return hipErrorInvalidValue;
}

hipError_t run_i64_lift(const Dims& d, const int64_t* in, double* ext, const Tables& tb,
                        hipStream_t st, const int64_t* in2) {
  const size_t first = (size_t)d.n_ct * 2, np = in2 ? 2 * first : first;
  switch (d.L) {
#define C_(L_)                                                                                 \
  case L_:                                                                                     \
    hipLaunchKernelGGL(k_i64_lift<L_>, poly_grid(d, np), dim3(poly_threads(d)), 0, st, d.n, np, \
                       in, in2, first, ext, tb);                                               \
    break;
    NSHE_L_CASES(C_)
#undef C_
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t run_sub_lift(const Dims& d, const int64_t* x, const int64_t* y, int y_bcast,
                        double* ext, const Tables& tb, hipStream_t st) {
  const size_t np = (size_t)d.n_ct * 2;
  switch (d.L) {
#define C_(L_)                                                                            \
  case L_:                                                                                \
    if (d.fused)                                                                          \
      hipLaunchKernelGGL((k_sub_lift<L_, MARGIN_SUB_LIFT>), poly_grid(d, np),             \
                         dim3(poly_threads(d)), 0, st, d.n, np, x, y, y_bcast, ext, tb, d.tab); \
    else                                                                                  \
      hipLaunchKernelGGL((k_sub_lift<L_, MARGIN_LIFT>), poly_grid(d, np),                 \
                         dim3(poly_threads(d)), 0, st, d.n, np, x, y, y_bcast, ext, tb, d.tab); \
    break;
    NSHE_L_CASES(C_)
#undef C_
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t run_scale(const Dims& d, double* dt, const Tables& tb, hipStream_t st,
                     int digit_pairs, double* src) {
  const size_t np = (size_t)d.n_ct * 3;
  Tables t = tb;
  t.dig_src = src;
  // the split-inverse variant takes whole blocks (see k_scale)
  if (d.fused && d.n % poly_threads(d)) return hipErrorInvalidValue;
#define C_(L_, A_) \
  case L_:                                                                                     \
    if (d.fused)                                                                               \
      hipLaunchKernelGGL((k_scale<L_, true, A_>), poly_grid(d, np), dim3(poly_threads(d)),  \
                         0, st, d.n, np, dt, t);          \
    else                                                                                       \
      hipLaunchKernelGGL((k_scale<L_, false, A_>), poly_grid(d, np), dim3(poly_threads(d)), \
                         0, st, d.n, np, dt, t);          \
    break;
#define C1_(L_) C_(L_, 1)
#define C2_(L_) C_(L_, 2)
#define C3_(L_) C_(L_, 3)
  if (!digit_pairs) {
    switch (d.L) {
      NSHE_L_CASES(C1_)
      default: return hipErrorInvalidValue;
    }
  } else if (d.alpha == 2) {
    switch (d.L) {
      NSHE_L2_CASES(C2_)
      default: return hipErrorInvalidValue;
    }
  } else if (d.alpha == 3) {
    switch (d.L) {
      NSHE_L3_CASES(C3_)
      default: return hipErrorInvalidValue;
    }
  } else {
    return hipErrorInvalidValue;
  }
#undef C1_
#undef C2_
#undef C3_
#undef C_
  return hipGetLastError();
}

hipError_t run_ks_mac(const Dims& d, const double* dig, const double* evk, double* acc,
                      const Tables& tb, hipStream_t st) {
  const size_t total = (size_t)(d.L + d.alpha) * d.n;
  // a chunk wider than the ciphertexts present would only repeat its
  // (clamped) loads and products: the narrowest that holds them
  int ch = d.ks_chunk;
  while (ch > 1 && ch / 2 >= d.n_ct) ch /= 2;
  if (d.parity) {
    // four sums per ciphertext of a chunk: at most 16 ciphertexts
    if (d.n != (1 << 15)) return hipErrorInvalidValue;
    const size_t tp = (size_t)(d.L + d.alpha) * (d.n / 2);
    if (ch > 16) ch = 16;
    // as few passes over the key as the widest chunk takes, evenly filled: 11
    // ciphertexts run 12 wide, 20 as two chunks of 10 (12 wide)
    const int passes = (d.n_ct + ch - 1) / ch, even = (d.n_ct + passes - 1) / passes;
    for (int w : {1, 2, 3, 4, 6, 8, 12, 16})
      if (w >= even) {
        ch = std::min(ch, w);
        break;
      }
#define P0_(L_, A_, CH_)                                                                         \
  hipLaunchKernelGGL((k_ks_mac_par<L_, A_, CH_>), grid_for(tp), dim3(256), 0, st, d.n_ct, dig, evk, \
                     acc, tb);
#define P_(L_, A_) \
  case L_:                                                                                     \
    if (ch == 1) P0_(L_, A_, 1)                                                                \
    else if (ch == 2) P0_(L_, A_, 2)                                                           \
    else if (ch == 3) P0_(L_, A_, 3)                                                           \
    else if (ch == 4) P0_(L_, A_, 4)                                                           \
    else if (ch == 6) P0_(L_, A_, 6)                                                           \
    else if (ch == 8) P0_(L_, A_, 8)                                                           \
    else if (ch == 12) P0_(L_, A_, 12)                                                         \
    else P0_(L_, A_, 16)                                                                       \
    break;
#define P1_(L_) P_(L_, 1)
#define P2_(L_) P_(L_, 2)
#define P3_(L_) P_(L_, 3)
    if (d.alpha == 1) {
      switch (d.L) {
        NSHE_L_CASES(P1_)
        default: return hipErrorInvalidValue;
      }
    } else if (d.alpha == 2) {
      switch (d.L) {
        NSHE_L2_CASES(P2_)
        default: return hipErrorInvalidValue;
      }
    } else if (d.alpha == 3) {
      switch (d.L) {
        NSHE_L3_CASES(P3_)
        default: return hipErrorInvalidValue;
      }
    } else {
      return hipErrorInvalidValue;
    }
#undef P1_
#undef P2_
#undef P3_
#undef P_
#undef P0_
    return hipGetLastError();
  }
#define C0_(L_, A_, CH_)                                                                         \
  hipLaunchKernelGGL((k_ks_mac<L_, A_, CH_>), grid_for(total), dim3(256), 0, st, d.n, d.n_ct, dig, \
                     evk, acc, tb);
#define C_(L_, A_) \
  case L_:                                                                                     \
    if (ch == 1) C0_(L_, A_, 1)                                                                \
    else if (ch == 2) C0_(L_, A_, 2)                                                           \
    else if (ch == 4) C0_(L_, A_, 4)                                                           \
    else if (ch == 8) C0_(L_, A_, 8)                                                           \
    else if (ch == 32) C0_(L_, A_, 32)                                                         \
    else C0_(L_, A_, 16)                                                                       \
    break;
#define C1_(L_) C_(L_, 1)
#define C2_(L_) C_(L_, 2)
#define C3_(L_) C_(L_, 3)
  if (d.alpha == 1) {
    switch (d.L) {
      NSHE_L_CASES(C1_)
      default: return hipErrorInvalidValue;
    }
  } else if (d.alpha == 2) {
    switch (d.L) {
      NSHE_L2_CASES(C2_)
      default: return hipErrorInvalidValue;
    }
  } else if (d.alpha == 3) {
    switch (d.L) {
      NSHE_L3_CASES(C3_)
      default: return hipErrorInvalidValue;
    }
  } else {
    return hipErrorInvalidValue;
  }
#undef C1_
#undef C2_
#undef C3_
#undef C_
#undef C0_
  return hipGetLastError();
}

hipError_t run_digit_mrc(const Dims& d, double* src, size_t src_stride, const Tables& tb,
                         hipStream_t st) {
  if (d.alpha < 2 || d.alpha > 3 || d.L % d.alpha) return hipErrorInvalidValue;
  const size_t total = (size_t)d.n_ct * (d.L / d.alpha) * d.n;
  if (d.alpha == 2)
    hipLaunchKernelGGL(k_digit_mrc<2>, grid_for(total), dim3(256), 0, st, d.n, d.L, d.n_ct, src,
                       src_stride, tb);
  else
    hipLaunchKernelGGL(k_digit_mrc<3>, grid_for(total), dim3(256), 0, st, d.n, d.L, d.n_ct, src,
                       src_stride, tb);
  return hipGetLastError();
}

hipError_t run_digit_split(const Dims& d, const double* dt, double* src, size_t src_stride,
                           hipStream_t st) {
  const size_t total = (size_t)d.n_ct * d.L * d.n;
  hipLaunchKernelGGL(k_digit_split, grid_for(total), dim3(256), 0, st, d.n, d.L, d.n_ct, dt, src,
                     src_stride);
  return hipGetLastError();
}

hipError_t run_basis_plain(int n, uint64_t t, uint64_t zinv, uint64_t ninv_t, int64_t* out,
                           hipStream_t st) {
  hipLaunchKernelGGL(k_basis_plain, grid_for(n), dim3(256), 0, st, n, t, zinv, ninv_t, out);
  return hipGetLastError();
}

hipError_t run_plain_limbs(const Dims& d, int64_t t, const int64_t* pt, double* out,
                           const Tables& tb, hipStream_t st) {
  hipLaunchKernelGGL(k_plain_limbs, grid_for((size_t)d.L * d.n), dim3(256), 0, st, d.n, d.L, t, pt,
                     out, tb);
  return hipGetLastError();
}

hipError_t run_pointwise_plain(const Dims& d, const double* fx, double* out, const double* pt,
                               const Tables& tb, hipStream_t st) {
  const size_t total = (size_t)d.n_ct * 2 * d.L * d.n;
  hipLaunchKernelGGL(k_pointwise_plain, grid_for(total), dim3(256), 0, st, d.n, d.L, d.n_ct, fx, out,
                     pt, tb);
  return hipGetLastError();
}

hipError_t run_tensor_mac(const Dims& d, int k, const double* fa, const double* fb, double* acc,
                          int first, const Tables& tb, hipStream_t st) {
  const int W = 2 * d.L + 1;
  const size_t total = (size_t)d.n_ct * W * d.n;
  hipLaunchKernelGGL(k_tensor_mac, grid_for(total), dim3(256), 0, st, d.n, W, total, k, fa, fb,
                     acc, first, tb);
  return hipGetLastError();
}

hipError_t run_lincomb(const Dims& d, int k, const BabyPtrs& b, const double* coef, int J,
                       int64_t* out, size_t out_stride, const Tables& tb, hipStream_t st) {
  const size_t per = (size_t)d.n_ct * 2 * d.L * d.n;
  if (k < 1 || k > BabyPtrs::CAP || J < 1 || J > 16 || (J > 1 && out_stride < per))
    return hipErrorInvalidValue;
  if (J == 1)
    hipLaunchKernelGGL(k_lincomb<1>, grid_for(per), dim3(256), 0, st, d.n, d.L, per, k, b, coef,
                       J, out, out_stride, tb);
  else
    hipLaunchKernelGGL(k_lincomb<0>, grid_for(per), dim3(256), 0, st, d.n, d.L, per, k, b, coef,
                       J, out, out_stride, tb);
  return hipGetLastError();
}

bool lincomb_mx_fits(const Dims& d, int k, int J, const std::vector<double>& c) {
  if (k != LINCOMB_K || J != LINCOMB_J || d.n % LC_RES) return false;
  for (double x : c)
    if (x < LINCOMB_BIAS - 32896 || x > LINCOMB_BIAS + 32639) return false;
  return true;
}

std::vector<double> lincomb_mx_table(const std::vector<double>& c) {
  std::vector<double> tab((size_t)LINCOMB_K * LINCOMB_J * 2 / sizeof(double));
  int8_t* bytes = reinterpret_cast<int8_t*>(tab.data());
  for (int j = 0; j < LINCOMB_J; ++j)
    for (int t = 0; t < LINCOMB_K; ++t) {
      const int x = (int)c[(size_t)j * LINCOMB_K + t] - LINCOMB_BIAS;
      const int b0 = ((x + 128) & 255) - 128, b1 = (x - b0) / 256;
      const int lane = (t / 16 % 2) * 32 + j % 32;
      const size_t at = (((size_t)(j / 32) * (LINCOMB_K / 32) + t / 32) * 2 * 64 + lane) * 16 + t % 16;
      bytes[at] = (int8_t)b0;
      bytes[at + 64 * 16] = (int8_t)b1;
    }
  return tab;
}

hipError_t run_lincomb_mx(const Dims& d, const int64_t* in, size_t in_stride, const double* tab,
                          int64_t* out, size_t out_stride, const Tables& tb, hipStream_t st) {
  const size_t per = (size_t)d.n_ct * 2 * d.L * d.n;
  if (d.n % LC_RES || in_stride < per || out_stride < per) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_lincomb_mx, dim3((unsigned)(per / LC_RES)), dim3(256), 0, st, d.n, d.L, in,
                     in_stride, tab, out, out_stride, tb);
  return hipGetLastError();
}

hipError_t run_fill_one(const Dims& d, int64_t* out, const Tables& tb, hipStream_t st) {
  const size_t total = (size_t)d.n_ct * 2 * d.L * d.n;
  hipLaunchKernelGGL(k_fill_one, grid_for(total), dim3(256), 0, st, d.n, d.L, total, out, tb);
  return hipGetLastError();
}

hipError_t run_diff_i64(const Dims& d, const int64_t* x, const int64_t* y, int y_bcast,
                        int negate, int64_t* out, const Tables& tb, hipStream_t st) {
  const size_t total = (size_t)d.n_ct * 2 * d.L * d.n;
  hipLaunchKernelGGL(k_diff_i64, grid_for(total), dim3(256), 0, st, d.n, d.L, total, x, y,
                     y_bcast, negate, out, tb);
  return hipGetLastError();
}

hipError_t run_rotation_digits(const Dims& d, double* ext, const Tables& tb, hipStream_t st) {
  if (d.alpha < 1 || d.alpha > 3 || d.L % d.alpha) return hipErrorInvalidValue;
  const dim3 grid = grid_for((size_t)d.n_ct * (d.L / d.alpha) * d.n);
  if (d.alpha == 1)
    hipLaunchKernelGGL(k_rotation_digits<1>, grid, dim3(256), 0, st, d.n, d.L, d.n_ct, ext, tb);
  else if (d.alpha == 2)
    hipLaunchKernelGGL(k_rotation_digits<2>, grid, dim3(256), 0, st, d.n, d.L, d.n_ct, ext, tb);
  else
    hipLaunchKernelGGL(k_rotation_digits<3>, grid, dim3(256), 0, st, d.n, d.L, d.n_ct, ext, tb);
  return hipGetLastError();
}

hipError_t run_automorph(const Dims& d, unsigned ginv, const double* ext, double* dt,
                         const Tables& tb, hipStream_t st, double* src, size_t src_stride,
                         int src_split, int sum) {
  const size_t items = (size_t)d.n_ct * 2 * d.L;
  const dim3 grid((unsigned)items);
#define C_(E_)                                                                                  \
  case 1024 * E_:                                                                               \
    hipLaunchKernelGGL(k_automorph_lds<E_>, grid, dim3(1024), 0, st, d.L, d.alpha, ginv, ext, dt, \
                       src, src_stride, src_split, sum, tb);                                    \
    return hipGetLastError();
  if (items >= 90) {
    switch (d.n) { C_(1) C_(2) C_(4) C_(8) C_(16) C_(32) }
  }
#undef C_
  hipLaunchKernelGGL(k_automorph, grid_for(items * d.n), dim3(256), 0, st, d.n, d.L, d.alpha,
                     d.n_ct, ginv, ext, dt, src, src_stride, src_split, sum, tb);
  return hipGetLastError();
}

hipError_t run_sum_i64(const Dims& d, const int64_t* a, const int64_t* b, size_t stride, int k,
                       int64_t* out, const Tables& tb, hipStream_t st) {
  const size_t total = (size_t)d.n_ct * 2 * d.L * d.n;
  hipLaunchKernelGGL(k_sum_i64, grid_for(total), dim3(256), 0, st, d.n, d.L, total, a, b, stride,
                     k, out, tb);
  return hipGetLastError();
}

hipError_t run_fill_table(const TableChunk& ch, CtPtrs* table, hipStream_t st) {
  hipLaunchKernelGGL(k_fill_table, dim3(1), dim3(TableChunk::CAP), 0, st, ch, table);
  return hipGetLastError();
}

hipError_t run_set_counter(int* counter, int v, hipStream_t st) {
  hipLaunchKernelGGL(k_set_counter, dim3(1), dim3(64), 0, st, counter, v);
  return hipGetLastError();
}

hipError_t run_bump_counter(int* counter, int step, hipStream_t st) {
  hipLaunchKernelGGL(k_bump_counter, dim3(1), dim3(64), 0, st, counter, step);
  return hipGetLastError();
}

hipError_t run_sub_i64(const Dims& d, const int64_t* x, const int64_t* y, int64_t* out,
                       const Tables& tb, hipStream_t st) {
  const size_t total = (size_t)d.n_ct * 2 * d.L * d.n;
  hipLaunchKernelGGL(k_sub_i64, grid_for(total), dim3(256), 0, st, d.n, d.L, total, x, y, out, tb);
  return hipGetLastError();
}

hipError_t run_i64_to_polys(const Dims& d, const int64_t* in, int npoly_in, double* out,
                            size_t out_ct_stride, size_t out_poly_stride, int canon_from,
                            const Tables& tb, hipStream_t st) {
  const size_t total = (size_t)d.n_ct * npoly_in * d.L * d.n;
  hipLaunchKernelGGL(k_i64_to_polys, grid_for(total), dim3(256), 0, st, d.n, d.L, npoly_in, total,
                     in, out, out_ct_stride, out_poly_stride, canon_from, tb);
  return hipGetLastError();
}

hipError_t run_polys_to_i64(const Dims& d, const double* in, int npoly, size_t in_ct_stride,
                            size_t in_poly_stride, int64_t* out, const Tables& tb,
                            hipStream_t st) {
  const size_t total = (size_t)d.n_ct * npoly * d.L * d.n;
  hipLaunchKernelGGL(k_polys_to_i64, grid_for(total), dim3(256), 0, st, d.n, d.L, npoly, total,
                     in, in_ct_stride, in_poly_stride, out, tb);
  return hipGetLastError();
}

hipError_t run_i64_to_dbl_limbs(size_t rows, int n, const int64_t* in, double* out,
                                const int* row_prime, int nprime_rows, const Tables& tb,
                                hipStream_t st) {
  const size_t total = rows * n;
  hipLaunchKernelGGL(k_i64_rows, grid_for(total), dim3(256), 0, st, total, n, in, out, row_prime,
                     nprime_rows, tb);
  return hipGetLastError();
}

hipError_t run_fill_u64(void* p, size_t words, uint64_t v, hipStream_t st) {
  if (!words) return hipSuccess;
  hipLaunchKernelGGL(k_fill_u64, grid_for(words), dim3(256), 0, st, static_cast<uint64_t*>(p),
                     words, v);
  return hipGetLastError();
}

hipError_t run_check_residues(int n, int L, size_t n_poly, const int64_t* in, const Tables& tb,
                              hipStream_t st) {
  const size_t total = n_poly * L * (size_t)n;
  if (!total) return hipSuccess;
  hipLaunchKernelGGL(k_check_residues, grid_for(total), dim3(256), 0, st, n, L, total, in, tb);
  return hipGetLastError();
}

hipError_t run_ntt_order(int log2n, size_t rows, const double* in, int64_t* out,
                         const int* row_prime, int nprime_rows, int to_natural,
                         const Tables& tb, hipStream_t st) {
  int loge = 0, r0 = 0;
  if (ntt_rounds(log2n, &loge, &r0) < 0 || !to_natural) return hipErrorInvalidValue;
  const size_t total = rows << log2n;
  hipLaunchKernelGGL(k_ntt_order, grid_for(total), dim3(256), 0, st, total, log2n, loge, in, out,
                     row_prime, nprime_rows, tb);
  return hipGetLastError();
}

}  // namespace nshe
