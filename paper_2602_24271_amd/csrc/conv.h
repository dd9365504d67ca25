// Base conversions sum_i y_i M_ik (mod m_k) from one residue basis to another
// on the integer matrix cores, shared by the per-coefficient kernels and the
// conversion probe.
#pragma once
#include <cstdint>
#include <vector>

#include "modarith.h"

namespace nshe {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

// Conversion on the integer matrix cores (v_mfma_i32_32x32x32_i8).  Each input
// (an integer |y| <= 2^48) is eight signed bytes B_a: one addition of
// 1.5 2^52 + 0x808080808080 leaves y + sum_{a<6} 128 2^(8a) in the mantissa,
// bytes 0..5 XOR 0x80 are the balanced digits b_a, byte 6 is 56 + f (the
// addend's and the exponent's bits above f) and byte 7 is 67 (the exponent's):
//   y = sum_{a<6} 2^(8a) b_a + 2^48 f,  f in {-1, 0, 1}.
// Each constant is spread the same way per input byte: C_a = [M 2^(8a)]_m for
// a < 7 (balanced, |C_a| < 2^48), and C_7 = [-56 M 2^48 67^-1]_m so that the
// fixed parts of bytes 6 and 7 cancel mod m: sum_a B_a C_a = y M (mod m).
// With C_a = sum_{o<7} 2^(8o) c_ao (signed bytes, |c_a6| <= 1) the matrix
// cores form, for every output and all inputs at once, the seven sums
// s_o = sum_{i,a} B_ia c_iao (|s_o| <= 8 NT 2^14), exact in 32 bits.
//
// Tiles: a wave converts its 64 lanes' coefficients as two groups of 32
// columns.  Step s of the contraction takes inputs 4s..4s+3 (16 bytes per
// lane: half h of the lanes supplies inputs 4s + 2h and 4s + 2h + 1), tile t
// of the result outputs 4t..4t+3 (rows so placed that half h of the lanes
// receives the eight sums of outputs 4t + 2h and 4t + 2h + 1).  One
// v_permlane32_swap per register moves between "every lane one coefficient"
// and the two groups, so all other arithmetic keeps uniform (scalar)
// constants.
constexpr int conv_steps(int nt) { return (nt + 3) / 4; }
constexpr int conv_tiles(int no) { return (no + 3) / 4; }
// int4 entries of a conversion's constant matrix (one per lane, step and tile)
constexpr int conv_entries(int nt, int no) { return conv_steps(nt) * conv_tiles(no) * 64; }

constexpr double CONV_BIAS = 0x1.8p52 + 141289400074368.0;   // 1.5 2^52 + 0x808080808080

// Inputs 4s..4s+3 of every lane -> step s's operands of the two groups.
// use: how many of the four exist (the others' constants are zero).
__device__ __forceinline__ void conv_pack(const double (&y)[4], int use, v4i& g0, v4i& g1) {
  unsigned lo[4], hi[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const unsigned long long b = __double_as_longlong(y[j] + CONV_BIAS);
    lo[j] = j < use ? (unsigned)b ^ 0x80808080u : 0u;
    hi[j] = j < use ? (unsigned)(b >> 32) ^ 0x00008080u : 0u;
  }
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const auto l = __builtin_amdgcn_permlane32_swap(lo[j], lo[j + 2], false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(hi[j], hi[j + 2], false, false);
    g0[2 * j] = (int)l[0];
    g0[2 * j + 1] = (int)h[0];
    g1[2 * j] = (int)l[1];
    g1[2 * j + 1] = (int)h[1];
  }
}

// One output's sums as the three integers u = s_0 + 2^8 s_1, w = s_2 + 2^8 s_3
// and x = s_4 + 2^8 s_5 + 2^16 s_6 (and s_6 apart when x could pass 2^31: it
// is below 8 NT (2^14 + 2^22 + 2^23) < 2^31 for NT <= 21).
struct ConvSum {
  int u, w, x, x6;
};

// Tile t of a conversion of NT inputs: the four outputs' sums, every lane its
// own coefficient.  tab: the tile's constants (in LDS), entry s 64 + lane.
template <int NT>
__device__ __forceinline__ void conv_tile(const v4i* tab, const v4i (&g0)[conv_steps(NT)],
                                          const v4i (&g1)[conv_steps(NT)], ConvSum (&out)[4]) {
  constexpr bool X6 = NT > 21;
  const int lane = (int)threadIdx.x & 63;
  v16i a0{}, a1{};
#pragma unroll
  for (int s = 0; s < conv_steps(NT); ++s) {
    const v4i c = tab[s * 64 + lane];
    a0 = __builtin_amdgcn_mfma_i32_32x32x32_i8(c, g0[s], a0, 0, 0, 0);
    a1 = __builtin_amdgcn_mfma_i32_32x32x32_i8(c, g1[s], a1, 0, 0, 0);
  }
  auto pick = [](int p, int q, int& lo, int& hi) {
    const auto r = __builtin_amdgcn_permlane32_swap((unsigned)p, (unsigned)q, false, false);
    lo = (int)r[0];
    hi = (int)r[1];
  };
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int e = 8 * j;
    ConvSum& l = out[j];
    ConvSum& h = out[j + 2];
    pick(a0[e] + 256 * a0[e + 1], a1[e] + 256 * a1[e + 1], l.u, h.u);
    pick(a0[e + 2] + 256 * a0[e + 3], a1[e + 2] + 256 * a1[e + 3], l.w, h.w);
    if constexpr (X6) {
      pick(a0[e + 4] + 256 * a0[e + 5], a1[e + 4] + 256 * a1[e + 5], l.x, h.x);
      pick(a0[e + 6], a1[e + 6], l.x6, h.x6);
    } else {
      pick(a0[e + 4] + 256 * (a0[e + 5] + 256 * a0[e + 6]),
           a1[e + 4] + 256 * (a1[e + 5] + 256 * a1[e + 6]), l.x, h.x);
    }
  }
}

// An output from its sums, unreduced: u + 2^16 w + 2^32 x mod m, |result| <
// m / 2 + 2^47.7.  T = 2^32 x is an exact double below 2^63, and T - q m with
// q = rint(T fl(1/m)) is an integer below m, so the FMA returns it exactly.
template <int NT>
__device__ __forceinline__ double conv_value(const ConvSum& c, double m, double minv) {
  double x = (double)c.x;
  if constexpr (NT > 21) x = __builtin_fma((double)c.x6, 0x1p16, x);   // below 2^39
  const double t = x * 0x1p32;
  const double r = __builtin_fma(-__builtin_rint(t * minv), m, t);
  return r + __builtin_fma((double)c.w, 0x1p16, (double)c.u);
}

// A block's copy of a constant matrix into LDS (a barrier follows before use).
template <int ENTRIES>
__device__ __forceinline__ void conv_table(v4i* lds, const double* tab) {
  const v4i* g = reinterpret_cast<const v4i*>(tab);
  for (int i = (int)threadIdx.x; i < ENTRIES; i += (int)blockDim.x) lds[i] = g[i];
}

// Host: the constant matrix of a conversion, M[i][k] the canonical residue mod
// out[k] of input i's constant, as int4 entries (tile, step, lane).  Lane l of
// tile t: row l mod 32 holds sum b of output 4t + 2h + j, where the result's
// register r = 4 (row / 8) + row mod 4 = 8 j + b sits in half h = (row / 4)
// mod 2; byte 8 i' + a of lane half g is input 4s + 2g + i', byte a.
inline std::vector<int32_t> conv_matrix(const std::vector<uint64_t>& M, int nt,
                                        const std::vector<uint64_t>& out) {
  typedef unsigned __int128 u128;
  const int no = (int)out.size(), ns = conv_steps(nt);
  std::vector<int32_t> tab((size_t)conv_entries(nt, no) * 4, 0);
  uint8_t* bytes = reinterpret_cast<uint8_t*>(tab.data());
  for (int k = 0; k < no; ++k) {
    const uint64_t m = out[k];
    auto mul = [m](uint64_t a, uint64_t b) { return (uint64_t)((u128)a * b % m); };
    uint64_t inv67 = 1, b = 67, e = m - 2;
    for (; e; e >>= 1, b = mul(b, b))
      if (e & 1) inv67 = mul(inv67, b);
    const int t = k / 4, h = (k >> 1) & 1, j = k & 1;
    for (int i = 0; i < nt; ++i) {
      const int s = i / 4, g = (i >> 1) & 1, ip = i & 1;
      uint64_t c[8];
      c[0] = M[(size_t)i * no + k] % m;
      for (int a = 1; a < 7; ++a) c[a] = mul(c[a - 1], 256);
      c[7] = mul(mul(c[6], 56), inv67);
      c[7] = c[7] ? m - c[7] : 0;
      for (int a = 0; a < 8; ++a) {
        const int64_t v = c[a] > m / 2 ? (int64_t)c[a] - (int64_t)m : (int64_t)c[a];
        const int64_t w = v + 141289400074368ll;
        for (int o = 0; o < 7; ++o) {
          const int d = o < 6 ? (int)((w >> (8 * o)) & 255) - 128 : (int)(w >> 48);
          const int r = 8 * j + o, row = 8 * (r / 4) + 4 * h + r % 4;
          bytes[(((size_t)(t * ns + s) * 64) + g * 32 + row) * 16 + 8 * ip + a] = (uint8_t)(int8_t)d;
        }
      }
    }
  }
  return tab;
}

}  // namespace nshe
