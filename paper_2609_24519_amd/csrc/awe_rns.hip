// Residue number system around the mod-m products (Sec. 5.3): residues of
// int64 matrices for every modulus in one pass, and the Chinese-remainder
// reconstruction of the exact integer (Garner's mixed-radix form) with its
// correctly rounded double.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <bitset>
#include <cstdint>
#include <map>
#include <mutex>
#include <string>
#include <type_traits>

#include "awe_internal.h"
#include "plane_pack.h"

namespace awe {
namespace {

// x mod m for 0 <= x < 2^23 and 2 <= m <= 256, in full-rate arithmetic: x is exact
// in fp32 and x * inv (inv = 1/m in fp32) lies within 1/2 of x/m (two roundings of
// relative size 2^-24 on a quotient below 2^22), so the truncated quotient q is
// floor(x/m) - 1, floor(x/m) or floor(x/m) + 1; x + m - q m then lies in [0, 3m)
// and two unsigned-minimum steps (r - m wraps when r < m) bring it to [0, m).
__device__ __forceinline__ uint32_t mod_f(uint32_t x, uint32_t m, float inv) {
  const int32_t q = (int32_t)(uint32_t)((float)x * inv);  // below 2^22 + 1: a 24-bit operand
  uint32_t r = (uint32_t)((int32_t)(x + m) - __mul24(q, (int32_t)m));
  r = min(r, r - m);
  return min(r, r - m);
}

// Residue of one int64 value, given as its four 16-bit digits d0..d3 (two's
// complement) and its sign: u = sum_i d_i 2^(16 i) and x = u - 2^64 [x < 0], so
// x = d0 + d1 w16 + d2 w32 + d3 w48 - [x < 0] (2^64 mod m)  (mod m), with every
// product below 2^24 (24-bit multiplies) and the sum below 2^27; one more digit
// split brings it below 2^19 for mod_f.
struct ModConsts {
  uint32_t m, w16, w32, w48, negc;
  float inv;
  double dm, dinv;
};

__device__ __forceinline__ ModConsts mod_consts(const ResidueParams& P, int j) {
  return ModConsts{P.m[j], P.w16[j], P.w32[j], P.w48[j], P.negc[j], P.inv[j], (double)P.m[j], P.dinv[j]};
}

// Residue of an integer x with |x| < 2^53, held exactly as a double: q = floor(x * dinv)
// (dinv = 1/m in fp64) is within one of floor(x/m), since the product is within
// |x/m| 2^-52 <= 1 of x/m; x - q m is then an integer in [-m, 2m), computed exactly by
// one fused multiply-add, and brought to [0, m) as in mod_f.
__device__ __forceinline__ uint32_t residue_f64(double x, const ModConsts& k) {
  const double q = floor(x * k.dinv);
  uint32_t r = (uint32_t)((int32_t)fma(-q, k.dm, x) + (int32_t)k.m);
  r = min(r, r - k.m);
  return min(r, r - k.m);
}

// (neg_mask is all ones for a negative x, else zero: a select without a branch.)
__device__ __forceinline__ uint32_t residue_of(const uint32_t (&d)[4], uint32_t neg_mask, const ModConsts& k) {
  uint32_t t = d[0] + __umul24(d[1], k.w16) + __umul24(d[2], k.w32) + __umul24(d[3], k.w48) +
               (k.negc & neg_mask);
  t = __umul24(t >> 16, k.w16) + (t & 0xffffu);
  return mod_f(t, k.m, k.inv);
}

__device__ __forceinline__ void digits_of(int64_t v, uint32_t (&d)[4]) {
  const uint64_t u = (uint64_t)v;
  d[0] = (uint32_t)u & 0xffffu;
  d[1] = (uint32_t)(u >> 16) & 0xffffu;
  d[2] = (uint32_t)(u >> 32) & 0xffffu;
  d[3] = (uint32_t)(u >> 48);
}

// Residues of a rows x cols int64 matrix for every modulus: out[j * out_stride + r * cols + c].
// A thread takes 16 consecutive entries of a row.  kVec: cols and ld are multiples of 16 and
// the rows 128-byte aligned, so the entries come in as eight 16-byte loads and each modulus's
// 16 residues leave as one 16-byte store.
template <bool kVec>
__global__ __launch_bounds__(256) void residues_kernel(const int64_t* __restrict__ x, int64_t rows,
                                                       int64_t cols, int64_t ld, int64_t bound,
                                                       ResidueParams P, uint8_t* __restrict__ out,
                                                       int64_t out_stride, int32_t* flag) {
  constexpr int V = 16;
  const int64_t gpr = (cols + V - 1) / V;  // groups per row
  const int64_t total = rows * gpr;
  bool out_of_range = false;
  for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < total;
       g += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = g / gpr, c0 = (g - r * gpr) * V;
    const int64_t* src = x + r * ld + c0;
    uint8_t* dst = out + r * cols + c0;
    if (kVec) {
      int64_t v[V];
#pragma unroll
      for (int q = 0; q < V / 2; ++q) {
        const longlong2 w = reinterpret_cast<const longlong2*>(src)[q];
        v[2 * q] = w.x;
        v[2 * q + 1] = w.y;
      }
      bool small = true;  // every entry below 2^53 in magnitude: exact as a double
#pragma unroll
      for (int e = 0; e < V; ++e) {
        out_of_range |= v[e] > bound || v[e] < -bound;
        small &= v[e] < (int64_t(1) << 53) && v[e] > -(int64_t(1) << 53);
      }
      if (small) {
        double xd[V];
#pragma unroll
        for (int e = 0; e < V; ++e) xd[e] = (double)v[e];
        for (int j = 0; j < P.n; ++j) {
          const ModConsts k = mod_consts(P, j);
          uint32_t w[V / 4] = {};
#pragma unroll
          for (int e = 0; e < V; ++e) w[e >> 2] |= residue_f64(xd[e], k) << (8 * (e & 3));
          *reinterpret_cast<uint4*>(dst + j * out_stride) = make_uint4(w[0], w[1], w[2], w[3]);
        }
      } else {
        uint32_t d[V][4], negm[V];
#pragma unroll
        for (int e = 0; e < V; ++e) {
          digits_of(v[e], d[e]);
          negm[e] = (uint32_t)(v[e] >> 63);
        }
        for (int j = 0; j < P.n; ++j) {
          const ModConsts k = mod_consts(P, j);
          uint32_t w[V / 4] = {};
#pragma unroll
          for (int e = 0; e < V; ++e) w[e >> 2] |= residue_of(d[e], negm[e], k) << (8 * (e & 3));
          *reinterpret_cast<uint4*>(dst + j * out_stride) = make_uint4(w[0], w[1], w[2], w[3]);
        }
      }
    } else {
      const int n = (int)min((int64_t)V, cols - c0);
      for (int e = 0; e < n; ++e) {
        const int64_t v = src[e];
        out_of_range |= v > bound || v < -bound;
        uint32_t d[4];
        digits_of(v, d);
        for (int j = 0; j < P.n; ++j)
          dst[j * out_stride + e] = (uint8_t)residue_of(d, (uint32_t)(v >> 63), mod_consts(P, j));
      }
    }
  }
  if (out_of_range && flag) *flag = 1;
}

// ---------------------------------------------------------------------------
// Residues of an int64 operand for every modulus, turned straight into each modulus's stored E2M1
// planes (Alg. 1's table lookup applied to the residue), without the dense residue matrices in
// between.  One wave per brick of the plane layout, as the encoder: lane L = 32 h + t produces row t
// of the brick at reduction indices 32 h .. 32 h + 31 from that row's 32 entries, which it reads
// itself: on the A side 256 consecutive bytes, on the B side (x is K x N) one entry of each of 32
// rows, 256 bytes of a row per half wave, so nothing has to be transposed.
//
// Bound by its instructions (23 residues per entry), so a residue takes as few as possible.  With the
// sign bit flipped an entry is the unsigned u = x + 2^63, eight bytes b_i, and
// x = sum_i b_i (2^(8 i) mod m) - 2^63 (mod m): two four-way byte dot products onto the constant
// (-2^63 mod m), t < 8 255^2 + 256 < 2^20.  One fused multiply-add with 2^23 leaves
// q = round(t / m) in the low bits of a float (t 1/m is within 2^-4 / m of t / m), a 24-bit
// multiply-add the remainder t - q m, within m / 2 + 1 of zero, and that indexes the modulus's table
// directly, which is laid out for remainders -kLutHalf .. kLutHalf - 1.  Its entries hold one
// plane's code per byte, so a pair of entries packs with one shift-or and four pairs with a byte
// transpose.  1024 x 4096 and 4096 x 1024 entries, 23 moduli: 155 us for both operands with
// double-precision reductions to [0, m) and codes packed nibble by nibble, 92 us now.
// ---------------------------------------------------------------------------
constexpr int kLutHalf = 136;  // remainders lie within 129
constexpr int kLutSize = 2 * kLutHalf;

// Per side and modulus (index m - 2): the table above, written once per device.
__device__ uint32_t g_mod_lut[2][255][kLutSize];

// Some of these tables, from the modulus's packed codes of residues 0 .. m - 1 (plane p in bits
// 4p .. 4p + 3), one workgroup each.  The codes are kernel arguments: no copy, no host buffer to keep.
constexpr int kTablesPerLaunch = 7;  // 3.6 KB of arguments
struct TableArgs {
  uint16_t code[kTablesPerLaunch][256];
  uint16_t side[kTablesPerLaunch], m[kTablesPerLaunch];
};
__global__ __launch_bounds__(256) void mod_table_kernel(TableArgs t) {
  const int b = blockIdx.x, m = t.m[b];
  uint32_t* dst = g_mod_lut[t.side[b]][m - 2];
  for (int i = threadIdx.x; i < kLutSize; i += 256) {
    const int r = (i - kLutHalf) % m;
    const uint32_t c = t.code[b][r < 0 ? r + m : r];
    dst[i] = (c & 0xfu) | (((c >> 4) & 0xfu) << 8) | (((c >> 8) & 0xfu) << 16);
  }
}

struct ResidueSide {
  const int64_t* x;
  int64_t rows, K, ld, KS, R32, nbricks, bound;
  uint8_t* planes;
  int64_t plane_stride;
  int64_t off[kMaxModuli];  // modulus j's planes at planes + off[j]
  int32_t* flag;
};
struct ResidueModulus {
  uint32_t m, w_lo, w_hi, init;  // w: 2^(8 i) mod m as bytes; init: -2^63 mod m
  float inv;                     // 1/m
  int32_t np[2];                 // planes on the A and the B side
};
struct ResidueArgs {
  ResidueSide side[2];
  ResidueModulus mod[kMaxModuli];
  int32_t n, per_group;  // moduli, and moduli per workgroup (blockIdx.y)
  unsigned blocks_a;     // workgroups of the A side; the rest are B's
};

template <int SIDE>
__device__ __forceinline__ void residue_encode_side(const ResidueArgs& g, const uint32_t* slut, int j0, int j1,
                                                    int64_t brick) {
  const ResidueSide& a = g.side[SIDE];
  if (brick >= a.nbricks) return;
  const int lane = threadIdx.x & 63;
  int64_t rb, ks;
  if (SIDE == 0) {
    rb = brick / a.KS;
    ks = brick - rb * a.KS;
  } else {
    ks = brick / a.R32;
    rb = brick - ks * a.R32;
  }
  const int64_t row = rb * kBrickRows + (lane & 31), k0 = ks * kBrickK + (lane >> 5) * 32;
  // entries past the operand read as 0, whose codes are 0
  uint32_t lo[32], hi[32];
  const int64_t* src = SIDE == 0 ? a.x + row * a.ld + k0 : a.x + k0 * a.ld + row;
  if (row < a.rows && k0 + 32 <= a.K) {
#pragma unroll
    for (int e = 0; e < 32; ++e) {
      const uint64_t v = (uint64_t)src[SIDE == 0 ? e : e * a.ld];
      lo[e] = (uint32_t)v;
      hi[e] = (uint32_t)(v >> 32);
    }
  } else {
#pragma unroll
    for (int e = 0; e < 32; ++e) lo[e] = hi[e] = 0;
    if (row < a.rows && k0 < a.K) {
#pragma unroll
      for (int e = 0; e < 32; ++e)
        if (k0 + e < a.K) {
          const uint64_t v = (uint64_t)src[SIDE == 0 ? e : e * a.ld];
          lo[e] = (uint32_t)v;
          hi[e] = (uint32_t)(v >> 32);
        }
    }
  }
  if (a.flag && j0 == 0) {
    bool out = false;
#pragma unroll
    for (int e = 0; e < 32; ++e) {
      const int64_t v = (int64_t)(((uint64_t)hi[e] << 32) | lo[e]);
      out |= v > a.bound || v < -a.bound;
    }
    if (out) *a.flag = 1;
  }
#pragma unroll
  for (int e = 0; e < 32; ++e) hi[e] ^= 0x80000000u;
  for (int j = j0; j < j1; ++j) {
    const ResidueModulus& k = g.mod[j];
    const uint32_t w_lo = k.w_lo, w_hi = k.w_hi, init = k.init;
    const int32_t negm = -(int32_t)k.m;
    const float inv = k.inv;
    const uint32_t* lut = slut + (j - j0) * kLutSize + kLutHalf;
    uint32_t x[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      uint32_t c[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint32_t t = __builtin_amdgcn_udot4(hi[2 * i + h], w_hi, __builtin_amdgcn_udot4(lo[2 * i + h], w_lo, init, false), false);
        const uint32_t q = __float_as_uint(__builtin_fmaf((float)t, inv, 8388608.0f));
        c[h] = lut[__mul24((int32_t)q, negm) + (int32_t)t];
      }
      x[i] = c[0] | (c[1] << 4);
    }
    uint8_t* dst = a.planes + a.off[j] + (ks * a.R32 + rb) * kBrickBytes + lane * 16;
    auto store = [&](auto npc) {
      constexpr int NP = decltype(npc)::value;
      uint32_t d[4][4];  // [dword][plane]
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const uint32_t v[4] = {x[4 * w], x[4 * w + 1], x[4 * w + 2], x[4 * w + 3]};
        transpose4x4(v, d[w]);
      }
#pragma unroll
      for (int p = 0; p < NP; ++p)
        *reinterpret_cast<uint4*>(dst + p * a.plane_stride) = make_uint4(d[0][p], d[1][p], d[2][p], d[3][p]);
    };
    const int np = k.np[SIDE];
    if (np == 1)
      store(std::integral_constant<int, 1>{});
    else if (np == 2)
      store(std::integral_constant<int, 2>{});
    else
      store(std::integral_constant<int, 3>{});
  }
}

// Both operands: workgroups 0 .. blocks_a - 1 of a row A's, the others B's; row y takes the moduli
// y per_group .. of the set.
__global__ __launch_bounds__(256) void residue_encode_kernel(ResidueArgs g) {
  __shared__ uint32_t slut[kMaxModuli * kLutSize];
  const int side = blockIdx.x < g.blocks_a ? 0 : 1;
  const int j0 = blockIdx.y * g.per_group, j1 = min(g.n, j0 + g.per_group);
  for (int j = j0; j < j1; ++j) {
    const uint32_t* src = g_mod_lut[side][g.mod[j].m - 2];
    for (int i = threadIdx.x; i < kLutSize; i += blockDim.x) slut[(j - j0) * kLutSize + i] = src[i];
  }
  __syncthreads();
  const int wave = threadIdx.x >> 6;
  if (side == 0)
    residue_encode_side<0>(g, slut, j0, j1, (int64_t)blockIdx.x * 4 + wave);
  else
    residue_encode_side<1>(g, slut, j0, j1, (int64_t)(blockIdx.x - g.blocks_a) * 4 + wave);
}

// |X| < 2^127 (two's complement in lo/hi) -> nearest double, ties to even.
// The magnitude is shifted right until it fits in 64 bits, with every bit
// shifted out ORed into the lowest kept bit (a sticky bit), so that the one
// rounding of the 64-bit integer to 53 bits rounds as the full value would;
// the power-of-two scaling afterwards is exact.
__device__ __forceinline__ double wide_to_double(uint64_t lo, uint64_t hi) {
  const bool neg = (int64_t)hi < 0;
  if (neg) {  // negate the 128-bit value
    lo = ~lo + 1;
    hi = ~hi + (lo == 0 ? 1 : 0);
  }
  double d;
  if (hi == 0) {
    d = (double)lo;
  } else {
    const int s = 64 - __clzll((long long)hi);  // 1 .. 63: bits of hi in use
    const uint64_t sticky = (lo << (64 - s)) != 0 ? 1u : 0u;
    const uint64_t t = (hi << (64 - s)) | (lo >> s) | sticky;
    d = ldexp((double)t, s);
  }
  return neg ? -d : d;
}

// The reconstruction's constants (about 1.6 KiB: the digit coefficients alone are
// n(n-1)/2 bytes) are staged once per workgroup in LDS and read there as uniform
// 16-byte words; held in scalar registers they would not fit.  Residues come as int32 or as
// bytes (RT).
template <int NMAX, class RT>
__global__ __launch_bounds__(256) void crt_kernel(const RT* __restrict__ res, int64_t res_stride,
                                                  int64_t rows, int64_t cols, int64_t ld_res,
                                                  CrtParams P, int64_t* __restrict__ c128,
                                                  double* __restrict__ c64, int64_t ldc) {
  __shared__ CrtParams sp;
  static_assert(sizeof(CrtParams) % 16 == 0 && sizeof(CrtParams) / 16 <= 256, "one 16-byte word per thread");
  if (threadIdx.x < sizeof(CrtParams) / 16)
    reinterpret_cast<uint4*>(&sp)[threadIdx.x] = reinterpret_cast<const uint4*>(&P)[threadIdx.x];
  __syncthreads();
  const int n = P.n;
  const int64_t total = rows * cols;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
       i += (int64_t)gridDim.x * blockDim.x) {
    asm volatile("" ::: "memory");  // read the constants from LDS where used, not hoisted into registers
    const int64_t r = i / cols, c = i - r * cols;
    const RT* src = res + r * ld_res + c;
    // Mixed-radix digits: X = v_0 + v_1 P_1 + ... + v_{n-1} P_{n-1}, P_j = m_0 ... m_{j-1},
    // v_j = (r_j - sum_{i<j} v_i (P_i mod m_j)) (P_j^-1 mod m_j)  mod m_j
    //     = r_j d_j + sum_{i<j} v_i c_ji  mod m_j,  c_ji = -P_i d_j mod m_j, d_j = P_j^-1 mod m_j:
    // the digits are bytes, packed four to a word, so the sum is a chain of byte dot products
    // onto r_j d_j.  It stays below 2^21 + 2^16, and one reduction as in the residue encoder
    // leaves a remainder within 0.7 m_j of zero (t / m_j is off by less than 2^-3), brought to [0, m_j)
    // by an unsigned minimum.  (23 moduli, 1024^2 outputs: 46 us with one 24-bit multiply-add and a
    // byte extraction per coefficient and two reductions per digit, 33 us now.)
    int32_t rj[NMAX];
#pragma unroll
    for (int j = 0; j < NMAX; ++j) rj[j] = j < n ? (int32_t)src[j * res_stride] : 0;
    uint32_t v[NMAX], packed[(NMAX + 3) / 4];
#pragma unroll
    for (int q = 0; q < (NMAX + 3) / 4; ++q) packed[q] = 0;
#pragma unroll
    for (int j = 0; j < NMAX; ++j) {
      v[j] = 0;
      if (j < n) {
        const uint4 k = *reinterpret_cast<const uint4*>(&sp.mod[j]);  // m, inv, d
        uint32_t t = __umul24((uint32_t)rj[j], k.z);
#pragma unroll
        for (int q = 0; q < (j + 15) / 16; ++q) {
          const uint4 cw = *reinterpret_cast<const uint4*>(&sp.c[j][16 * q]);
          const uint32_t w[4] = {cw.x, cw.y, cw.z, cw.w};
#pragma unroll
          for (int u = 0; u < 4 && 16 * q + 4 * u < j; ++u) t = __builtin_amdgcn_udot4(packed[4 * q + u], w[u], t, false);
        }
        const uint32_t qt = __float_as_uint(__builtin_fmaf((float)t, __uint_as_float(k.y), 8388608.0f));
        const uint32_t r = (uint32_t)((int32_t)t - __mul24((int32_t)qt, (int32_t)k.x));
        v[j] = min(r, r + k.x);
        packed[j >> 2] |= v[j] << (8 * (j & 3));
      }
    }
    // Horner over groups of three digits, from the top: X = D_0 + B_0 (D_1 + B_1 (D_2 + ...)),
    // D_g = v_j + m_j (v_{j+1} + m_{j+1} v_{j+2}) < B_g = m_j m_{j+1} m_{j+2} <= 2^24 (j = 3 g),
    // on four 32-bit limbs with 32 x 32 + 64-bit multiply-adds.
    constexpr int NG = (NMAX + 2) / 3;
    uint32_t X[4] = {0, 0, 0, 0};
#pragma unroll
    for (int gi = NG - 1; gi >= 0; --gi) {
      const int j = 3 * gi;
      if (j >= n) continue;
      const uint32_t m0 = sp.mod[j].m, m1 = j + 1 < n ? sp.mod[j + 1].m : 0u;
      const uint32_t v1 = j + 1 < NMAX ? v[j + 1] : 0u, v2 = j + 2 < NMAX ? v[j + 2] : 0u;
      const uint32_t D = v[j] + __umul24(m0, v1 + __umul24(m1, v2));
      if (j + 3 >= n) {  // the top group starts the Horner chain
        X[0] = D;
      } else {
        const uint32_t B = m0 * m1 * sp.mod[j + 2].m;
        uint64_t t = (uint64_t)X[0] * B + D;
        X[0] = (uint32_t)t;
#pragma unroll
        for (int q = 1; q < 4; ++q) {
          t = (uint64_t)X[q] * B + (t >> 32);
          X[q] = (uint32_t)t;
        }
      }
    }
    uint64_t lo = ((uint64_t)X[1] << 32) | X[0], hi = ((uint64_t)X[3] << 32) | X[2];
    // into (-M/2, M/2], two's complement: subtract M when X > floor(M/2)
    if (hi > P.half_hi || (hi == P.half_hi && lo > P.half_lo)) {
      const uint64_t nlo = lo - P.M_lo;
      hi = hi - P.M_hi - (lo < P.M_lo ? 1u : 0u);
      lo = nlo;
    }
    const int64_t o = r * ldc + c;
    if (c128) {
      c128[2 * o] = (int64_t)lo;
      c128[2 * o + 1] = (int64_t)hi;
    }
    if (c64) c64[o] = wide_to_double(lo, hi);
  }
}

unsigned grid_for(int64_t total) {
  const int64_t blocks = (total + 255) / 256;
  return (unsigned)(blocks < 4096 ? (blocks > 0 ? blocks : 1) : 4096);
}

}  // namespace

awe_status launch_residues(const int64_t* x, int64_t rows, int64_t cols, int64_t ld, int64_t bound,
                           const ResidueParams& P, uint8_t* out, int64_t out_stride, int32_t* flag,
                           hipStream_t stream) {
  if (rows == 0 || cols == 0) return AWE_OK;
  const bool vec = cols % 16 == 0 && ld % 16 == 0 && (reinterpret_cast<uintptr_t>(x) & 127) == 0 &&
                   (reinterpret_cast<uintptr_t>(out) & 15) == 0 && (P.n == 1 || out_stride % 16 == 0);
  const unsigned grid = grid_for(rows * ((cols + 15) / 16));
  if (vec)
    hipLaunchKernelGGL(residues_kernel<true>, dim3(grid), dim3(256), 0, stream, x, rows, cols, ld, bound,
                       P, out, out_stride, flag);
  else
    hipLaunchKernelGGL(residues_kernel<false>, dim3(grid), dim3(256), 0, stream, x, rows, cols, ld, bound,
                       P, out, out_stride, flag);
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) {
    set_error(std::string("residues launch: ") + hipGetErrorString(err));
    return AWE_ERR_HIP;
  }
  return AWE_OK;
}

namespace {
// While it lives, calls of this thread may be ones that a capture of the global kind, open in any thread,
// would otherwise be invalidated by (none of them touches a capturing stream).
class RelaxedCapture {
 public:
  RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode_); }
  ~RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode_); }
  RelaxedCapture(const RelaxedCapture&) = delete;

 private:
  hipStreamCaptureMode mode_ = hipStreamCaptureModeRelaxed;
};

// The tables of g_mod_lut on one device.  They are written on a stream of their own, which waits for
// no other; `done` is recorded behind the latest, and other streams wait for it until it is seen
// complete.  (On the first caller's stream, every other stream's first call would wait for all that the
// former still has to do.  Creating the stream is 2.4 of the 5.1 ms that a process's first awe_gemm_crt
// takes with 23 moduli; later calls return after 22 us either way.)
struct ModTables {
  std::bitset<2 * 255> have;  // side 255 + m - 2: written, or being written before `done`
  hipStream_t stream = nullptr;
  hipEvent_t done = nullptr;
  bool pending = false;  // `done` has not been seen complete
};

// Makes the tables of both operands' moduli readable by what `stream` is given next, each written once per device (a table depends on its modulus alone).  The
// host does not wait, unless `stream` is being captured before tables it needs are seen complete: a
// captured wait could not refer to them.
hipError_t ensure_mod_tables(const ResidueEncodeArgs (&sides)[2], const uint32_t* m, int n, hipStream_t stream) {
  static std::mutex mu;
  static std::map<int, ModTables> devices;
  int dev = 0;
  hipError_t err = hipGetDevice(&dev);
  if (err != hipSuccess) return err;
  std::lock_guard<std::mutex> lk(mu);
  ModTables& t = devices[dev];
  int missing[2 * kMaxModuli], count = 0;  // side n + j
  for (int s = 0; s < 2; ++s)
    for (int j = 0; j < n; ++j)
      if (!t.have[s * 255 + m[j] - 2]) missing[count++] = s * n + j;
  if (count == 0 && !t.pending) return hipSuccess;

  const RelaxedCapture relaxed;
  if (count > 0) {
    if (!t.stream) err = hipStreamCreateWithFlags(&t.stream, hipStreamNonBlocking);
    if (err == hipSuccess && !t.done) err = hipEventCreateWithFlags(&t.done, hipEventDisableTiming);
    for (int i = 0; i < count && err == hipSuccess; i += kTablesPerLaunch) {
      TableArgs a{};
      const int k = std::min(kTablesPerLaunch, count - i);
      for (int b = 0; b < k; ++b) {
        const int s = missing[i + b] / n, j = missing[i + b] % n;
        a.side[b] = (uint16_t)s;
        a.m[b] = (uint16_t)m[j];
        for (uint32_t r = 0; r < m[j]; ++r) a.code[b][r] = (uint16_t)(sides[s].luts[j][r] & 0xfffu);
      }
      hipLaunchKernelGGL(mod_table_kernel, dim3((unsigned)k), dim3(256), 0, t.stream, a);
      err = hipGetLastError();
    }
    if (err == hipSuccess) err = hipEventRecord(t.done, t.stream);
    if (err != hipSuccess) return err;
    for (int i = 0; i < count; ++i) t.have.set((size_t)(missing[i] / n) * 255 + m[missing[i] % n] - 2);
    t.pending = true;
  } else if (hipEventQuery(t.done) == hipSuccess) {
    t.pending = false;
    return hipSuccess;
  } else {
    (void)hipGetLastError();  // (not ready yet, which the check of the next launch would report)
  }
  hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(stream, &capture) == hipSuccess && capture != hipStreamCaptureStatusNone) {
    err = hipEventSynchronize(t.done);
    if (err == hipSuccess) t.pending = false;
    return err;
  }
  return hipStreamWaitEvent(stream, t.done, 0);
}
}  // namespace

awe_status launch_residue_encode(const ResidueEncodeArgs (&sides)[2], const ResidueParams& P, hipStream_t stream) {
  ResidueArgs g{};
  int64_t blocks[2] = {0, 0}, bricks = 0;
  for (int j = 0; j < P.n; ++j) {
    const uint32_t m = P.m[j];
    uint32_t pw[8], x = 1;
    for (int i = 0; i < 8; ++i) {
      pw[i] = x % m;
      x = pw[i] * 256;
    }
    ResidueModulus& k = g.mod[j];
    k.m = m;
    k.inv = P.inv[j];
    k.w_lo = pw[0] | (pw[1] << 8) | (pw[2] << 16) | (pw[3] << 24);
    k.w_hi = pw[4] | (pw[5] << 8) | (pw[6] << 16) | (pw[7] << 24);
    k.init = (m - pw[7] * 128 % m) % m;
  }
  for (int s = 0; s < 2; ++s) {
    const ResidueEncodeArgs& a = sides[s];
    ResidueSide& o = g.side[s];
    o.x = a.x;
    o.rows = a.rows;
    o.K = a.K;
    o.ld = a.ld;
    o.KS = a.KS;
    o.R32 = a.R32;
    o.nbricks = a.nbricks;
    o.bound = a.bound;
    o.planes = a.planes;
    o.plane_stride = a.plane_stride;
    o.flag = a.flag;
    for (int j = 0; j < P.n; ++j) {
      if (a.np[j] > 3) {
        set_error("residue encoder: more than three planes");
        return AWE_ERR_UNSUPPORTED;
      }
      o.off[j] = a.off[j];
      g.mod[j].np[s] = a.np[j];
    }
    blocks[s] = (a.nbricks + 3) / 4;
    bricks += a.nbricks;
  }
  if (bricks == 0) return AWE_OK;
  if (blocks[0] + blocks[1] > (int64_t(1) << 24) - 1) {
    set_error("operands too large for the residue encoder");
    return AWE_ERR_UNSUPPORTED;
  }
  hipError_t err = ensure_mod_tables(sides, P.m, P.n, stream);
  if (err != hipSuccess) {
    set_error(std::string("residue tables: ") + hipGetErrorString(err));
    return AWE_ERR_HIP;
  }
  // A wave takes all moduli of its brick, or with few bricks a part of them (which reads the entries
  // once per part), up to 12288 waves: three times the 4 a SIMD holds, so that one wave's loads
  // meet another's arithmetic.  Whole awe_gemm_crt calls with 1, 3, 12 parts (us): 1024^2 x 4096
  // (4096 bricks) 338, 318, 373; 2048^3 (8192) 558, 572, 633; 300 x 200 x 1000 (272) 77, 58, 54.
  const int groups = (int)std::max<int64_t>(1, std::min<int64_t>(P.n, 12288 / bricks));
  g.n = P.n;
  g.per_group = (P.n + groups - 1) / groups;
  g.blocks_a = (unsigned)blocks[0];
  hipLaunchKernelGGL(residue_encode_kernel,
                     dim3((unsigned)(blocks[0] + blocks[1]), (unsigned)((P.n + g.per_group - 1) / g.per_group)),
                     dim3(256), 0, stream, g);
  err = hipGetLastError();
  if (err != hipSuccess) {
    set_error(std::string("residue encode launch: ") + hipGetErrorString(err));
    return AWE_ERR_HIP;
  }
  return AWE_OK;
}

template <class RT>
awe_status launch_crt_t(const RT* res, int64_t res_stride, int64_t rows, int64_t cols, int64_t ld_res,
                        const CrtParams& P, int64_t* c128, double* c64, int64_t ldc, hipStream_t stream) {
  if (rows == 0 || cols == 0) return AWE_OK;
  const dim3 grid(grid_for(rows * cols)), block(256);
  if (P.n <= 8)
    hipLaunchKernelGGL((crt_kernel<8, RT>), grid, block, 0, stream, res, res_stride, rows, cols, ld_res, P,
                       c128, c64, ldc);
  else if (P.n <= 16)
    hipLaunchKernelGGL((crt_kernel<16, RT>), grid, block, 0, stream, res, res_stride, rows, cols, ld_res, P,
                       c128, c64, ldc);
  else
    hipLaunchKernelGGL((crt_kernel<32, RT>), grid, block, 0, stream, res, res_stride, rows, cols, ld_res, P,
                       c128, c64, ldc);
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) {
    set_error(std::string("crt launch: ") + hipGetErrorString(err));
    return AWE_ERR_HIP;
  }
  return AWE_OK;
}

awe_status launch_crt(const int32_t* res, int64_t res_stride, int64_t rows, int64_t cols,
                      int64_t ld_res, const CrtParams& P, int64_t* c128, double* c64, int64_t ldc,
                      hipStream_t stream) {
  return launch_crt_t(res, res_stride, rows, cols, ld_res, P, c128, c64, ldc, stream);
}

awe_status launch_crt(const uint8_t* res, int64_t res_stride, int64_t rows, int64_t cols,
                      int64_t ld_res, const CrtParams& P, int64_t* c128, double* c64, int64_t ldc,
                      hipStream_t stream) {
  return launch_crt_t(res, res_stride, rows, cols, ld_res, P, c128, c64, ldc, stream);
}

}  // namespace awe
