// Device helpers of the GEMM kernels: copies into LDS, waits, operand fragments and the scaled
// MFMAs.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "gemm_layout.h"

namespace awe {
namespace {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v2i __attribute__((ext_vector_type(2)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));

constexpr uint32_t kScale2 = 0x80808080u;  // E8M0 2^1 in every byte

// f(integral_constant<int, Q>) for Q = I .. N - 1, unrolled at compile time.
template <int I, int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}

// One 16-byte-per-lane global -> LDS copy: the wave's 64 lanes fill the 1 KiB
// at LDS byte address `lds` (wave-uniform, in M0).  The brick's base address
// is wave-uniform (SGPRs); every lane adds its own 16-byte offset `voff`.
// Issued as inline assembly so that the compiler does not serialise the
// copies; completion is awaited explicitly with vmcnt.
__device__ __forceinline__ void dma_brick(const uint8_t* base, uint32_t voff, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(base), "s"(lds)
               : "memory");
}

template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Workgroup barrier that is also a compiler memory barrier: no LDS access may
// move across it.  The caller has already waited for its own copies (vmcnt)
// and LDS reads (lgkmcnt) as the protocol needs.
__device__ __forceinline__ void block_barrier() { asm volatile("s_barrier" ::: "memory"); }

__device__ __forceinline__ void wait_lgkm0() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

__device__ __forceinline__ v8i frag(const uint8_t* p) {
  const int4 x = *reinterpret_cast<const int4*>(p);
  v8i v = {x.x, x.y, x.z, x.w, 0, 0, 0, 0};
  return v;
}

// A lane's fragment of k-step i of a unit (the spans of frag_spans): E2M1 16 bytes, E4M3 32
// bytes, E2M3 24 bytes (the MFMA reads 6 of the 8 operand registers for E2M3, so the last two
// are left undefined instead of zeroed, which would cost two registers per fragment).
template <int FMT>
__device__ __forceinline__ v8i frag_fmt(const uint8_t* unit, int i, int lane) {
  constexpr Spans z = frag_spans<FMT>(0, 0);
  const Spans sp = frag_spans<FMT>(i, lane);
  if constexpr (FMT == 0) {
    return frag(unit + sp.off[0]);
  } else if constexpr (FMT == 1) {
    const int4 x = *reinterpret_cast<const int4*>(unit + sp.off[0]);
    const int4 y = *reinterpret_cast<const int4*>(unit + sp.off[0] + 16);
    v8i v = {x.x, x.y, x.z, x.w, y.x, y.y, y.z, y.w};
    return v;
  } else {
    static_assert(z.n == 2 && z.len[0] == 16 && z.len[1] == 8, "E2M3 spans");
    const v4i x = *reinterpret_cast<const v4i*>(unit + sp.off[0]);
    const v2i y = *reinterpret_cast<const v2i*>(unit + sp.off[1]);
    const v4i y4 = __builtin_shufflevector(y, y, 0, 1, -1, -1);
    return __builtin_shufflevector(x, y4, 0, 1, 2, 3, 4, 5, -1, -1);
  }
}

__device__ __forceinline__ void mfma_block(v16f& acc, const v8i& a, const v8i& b) {
  acc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, acc, 4, 4, 0, kScale2, 0, kScale2);
}

// E4M3 x E4M3 (format selects 0): the stored E4M3 values are the integers
// themselves, so both block scales are 2^0 (byte 127).
constexpr uint32_t kScale1 = 0x7f7f7f7fu;
__device__ __forceinline__ void mfma_block8(v16f& acc, const v8i& a, const v8i& b) {
  acc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, acc, 0, 0, 0, kScale1, 0, kScale1);
}

// E2M3 x E2M3 (format selects 2): a stored integer n is the E2M3 value n / 8, so
// both block scales are 2^3 (byte 130) and each product of codes is n_a n_b.
constexpr uint32_t kScale8 = 0x82828282u;
__device__ __forceinline__ void mfma_block6(v16f& acc, const v8i& a, const v8i& b) {
  acc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, acc, 2, 2, 0, kScale8, 0, kScale8);
}

// val mod m in [0, m) for an int32: q = round(val / m) and val - q m exactly in doubles (a remainder
// within m / 2 + 1 of zero).  Seven instructions; an integer division by a variable takes about 35,
// which cost the residue epilogues more than their stores.
struct ModReducer {
  double m, inv;
  int32_t mi;
  __device__ __forceinline__ explicit ModReducer(int32_t modulus)
      : m((double)modulus), inv(1.0 / (double)modulus), mi(modulus) {}
  __device__ __forceinline__ int32_t operator()(int32_t val) const {
    const double x = (double)val;
    const int32_t r = (int32_t)__builtin_fma(-__builtin_rint(x * inv), m, x);
    return (int32_t)min((uint32_t)r, (uint32_t)(r + mi));
  }
};

}  // namespace
}  // namespace awe
