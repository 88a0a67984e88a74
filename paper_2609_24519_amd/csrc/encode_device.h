// Device helpers of the byte encoder: the packed codes of one brick's inputs.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>

#include "awe_internal.h"
#include "plane_pack.h"

namespace awe {
namespace {

struct LutArg {
  uint32_t v[256];
};

struct EncodeArgs {
  const uint8_t* x;
  int64_t rows, K, ld, KS, R32, nbricks;
  int nplanes, nplanes8;
  bool fp6;
  uint8_t* planes;
  int64_t plane_stride;
  int32_t* flag;
};

// 16 and 8 bytes from any address (the memory system takes unaligned vector loads; rows of an odd
// length were read byte by byte before: 14 us a side at 1001 x 2049 and 2049 x 1537).
struct __attribute__((packed)) Any16 {
  uint32_t w[4];
};
struct __attribute__((packed)) Any8 {
  uint32_t w[2];
};

// B side: a wave's 64 x 32 input block lies column-major in LDS, kTileCol bytes per column (64 rows +
// 16 bytes of padding, so that the 16-byte column reads hit distinct banks).
constexpr int kTileCol = 80;

// The packed codes e[j] of the 32 inputs this lane owns in brick (rb, ks) (0 past the operand): lane
// 32 h + t has row rb*32 + t at reduction indices ks*64 + 32 h + j.  tw: this wave's tile (B side).
template <bool kTransposed>
__device__ __forceinline__ void brick_codes(const EncodeArgs& a, int64_t rb, int64_t ks, const uint32_t* slut,
                                            uint8_t* tw, uint32_t (&e)[32]) {
  const uint8_t* __restrict__ x = a.x;
  const int64_t rows = a.rows, K = a.K, ld = a.ld;
  const int lane = threadIdx.x & 63;
  const int64_t row = rb * kBrickRows + (lane & 31);
  const int64_t k0 = ks * kBrickK + (lane >> 5) * 32;
  const bool row_ok = row < rows;

  if (!kTransposed) {
    const uint8_t* src = x + row * ld + k0;
    if (row_ok && k0 + 32 <= K) {
      const Any16 lo = *reinterpret_cast<const Any16*>(src), hi = *reinterpret_cast<const Any16*>(src + 16);
#pragma unroll
      for (int j = 0; j < 32; ++j) e[j] = slut[((j < 16 ? lo.w[j >> 2] : hi.w[(j - 16) >> 2]) >> (8 * (j & 3))) & 0xff];
    } else {
#pragma unroll
      for (int j = 0; j < 32; ++j) e[j] = 0u;
      if (row_ok && k0 < K) {
#pragma unroll
        for (int j = 0; j < 32; ++j)
          if (k0 + j < K) e[j] = slut[src[j]];
      }
    }
  } else {
    // B side, K x N row-major: the brick needs the 64 x 32 block of B at rows
    // (reduction indices) ks*64 .. +63 and columns rb*32 .. +31.  Lane l takes columns
    // 8 (l & 3) .. +7 of block rows 4 (l >> 2) .. +3, transposes them in registers and writes four
    // rows of each column as one word of this wave's column-major tile; lane 32 h + t then reads
    // rows 32 h .. 32 h + 31 of column t as two 16-byte words.
    const int64_t n0 = rb * kBrickRows;
    const int c0 = 8 * (lane & 3), r0 = 4 * (lane >> 2);
    const int64_t kr = ks * kBrickK + r0;
    const uint8_t* src = x + kr * ld + n0 + c0;
    uint32_t v[2][4];
    if (n0 + 32 <= rows && kr + 4 <= K) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const Any8 t = *reinterpret_cast<const Any8*>(src + i * ld);
        v[0][i] = t.w[0];
        v[1][i] = t.w[1];
      }
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        v[0][i] = v[1][i] = 0;
        if (kr + i < K)
          for (int c = 0; c < 8; ++c)
            if (n0 + c0 + c < rows) v[c >> 2][i] |= (uint32_t)src[i * ld + c] << (8 * (c & 3));
      }
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      uint32_t t[4];
      transpose4x4(v[h], t);
#pragma unroll
      for (int c = 0; c < 4; ++c) *reinterpret_cast<uint32_t*>(tw + (c0 + 4 * h + c) * kTileCol + r0) = t[c];
    }
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): this wave's LDS writes are done
    __builtin_amdgcn_wave_barrier();
    const uint8_t* col = tw + (lane & 31) * kTileCol + (lane >> 5) * 32;
    const uint4 q0 = *reinterpret_cast<const uint4*>(col);
    const uint4 q1 = *reinterpret_cast<const uint4*>(col + 16);
    const uint32_t cw[8] = {q0.x, q0.y, q0.z, q0.w, q1.x, q1.y, q1.z, q1.w};
#pragma unroll
    for (int j = 0; j < 32; ++j)
      e[j] = (row_ok && k0 + j < K) ? slut[(cw[j >> 2] >> (8 * (j & 3))) & 0xff] : 0u;
  }
}

// Kernel arguments and workgroups of one side (none for an empty one).
inline unsigned encode_args(const EncodeLaunch& e, EncodeArgs& a) {
  const int64_t rb = (e.rows + kBrickRows - 1) / kBrickRows;
  a.x = reinterpret_cast<const uint8_t*>(e.x);
  a.rows = e.rows;
  a.K = e.K;
  a.ld = e.ld;
  a.KS = (e.K + kKPad - 1) / kKPad * kKPad / kBrickK;
  a.R32 = rb;
  // one brick per wave (the B side in groups of four column blocks, the last group padded); past
  // 2^22 workgroups the waves walk several bricks each (both sides' workgroups go into one launch,
  // which takes fewer than 2^32 threads).  A wide encoding's workgroups stage 16 KiB of table
  // each: past 2048 of them (8 per CU) their waves walk several bricks.
  a.nbricks = e.transposed ? (rb + 3) / 4 * 4 * a.KS : rb * a.KS;
  a.nplanes = e.nplanes;
  a.nplanes8 = e.nplanes8;
  a.fp6 = e.fp6;
  a.planes = e.planes;
  a.plane_stride = e.plane_stride;
  a.flag = e.flag;
  return (unsigned)std::min<int64_t>((a.nbricks + 3) / 4, e.wide ? 2048 : (int64_t(1) << 22));
}

}  // namespace
}  // namespace awe
