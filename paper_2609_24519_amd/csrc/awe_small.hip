// The multi-plane GEMM for outputs of few tiles (gfx950): the waves of a workgroup split the
// reduction among themselves, so that a small output still fills the chip.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>
#include <mutex>
#include <set>
#include <string>

#include "awe_internal.h"
#include "encode_device.h"
#include "gemm_device.h"

namespace awe {
namespace {

// A workgroup of 8 waves computes one BM x BN tile of C: WK groups of WM x WN waves, each group
// over the whole tile and its own share of the reduction stream.  The stream of a workgroup is
// the products one after another, each over the launch's reduction range in items of 128 indices
// (two bricks, or one E2M3 unit, per row block); group i takes the i-th of WK equal consecutive
// shares, folds its FP32 partials into int32 with the product's coefficient wherever its share
// leaves a product (or has covered a fold segment), and at the end the groups' int32 sums meet in
// LDS.  So a tile needs no zeroed C and no atomics, and residues, which need the whole sum, are
// split like every other product.
//
// What bounds it: at 2048^3 (256 tiles of 128 x 128) the copies alone run at 28 TB/s and the MFMAs
// alone at 6.5 PF/s (the board's power limit); together, one barrier per 256 indices, a reduction
// index costs 11.9 ns where these take 7.0 and 7.7, and about 10 us of prologue, folds, sums and
// stores do not shrink with K.  Smaller tiles pull more bytes per MFMA (0.5, 0.75, 1 and 2 KiB for
// 128 x 128, 64 x 128, 64 x 64 and 32 x 32) but let 1/4 or 1/16 of the outputs fill the chip.
// GEMM times against the 256 x 128 and 256 x 256 tiles, in one process (us): AWE6 2048^3 38.8
// against 50.3, 1024^3 11.3 / 27.9, 512^3 7.7 / 18.2, 1001 x 1537 x 2049 25.3 / 57.3, 16 x 8192 x
// 8192 31.1 / 151, INT4 x INT8 8192 x 512 x 8192 74.8 / 104, base-13 1024^3 12.8 / 17.5, mod 89
// 1024^3 9.6 / 27.3, E2M3 (weights in the scales) 2048^3 30.4 / 40.6 and 1024^3 11.8 / 27.0.
template <int BMW_, int BNW_, int WM_, int WN_, int WK_, int NST_, int FMT_>
struct SliceCfg {
  static constexpr int BMW = BMW_, BNW = BNW_;       // 32x32 blocks per wave
  static constexpr int WM = WM_, WN = WN_, WK = WK_;  // waves: tile rows, tile columns, shares
  static constexpr int NST = NST_;                    // stages (items) of the LDS ring
  static constexpr int FMT = FMT_;                    // 0 E2M1, 2 E2M3
  static constexpr int NQ = WM * WN, NW = NQ * WK, THREADS = 64 * NW;
  static constexpr int AB = WM * BMW, BB = WN * BNW;  // row and column blocks of the tile
  static constexpr int BM = 32 * AB, BN = 32 * BB;
  static constexpr int COPIES = FMT == 2 ? 3 : 2;     // 1 KiB copies per row block and item
  static constexpr int BLOCK_BYTES = COPIES * kBrickBytes;
  static constexpr int ITEM_BYTES = (AB + BB) * BLOCK_BYTES;  // one group's item
  static constexpr int STAGE_BYTES = WK * ITEM_BYTES;
  static constexpr int PER = (AB + BB) * COPIES / NQ;  // copies per wave and item
  static_assert((AB + BB) * COPIES % NQ == 0, "an item's copies split evenly over its waves");
  static_assert(NST >= 2 && (NST - 1) * PER < 64, "copies in flight fit the counter");
  static constexpr int NV = BMW * BNW * 16;            // int32 sums per lane
  static constexpr int SUM_BYTES = NW * NV * 64 * 4;
  static constexpr int LDS_BYTES = NST * STAGE_BYTES > SUM_BYTES ? NST * STAGE_BYTES : SUM_BYTES;
  static_assert(LDS_BYTES <= 160 * 1024, "LDS of one CU");
};

struct SliceArgs {
  const uint8_t* pa;
  const uint8_t* pb;
  int64_t stride_a, stride_b;
  int32_t rba, rbb;         // row blocks of the A and B planes
  int32_t item0, items;     // the launch's reduction range, in items of 128 indices
  int32_t seg;              // fold segment in items
  int32_t r;
  uint64_t pidx_a, pidx_b;  // plane of product k in bits 4k .. 4k+3
  int32_t ell[kMaxProducts];
  void* C;
  int64_t ldc;
  int32_t M, N;
  int32_t c64;              // C's elements: 0 int32, 1 int64, 2 bytes (residues only)
  int32_t accumulate, log2D, modulus;
  int64_t outer;
  int32_t tiles_m, tiles_n;
  int32_t split;            // workgroups per tile (over consecutive parts of the range)
};

// Workgroup -> tile: workgroups go round-robin over the 8 XCDs; each XCD takes a consecutive run
// of tiles in bands of 4 tile rows, so that the tiles it runs at once share rows of A and
// columns of B in its L2.
__device__ __forceinline__ void slice_tile(const SliceArgs& g, int t, int& tm, int& tn) {
  const int tiles = g.tiles_m * g.tiles_n, x = t & 7, q = tiles >> 3, rem = tiles & 7;
  const int lin = x * q + min(x, rem) + (t >> 3);
  const int per = 4 * g.tiles_n, grp = lin / per, first = 4 * grp;
  const int gm = min(g.tiles_m - first, 4), in = lin - grp * per;
  tm = first + in % gm;
  tn = in / gm;
}

// One 4-column group of outputs from the int32 sums w (modulo 2^32).
__device__ __forceinline__ void slice_store(const SliceArgs& g, const ModReducer& mod, int row, int col, v4i w) {
  if (row >= g.M || col >= g.N) return;
  const int64_t off = (int64_t)row * g.ldc + col;
  const int n = min(4, g.N - col);
  if (g.modulus) {
    const int32_t m = g.modulus;
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = mod(w[e]);
    if (g.c64 == 2) {
      uint8_t* Cp = reinterpret_cast<uint8_t*>(g.C) + off;
      if (n == 4 && !g.accumulate && (reinterpret_cast<uintptr_t>(Cp) & 3) == 0) {
        *reinterpret_cast<uint32_t*>(Cp) = (uint32_t)(w[0] | (w[1] << 8) | (w[2] << 16) | (w[3] << 24));
        return;
      }
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (e < n) {
          const int32_t s = g.accumulate ? Cp[e] + w[e] : w[e];
          Cp[e] = (uint8_t)(s >= m ? s - m : s);
        }
      return;
    }
    int32_t* Cp = reinterpret_cast<int32_t*>(g.C) + off;
    if (g.accumulate) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (e < n) {
          const int32_t s = Cp[e] + w[e];
          w[e] = s >= m ? s - m : s;
        }
    }
    if (n == 4 && (reinterpret_cast<uintptr_t>(Cp) & 15) == 0) {
      *reinterpret_cast<v4i*>(Cp) = w;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (e < n) Cp[e] = w[e];
    }
    return;
  }
  if (g.c64) {
    int64_t* Cp = reinterpret_cast<int64_t*>(g.C) + off;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (e < n) {
        const int64_t t = (int64_t)(w[e] >> g.log2D) * g.outer;
        if (g.split > 1)
          atomicAdd(reinterpret_cast<unsigned long long*>(Cp + e), (unsigned long long)t);
        else
          Cp[e] = g.accumulate ? Cp[e] + t : t;
      }
    return;
  }
  // (int32 C takes the low word of outer (sum / D))
  int32_t* Cp = reinterpret_cast<int32_t*>(g.C) + off;
#pragma unroll
  for (int e = 0; e < 4; ++e) w[e] = (int32_t)((uint32_t)(w[e] >> g.log2D) * (uint32_t)g.outer);
  if (g.split > 1) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (e < n) atomicAdd(Cp + e, w[e]);
    return;
  }
  if (g.accumulate) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (e < n) w[e] = (int32_t)((uint32_t)w[e] + (uint32_t)Cp[e]);
  }
  if (n == 4 && (reinterpret_cast<uintptr_t>(Cp) & 15) == 0) {
    __builtin_nontemporal_store(w, reinterpret_cast<v4i*>(Cp));
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (e < n) Cp[e] = w[e];
  }
}

// (ell(p): the fold coefficient of product p)
template <class C, class Ell>
__device__ __forceinline__ void slice_body(const SliceArgs& g, Ell ell, int tile, int part) {
  extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int grp = wave / C::NQ, q = wave % C::NQ, wm = q / C::WN, wn = q % C::WN;
  int tm, tn;
  slice_tile(g, tile, tm, tn);
  // this workgroup's part of the range, then this group's share of its stream
  const int per = (g.items + g.split - 1) / g.split;
  const int i0 = part * per, PP = min(g.items, i0 + per) - i0;  // items per product
  if (PP <= 0) return;
  const int T = g.r * PP;
  const int beg = (int)((int64_t)grp * T / C::WK), count = (int)((int64_t)(grp + 1) * T / C::WK) - beg;
  // Groups whose waves share copies meet at a barrier in every stage, so all of them run the
  // longest share's number of stages (their sums past their own share are never folded).
  const int loops = C::NQ == 1 ? count : (T + C::WK - 1) / C::WK;
  const uint32_t lds0 = (uint32_t)(uintptr_t)smem;
  const uint32_t voff = lane * 16;

  int np, nt, left;  // product and item of the next copies, and how many follow within the share
  {
    const int s = min(beg, T - 1);
    np = s / PP;
    nt = s - np * PP;
    left = count - 1;
  }
  int cp = np, ct = nt;  // product and item being multiplied
  // This wave's copies of an item: copy c is 1 KiB of its group's block (q PER + c) / COPIES, off[c]
  // bytes from the item's first byte of that side (the rows past the planes repeat the last block;
  // the outputs they feed are not stored).
  uint32_t off[C::PER];
#pragma unroll
  for (int c = 0; c < C::PER; ++c) {
    const int id = q * C::PER + c, blk = id / C::COPIES, h = id % C::COPIES;
    const bool sideA = blk < C::AB;
    const int rbs = sideA ? g.rba : g.rbb;
    const int rb = min(sideA ? tm * C::AB + blk : tn * C::BB + blk - C::AB, rbs - 1);
    off[c] = C::FMT == 2 ? (uint32_t)(rb * 3 + h) * kBrickBytes : (uint32_t)(h * rbs + rb) * kBrickBytes;
  }
  const int64_t step_a = (int64_t)g.rba * C::BLOCK_BYTES, step_b = (int64_t)g.rbb * C::BLOCK_BYTES;
  const uint8_t *na, *nb;  // the next item's first byte of either side
  auto product_start = [&](int item) {
    na = g.pa + (int64_t)((g.pidx_a >> (4 * np)) & 15u) * g.stride_a + (int64_t)item * step_a;
    nb = g.pb + (int64_t)((g.pidx_b >> (4 * np)) & 15u) * g.stride_b + (int64_t)item * step_b;
  };
  product_start(g.item0 + i0 + nt);
  auto copy_one = [&](auto cc, int buf) {
    constexpr int c = decltype(cc)::value;
    const int id = q * C::PER + c;
    const uint8_t* src = (id / C::COPIES < C::AB ? na : nb) + off[c];
    dma_brick(src, voff, lds0 + buf * C::STAGE_BYTES + grp * C::ITEM_BYTES + id * kBrickBytes);
  };
  auto copy_next = [&]() {  // the item after the last one copied (the share's last item repeats)
    if (left > 0) {
      --left;
      na += step_a;
      nb += step_b;
      if (++nt == PP) {
        nt = 0;
        ++np;
        product_start(g.item0 + i0);
      }
    }
  };

  v16f acc[C::BMW][C::BNW];
  int32_t iacc[C::BMW][C::BNW][16];
#pragma unroll
  for (int i = 0; i < C::BMW; ++i)
#pragma unroll
    for (int j = 0; j < C::BNW; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        acc[i][j][v] = 0.0f;
        iacc[i][j][v] = 0;
      }

  // The wave's fragments of one item: k-step ks's A blocks, then its B blocks.
  constexpr int NF = C::BMW + C::BNW, NM = C::BMW * C::BNW;
  struct Frags {
    v8i f[2 * NF];
  };
  auto read_one = [&](Frags& fr, auto rc, int buf) {
    constexpr int r = decltype(rc)::value, ks = r / NF, i = r % NF;
    const int blk = i < C::BMW ? wm * C::BMW + i : C::AB + wn * C::BNW + i - C::BMW;
    const uint8_t* s = smem + buf * C::STAGE_BYTES + grp * C::ITEM_BYTES + blk * C::BLOCK_BYTES;
    fr.f[r] = frag_fmt<C::FMT>(s + (C::FMT == 2 ? 0 : ks * kBrickBytes), ks, lane);
  };
  auto multiply_one = [&](const Frags& fr, auto qc) {
    constexpr int ks = decltype(qc)::value / NM, i = decltype(qc)::value % NM / C::BNW, j = decltype(qc)::value % C::BNW;
    if constexpr (C::FMT == 2)
      mfma_block6(acc[i][j], fr.f[ks * NF + i], fr.f[ks * NF + C::BMW + j]);
    else
      mfma_block(acc[i][j], fr.f[ks * NF + i], fr.f[ks * NF + C::BMW + j]);
  };
  // Fold after the item just multiplied (the i-th of the share) if it ends a product, a fold segment
  // or the share.
  int run = 0;
  auto fold = [&](int i) {
    ++run;
    const bool end_p = ct + 1 == PP;
    if (i < count && (end_p || run == g.seg || i + 1 == count)) {
      const int32_t l = ell(cp);
#pragma unroll
      for (int a = 0; a < C::BMW; ++a)
#pragma unroll
        for (int b = 0; b < C::BNW; ++b)
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            iacc[a][b][v] += __mul24(l, (int32_t)acc[a][b][v]);
            acc[a][b][v] = 0.0f;
          }
      run = 0;
    }
    ct = end_p ? 0 : ct + 1;
    cp += end_p ? 1 : 0;
  };

  // Item i sits in buffer i % NST and its fragments are in registers when its MFMAs begin.  Between
  // the first 3/4 of these MFMAs the next item's fragments are read and the copies of item i + NST
  // are issued into item i's buffer, spread so that neither queues up.  Then the wave waits until item
  // i + 2 has landed and its reads are done; where waves share copies, a barrier makes that true of
  // all of them, and the last quarter of the MFMAs covers it.
#pragma unroll
  for (int s = 0; s < C::NST; ++s) {
    static_for<0, C::PER>([&](auto cc) { copy_one(cc, s); });
    copy_next();
  }
  Frags f0, f1;
  wait_vmcnt<(C::NST - 1) * C::PER>();
  if constexpr (C::NQ > 1) block_barrier();
  static_for<0, 2 * NF>([&](auto rc) { read_one(f0, rc, 0); });
  wait_vmcnt<(C::NST - 2) * C::PER>();
  wait_lgkm0();
  if constexpr (C::NQ > 1) block_barrier();
  int buf = 0;
  auto stage = [&](const Frags& cur, Frags& nxt, int i) {
    const int nbuf = buf + 1 == C::NST ? 0 : buf + 1;
    constexpr int BAR = 2 * NM * 3 / 4 > 0 ? 2 * NM * 3 / 4 : 1;  // MFMAs before the wait
    static_for<0, 2 * NM>([&](auto qc) {
      constexpr int q0 = decltype(qc)::value;
      multiply_one(cur, qc);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (q0 < BAR) {
        static_for<q0 * 2 * NF / BAR, (q0 + 1) * 2 * NF / BAR>([&](auto rc) { read_one(nxt, rc, nbuf); });
        static_for<q0 * C::PER / BAR, (q0 + 1) * C::PER / BAR>([&](auto cc) { copy_one(cc, buf); });
      }
      if constexpr (q0 == BAR - 1) {
        wait_vmcnt<(C::NST - 2) * C::PER>();
        wait_lgkm0();
        if constexpr (C::NQ > 1) block_barrier();
      }
      __builtin_amdgcn_sched_barrier(0);
    });
    copy_next();
    buf = nbuf;
    fold(i);
  };
  for (int i = 0; i < loops; i += 2) {
    stage(f0, f1, i);
    if (i + 1 == loops) break;
    stage(f1, f0, i + 1);
  }
  wait_vmcnt<0>();  // the copies past the share's end must land before their buffers are reused
  block_barrier();

  // The groups' sums meet in LDS: wave w writes value v of lane L at word (w NV + v) 64 + L, and the
  // WK waves of one position each add up and store every WK-th group of four values v.  A lane
  // takes four consecutive columns (lanes 4 (lane % 16) .. + 3 of value v).
  int32_t* const sums = reinterpret_cast<int32_t*>(smem);
#pragma unroll
  for (int a = 0; a < C::BMW; ++a)
#pragma unroll
    for (int b = 0; b < C::BNW; ++b)
#pragma unroll
      for (int v = 0; v < 16; ++v) sums[(wave * C::NV + (a * C::BNW + b) * 16 + v) * 64 + lane] = iacc[a][b][v];
  __syncthreads();
  const ModReducer mod(g.modulus ? g.modulus : 1);
  const int L4 = (lane & 15) * 4;
#pragma unroll
  for (int c = 0; c < (C::NV / 4 + C::WK - 1) / C::WK; ++c) {
    const int ch = grp + c * C::WK;
    if (C::NV / 4 % C::WK != 0 && ch >= C::NV / 4) break;
    const int v = ch * 4 + (lane >> 4);
    v4i w = {0, 0, 0, 0};
#pragma unroll
    for (int k = 0; k < C::WK; ++k) w += *reinterpret_cast<const v4i*>(sums + ((k * C::NQ + q) * C::NV + v) * 64 + L4);
    const int blk = v >> 4, vv = v & 15, a = blk / C::BNW, b = blk % C::BNW;
    const int row = tm * C::BM + (wm * C::BMW + a) * 32 + 8 * (vv >> 2) + 4 * (L4 >> 5) + (vv & 3);
    const int col = tn * C::BN + (wn * C::BNW + b) * 32 + (L4 & 31);
    slice_store(g, mod, row, col, w);
  }
}

template <class C>
__global__ __launch_bounds__(C::THREADS, 1) void slice_kernel(SliceArgs g) {
  slice_body<C>(g, [&](int p) { return g.ell[p]; }, blockIdx.x / g.split, blockIdx.x % g.split);
}

// Several GEMMs of one shape in one launch (the residue route's moduli): job j's tiles are workgroups
// j tiles .. j tiles + tiles - 1.
struct SliceJob {
  const uint8_t* pa;
  const uint8_t* pb;
  void* C;
  uint32_t pidx_a, pidx_b;
  int32_t ell[kGroupProducts];
  int32_t r, modulus, seg;
};
struct SliceGroupArgs {
  SliceArgs g;  // the fields all jobs share
  SliceJob job[kMaxModuli];
  int32_t tiles;
};

template <class C>
__global__ __launch_bounds__(C::THREADS, 1) void slice_group_kernel(SliceGroupArgs ga) {
  const int j = blockIdx.x / ga.tiles;
  const SliceJob& jb = ga.job[j];
  SliceArgs g = ga.g;
  g.pa = jb.pa;
  g.pb = jb.pb;
  g.C = jb.C;
  g.pidx_a = jb.pidx_a;
  g.pidx_b = jb.pidx_b;
  g.r = jb.r;
  g.modulus = jb.modulus;
  g.seg = jb.seg;
  static_assert(kGroupProducts == 4, "the fold coefficients below");
  const int32_t l0 = jb.ell[0], l1 = jb.ell[1], l2 = jb.ell[2], l3 = jb.ell[3];
  slice_body<C>(g, [=](int p) { return p == 0 ? l0 : p == 1 ? l1 : p == 2 ? l2 : l3; }, blockIdx.x - j * ga.tiles, 0);
}

// ---------------------------------------------------------------------------
// The whole of Alg. 1 in one kernel, for products so small that launches and the trip of the planes
// through memory are their time: a workgroup encodes its 32 rows of A and 32 columns of B into LDS in
// the stored plane layout, one brick per wave (W waves: W / 2 k-steps of either side), and its waves
// share out the products and k-steps; their int32 sums meet in LDS as above.  Every tile encodes its
// own operands, about 2 us of the kernel, so it serves reductions of one brick per wave and outputs of
// one round of tiles: with a second chunk of the reduction (512^3 on 8 waves) it took 11.4 us
// against 10.3 for encoder and GEMM, and at 1024^2 x 256, four rounds, 24.5 against 13.2.  AWE6 256^3:
// 7.2 us against 10.0, 512^2 x 256 7.4 against 9.6, {0, +-1} x INT8 700 x 300 x 200 8.9 against 11.3.
// E2M3 planes, slower to pack, gain nothing (9.2 against 9.1 at 256^3).
// ---------------------------------------------------------------------------
constexpr int kDirectPlanes = 12;  // planes of both sides whose bricks fit the LDS (16 waves: 96 KiB)
struct DirectArgs {
  EncodeArgs a, b;
  LutArg lut_a, lut_b;
  SliceArgs g;
};

// LDS: the planes of both sides (or, at the end, the sums), the B side's transpose tiles, the tables.
constexpr int direct_plane_bytes(int W) { return W / 2 * kBrickBytes; }
constexpr int direct_sum_bytes(int W) { return W * 16 * 64 * 4; }
inline int direct_lds(int W, int planes) {
  return std::max(planes * direct_plane_bytes(W), direct_sum_bytes(W)) + W / 2 * 32 * kTileCol + 2 * 256 * 4;
}

template <int W>
__global__ __launch_bounds__(64 * W) void direct_kernel(DirectArgs d) {
  extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
  const SliceArgs& g = d.g;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  constexpr int KST = W / 2, PB = direct_plane_bytes(W);
  const int plane_bytes = max((d.a.nplanes + d.b.nplanes) * PB, direct_sum_bytes(W));
  uint32_t* const luts = reinterpret_cast<uint32_t*>(smem + plane_bytes + KST * 32 * kTileCol);
  if (threadIdx.x < 512) luts[threadIdx.x] = threadIdx.x < 256 ? d.lut_a.v[threadIdx.x] : d.lut_b.v[threadIdx.x - 256];
  int tm, tn;
  slice_tile(g, blockIdx.x, tm, tn);
  __syncthreads();
  {
    const bool side_a = wave < KST;
    const int i = side_a ? wave : wave - KST;  // the k-step this wave encodes
    const int np = side_a ? d.a.nplanes : d.b.nplanes;
    uint8_t* const mine = smem + (side_a ? 0 : d.a.nplanes * PB) + i * kBrickBytes + lane * 16;
    uint32_t e[32], w[8][4];
    if (side_a)
      brick_codes<false>(d.a, tm, i, luts, nullptr, e);
    else
      brick_codes<true>(d.b, tn, i, luts + 256, smem + plane_bytes + i * (32 * kTileCol), e);
    uint32_t bad = 0;
#pragma unroll
    for (int j = 0; j < 32; ++j) bad |= e[j];
    if ((bad & kLutInvalid) && d.a.flag != nullptr) atomicOr(d.a.flag, 1);
    pack_e2m1_planes<8>(e, w);
#pragma unroll
    for (int p = 0; p < 8; ++p) {
      if (p >= np) break;
      *reinterpret_cast<uint4*>(mine + p * PB) = make_uint4(w[p][0], w[p][1], w[p][2], w[p][3]);
    }
  }
  __syncthreads();
  // this wave's share of the (product, k-step) units
  const int steps = (int)d.a.KS, U = g.r * steps, u1 = (wave + 1) * U / W;
  int32_t iacc[16];
#pragma unroll
  for (int v = 0; v < 16; ++v) iacc[v] = 0;
  for (int u = wave * U / W; u < u1;) {
    const int p = u / steps, k0 = u - p * steps, n = min(u1, (p + 1) * steps) - u;
    const uint8_t* fa = smem + (int)((g.pidx_a >> (4 * p)) & 15u) * PB + k0 * kBrickBytes + lane * 16;
    const uint8_t* fb = smem + (d.a.nplanes + (int)((g.pidx_b >> (4 * p)) & 15u)) * PB + k0 * kBrickBytes + lane * 16;
    v16f acc = {0.0f};
    for (int i = 0; i < n; ++i) mfma_block(acc, frag(fa + i * kBrickBytes), frag(fb + i * kBrickBytes));
    u += n;
    const int32_t l = g.ell[p];
#pragma unroll
    for (int v = 0; v < 16; ++v) iacc[v] += __mul24(l, (int32_t)acc[v]);
  }
  __syncthreads();
  int32_t* const sums = reinterpret_cast<int32_t*>(smem);
#pragma unroll
  for (int v = 0; v < 16; ++v) sums[(wave * 16 + v) * 64 + lane] = iacc[v];
  __syncthreads();
  if (wave >= 4) return;
  const ModReducer mod(g.modulus ? g.modulus : 1);
  const int L4 = (lane & 15) * 4, v = wave * 4 + (lane >> 4);
  v4i t = {0, 0, 0, 0};
#pragma unroll
  for (int k = 0; k < W; ++k) t += *reinterpret_cast<const v4i*>(sums + (k * 16 + v) * 64 + L4);
  slice_store(g, mod, tm * 32 + 8 * (v >> 2) + 4 * (L4 >> 5) + (v & 3), tn * 32 + (L4 & 31), t);
}

// Zeroes C before the parts of split tiles add into it, as words of 4 bytes: row_words per row,
// rows ld_words apart.
__global__ __launch_bounds__(256) void zero_kernel(uint32_t* C, int32_t rows, int64_t row_words, int64_t ld_words) {
  const int64_t total = rows * row_words;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = i / row_words;
    C[r * ld_words + (i - r * row_words)] = 0;
  }
}

template <class C>
awe_status launch_slices(SliceArgs& g, int split, hipStream_t stream) {
  g.tiles_m = (g.M + C::BM - 1) / C::BM;
  g.tiles_n = (g.N + C::BN - 1) / C::BN;
  g.split = split;
  const int64_t blocks = (int64_t)g.tiles_m * g.tiles_n * split;
  hipError_t err;
  if (split > 1 && !g.accumulate) {
    const int64_t words = g.c64 ? 2 : 1, total = (int64_t)g.M * g.N * words;
    hipLaunchKernelGGL(zero_kernel, dim3((unsigned)std::min<int64_t>((total + 255) / 256, 2048)), dim3(256), 0, stream,
                       reinterpret_cast<uint32_t*>(g.C), g.M, g.N * words, g.ldc * words);
    err = hipGetLastError();
    if (err != hipSuccess) {
      set_error(std::string("zero launch: ") + hipGetErrorString(err));
      return AWE_ERR_HIP;
    }
  }
  static std::mutex mu;
  static std::set<int> done;
  const awe_status st = set_lds_limit(reinterpret_cast<const void*>(&slice_kernel<C>), C::LDS_BYTES, mu, done);
  if (st != AWE_OK) return st;
  hipLaunchKernelGGL(slice_kernel<C>, dim3((unsigned)blocks), dim3(C::THREADS), C::LDS_BYTES, stream, g);
  err = hipGetLastError();
  if (err != hipSuccess) {
    set_error(std::string("gemm launch: ") + hipGetErrorString(err));
    return AWE_ERR_HIP;
  }
  return AWE_OK;
}

template <class C>
awe_status launch_slice_jobs(SliceGroupArgs& ga, int n, hipStream_t stream) {
  SliceArgs& g = ga.g;
  g.tiles_m = (g.M + C::BM - 1) / C::BM;
  g.tiles_n = (g.N + C::BN - 1) / C::BN;
  g.split = 1;
  ga.tiles = g.tiles_m * g.tiles_n;
  static std::mutex mu;
  static std::set<int> done;
  const awe_status st = set_lds_limit(reinterpret_cast<const void*>(&slice_group_kernel<C>), C::LDS_BYTES, mu, done);
  if (st != AWE_OK) return st;
  hipLaunchKernelGGL(slice_group_kernel<C>, dim3((unsigned)(ga.tiles * n)), dim3(C::THREADS), C::LDS_BYTES, stream, ga);
  const hipError_t err = hipGetLastError();
  if (err != hipSuccess) {
    set_error(std::string("grouped gemm launch: ") + hipGetErrorString(err));
    return AWE_ERR_HIP;
  }
  return AWE_OK;
}

// Blocks per wave, waves over the tile's rows and columns, shares, stages, format.
template <int FMT>
using Slice128 = SliceCfg<2, 2, 2, 2, 2, FMT == 2 ? 3 : 4, FMT>;      // 128 x 128
template <int FMT>
using Slice64x128 = SliceCfg<2, 2, 1, 2, 4, FMT == 2 ? 2 : 3, FMT>;   // 64 x 128
template <int FMT>
using Slice64 = SliceCfg<2, 2, 1, 1, FMT == 2 ? 4 : 8, FMT == 2 ? 3 : 2, FMT>;  // 64 x 64
template <int FMT>
using Slice32 = SliceCfg<1, 1, 1, 1, 8, FMT == 2 ? 3 : 4, FMT>;       // 32 x 32
template <int FMT>
using Slice32x64 = SliceCfg<1, 2, 1, 1, 8, FMT == 2 ? 2 : 3, FMT>;    // 32 x 64
template <int FMT>
using Slice64x32 = SliceCfg<2, 1, 1, 1, 8, FMT == 2 ? 2 : 3, FMT>;    // 64 x 32

template <int FMT>
awe_status launch_variant(int variant, SliceArgs& g, int split, hipStream_t stream) {
  switch (variant) {
    case 1: return launch_slices<Slice128<FMT>>(g, split, stream);
    case 2: return launch_slices<Slice64x128<FMT>>(g, split, stream);
    case 3: return launch_slices<Slice64<FMT>>(g, split, stream);
    case 4: return launch_slices<Slice32<FMT>>(g, split, stream);
    case 5: return launch_slices<Slice32x64<FMT>>(g, split, stream);
    default: return launch_slices<Slice64x32<FMT>>(g, split, stream);
  }
}

void fill_slice_args(const GemmLaunch& L, SliceArgs& g) {
  g.pa = L.planes_a;
  g.pb = L.planes_b;
  g.stride_a = L.stride_a;
  g.stride_b = L.stride_b;
  g.rba = (int32_t)((L.M + kBrickRows - 1) / kBrickRows);
  g.rbb = (int32_t)((L.N + kBrickRows - 1) / kBrickRows);
  g.item0 = (int32_t)(L.k_begin / 128);
  g.items = (int32_t)((std::min(L.k_end, L.K) - L.k_begin + 127) / 128);  // (not the padding's whole items)
  g.seg = (int32_t)(L.flat.k_seg / 128);
  g.r = L.flat.r;
  g.pidx_a = g.pidx_b = 0;
  for (int k = 0; k < L.flat.r; ++k) {
    g.pidx_a |= (uint64_t)(L.flat.pa[k] & 15) << (4 * k);
    g.pidx_b |= (uint64_t)(L.flat.pb[k] & 15) << (4 * k);
    g.ell[k] = L.flat.ell[k];
  }
  g.C = L.C;
  g.ldc = L.ldc;
  g.M = (int32_t)L.M;
  g.N = (int32_t)L.N;
  g.c64 = L.c_u8 && L.modulus ? 2 : (L.c_type == AWE_I64 ? 1 : 0);
  g.accumulate = L.accumulate;
  g.log2D = L.log2D;
  g.modulus = L.modulus;
  g.outer = L.outer;
}

template <int W>
awe_status launch_direct_waves(DirectArgs& d, hipStream_t stream) {
  SliceArgs& g = d.g;
  g.tiles_m = (g.M + 31) / 32;
  g.tiles_n = (g.N + 31) / 32;
  g.split = 1;
  static std::mutex mu;
  static std::set<int> done;
  const awe_status st =
      set_lds_limit(reinterpret_cast<const void*>(&direct_kernel<W>), direct_lds(W, kDirectPlanes), mu, done);
  if (st != AWE_OK) return st;
  hipLaunchKernelGGL(direct_kernel<W>, dim3((unsigned)(g.tiles_m * g.tiles_n)), dim3(64 * W),
                     direct_lds(W, d.a.nplanes + d.b.nplanes), stream, d);
  const hipError_t err = hipGetLastError();
  if (err != hipSuccess) {
    set_error(std::string("direct product launch: ") + hipGetErrorString(err));
    return AWE_ERR_HIP;
  }
  return AWE_OK;
}

// The variants' tiles and times on one MI355X: a tile takes about fixed + per_index * r K microseconds
// (r products, K reduction indices), by format, a round of tiles on all CUs that long, and a launch
// 4 us more.  Fitted to 2048^3, 1024^3, 512^2 x 8192 and 16 x 8192 x 8192 (E2M1) and 2048^3, 1024^3,
// 1024^2 x 4096 and 512 x 8192 x 8192 (E2M3), launched by themselves.  Launches of one graph against
// the estimate (us, variants 1 to 6): AWE6 2048^3 37, 46, 56, 103, 73, 70 / 36, 49, 57, 109, 76, 75; 1024^3
// 19, 14, 10, 18, 13, 12 / 25, 20, 13, 23, 17, 17 (all variants about 5 us less, so their order stands);
// weights in the scales 2048^3 28, 46, 60, 93, 66, 63 / 31, 49, 60, 102, 71, 70.  Over 45 drawn products (E2M1
// and E2M3, GEMM alone) the choice was within 6 % of the best variant or tile configuration in 42 and 8, 10
// and 50 % behind it in the others, the last a reduction of 64 indices, which the model takes for 256.
struct VariantCost {
  int bm, bn;
  double fixed, per_index[2];  // us, ns for E2M1 and E2M3
};
constexpr VariantCost kVariants[] = {
    {128, 128, 9.0, {1.90, 2.15}}, {64, 128, 9.0, {1.10, 1.65}}, {64, 64, 5.5, {0.62, 1.05}},
    {32, 32, 3.0, {0.29, 0.38}},   {32, 64, 4.3, {0.385, 0.50}}, {64, 32, 4.3, {0.375, 0.48}},
};

// A variant's tiles for an M x N output, or 0 for more than 64 rounds of them: past that it is no longer
// the better choice, and its kernel counts tiles and the bytes of row blocks in 32 bits.
int64_t variant_tiles(int variant, int64_t M, int64_t N, int cus) {
  const VariantCost& c = kVariants[variant - 1];
  const int64_t tiles = ((M + c.bm - 1) / c.bm) * ((N + c.bn - 1) / c.bn);
  return tiles <= 64 * (int64_t)cus ? tiles : 0;
}
// AWE_GEMM_SLICE's variant for a launch, where the kernel takes it: 1 .. 6, else 0.
int forced_variant(const char* e, const GemmLaunch& L, int cus) {
  const int v = atoi(e);
  return v >= 1 && v <= 6 && variant_tiles(v, L.M, L.N, cus) ? v : 0;
}

// Whether the environment asks for particular tile configurations or splits.
bool tuning_overrides() {
  for (const char* name : {"AWE_GEMM_CFG", "AWE_GEMM_CFG_E2M3", "AWE_GEMM_CFG_SHARED", "AWE_GEMM_ALLPAIRS",
                           "AWE_GEMM_CUS", "AWE_GEMM_SPLIT", "AWE_GEMM_SLICE"})
    if (tuning(name)) return true;
  return false;
}

}  // namespace

Slice choose_slice(const GemmLaunch& L, int cus, double tile_us) {
  if (L.flat.r == 0) return Slice{0, 1};
  // AWE_GEMM_SLICE: 0 none, 1 .. 6 that variant (AWE_GEMM_SLICE_SPLIT workgroups per tile); the
  // overrides of the tile configurations leave none.  They change no result.
  if (const char* e = tuning("AWE_GEMM_SLICE")) {
    const char* sp = tuning("AWE_GEMM_SLICE_SPLIT");
    const int split = sp && !L.modulus ? atoi(sp) : 1;
    return Slice{forced_variant(e, L, cus), split >= 1 && split <= 64 ? split : 1};
  }
  if (tuning_overrides()) return Slice{0, 1};
  const int64_t len = L.k_end - L.k_begin;
  const double rk = (double)L.flat.r * (double)len, outs = (double)L.M * (double)L.N;
  Slice best{0, 1};
  double best_us = tile_us;
  for (int v = 0; v < 6; ++v) {
    const VariantCost& c = kVariants[v];
    const int64_t tiles = variant_tiles(v + 1, L.M, L.N, cus);
    if (!tiles) continue;
    const double ns = c.per_index[L.fmt == kFmtE2M3 ? 1 : 0];
    const double us = 4.0 + (double)((tiles + cus - 1) / cus) * (c.fixed + ns * 1e-3 * rk);
    if (us < best_us) {
      best_us = us;
      best = Slice{v + 1, 1};
    }
    // S workgroups per tile while they fill one round: C zeroed first, S atomic additions per output
    // (270 per ns in all); at least two items per workgroup and product
    // on average, the padding counted (the last workgroups may have fewer or none)
    for (int s = 2; !L.modulus && s <= 64 && tiles * s <= cus && len >= 256 * s; s *= 2) {
      const double t = 8.0 + c.fixed + ns * 1e-3 * rk / s + s * outs / 270e3;
      if (t < best_us) {
        best_us = t;
        best = Slice{v + 1, s};
      }
    }
  }
  return best;
}

int choose_slice_group(const GemmLaunch* L, int n, int cus, double tile_us) {
  if (const char* e = tuning("AWE_GEMM_SLICE")) return forced_variant(e, L[0], cus);
  if (tuning("AWE_GEMM_CFG")) return 0;
  int best = 0;
  for (int v = 0; v < 6; ++v) {
    const VariantCost& c = kVariants[v];
    const int64_t tiles = variant_tiles(v + 1, L[0].M, L[0].N, cus);
    if (!tiles) continue;
    double sum = 0.0, longest = 0.0;
    for (int j = 0; j < n; ++j) {
      const double t = c.fixed + c.per_index[0] * 1e-3 * (double)L[j].r * (double)(L[j].k_end - L[j].k_begin);
      sum += t;
      longest = std::max(longest, t);
    }
    const double us = group_time(sum, longest, tiles, cus);
    if (us < tile_us) {
      tile_us = us;
      best = v + 1;
    }
  }
  return best;
}

awe_status launch_slice_group(const GemmLaunch* L, const int* order, int n, int variant, hipStream_t stream) {
  SliceGroupArgs ga{};
  fill_slice_args(L[order[0]], ga.g);
  for (int j = 0; j < n; ++j) {
    const GemmLaunch& Lj = L[order[j]];
    SliceJob& jb = ga.job[j];
    jb.pa = Lj.planes_a;
    jb.pb = Lj.planes_b;
    jb.C = Lj.C;
    for (int k = 0; k < Lj.flat.r; ++k) {
      jb.pidx_a |= (uint32_t)(Lj.flat.pa[k] & 15) << (4 * k);
      jb.pidx_b |= (uint32_t)(Lj.flat.pb[k] & 15) << (4 * k);
      jb.ell[k] = Lj.flat.ell[k];
    }
    jb.r = Lj.flat.r;
    jb.modulus = Lj.modulus;
    jb.seg = (int32_t)(Lj.flat.k_seg / 128);
  }
  switch (variant) {
    case 1: return launch_slice_jobs<Slice128<0>>(ga, n, stream);
    case 2: return launch_slice_jobs<Slice64x128<0>>(ga, n, stream);
    case 3: return launch_slice_jobs<Slice64<0>>(ga, n, stream);
    case 4: return launch_slice_jobs<Slice32<0>>(ga, n, stream);
    case 5: return launch_slice_jobs<Slice32x64<0>>(ga, n, stream);
    default: return launch_slice_jobs<Slice64x32<0>>(ga, n, stream);
  }
}

bool choose_direct(const GemmLaunch& L, int cus) {
  const EncodeLaunch* a = L.operands;
  if (!a || !L.from_operands || !a->other || L.flat.r == 0 || L.fmt != kFmtE2M1 || a->wide || a->nplanes8 || a->other->nplanes8 || a->fp6 ||
      a->nplanes + a->other->nplanes > kDirectPlanes)
    return false;
  if (L.k_begin != 0 || L.k_end < L.K || L.accumulate || L.k_end > 512) return false;
  const int64_t tiles = ((L.M + 31) / 32) * ((L.N + 31) / 32);
  if (tiles > 64 * cus) return false;
  if (const char* e = tuning("AWE_GEMM_DIRECT")) return atoi(e) != 0;
  if (tuning_overrides()) return false;
  // (two rounds' worth on 8 waves, whose 60 KiB of LDS let two workgroups share a CU: 1024 x 512 x
  // 256 9.1 us against 10.6)
  return tiles <= (L.k_end <= 256 ? 2 : 1) * cus;
}

awe_status launch_direct(const GemmLaunch& L, hipStream_t stream) {
  DirectArgs d{};
  const EncodeLaunch &a = *L.operands, &b = *a.other;
  encode_args(a, d.a);
  encode_args(b, d.b);
  std::copy(a.lut, a.lut + 256, d.lut_a.v);
  std::copy(b.lut, b.lut + 256, d.lut_b.v);
  fill_slice_args(L, d.g);
  return L.k_end <= 256 ? launch_direct_waves<8>(d, stream) : launch_direct_waves<16>(d, stream);
}

awe_status launch_slice(const GemmLaunch& L, Slice s, hipStream_t stream) {
  SliceArgs g{};
  fill_slice_args(L, g);
  return L.fmt == kFmtE2M3 ? launch_variant<2>(s.variant, g, s.split, stream)
                           : launch_variant<0>(s.variant, g, s.split, stream);
}

}  // namespace awe
