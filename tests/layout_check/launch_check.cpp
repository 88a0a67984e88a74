// Host-side checks of the encoder's and the small-output kernels' launch shapes (no GPU needed).
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <initializer_list>

#include "awe_small.hip"

// (what the launchers of this translation unit call; they are not run here)
namespace awe {
void set_error(const std::string&) {}
awe_status set_lds_limit(const void*, int, std::mutex&, std::set<int>&) { return AWE_ERR_HIP; }
}  // namespace awe

using namespace awe;

static int fails = 0;
static void check(bool ok, const char* what, long long a, long long b) {
  if (ok) return;
  std::printf("FAIL %s (%lld, %lld)\n", what, a, b);
  ++fails;
}

// A launch takes fewer than 2^32 threads: both operands' workgroups of 256 together.
static void encoder_grids() {
  for (int64_t rows_a : {1ll, 33ll, 8192ll, 65536ll, 1ll << 20, 1ll << 22})
    for (int64_t rows_b : {1ll, 100ll, 65536ll, 1ll << 20, 1ll << 22})
      for (int64_t K : {1ll, 257ll, 16384ll, 65536ll, 1ll << 20})
        for (bool wide : {false, true}) {
          EncodeLaunch a{}, b{};
          a.rows = rows_a;
          b.rows = rows_b;
          a.K = b.K = K;
          b.transposed = true;
          a.wide = b.wide = wide;
          EncodeArgs ea, eb;
          const uint64_t na = encode_args(a, ea), nb = encode_args(b, eb);
          check(na > 0 && nb > 0, "no workgroups", rows_a, K);
          check((na + nb) * 256 < (uint64_t)1 << 32, "threads of the joint encoder", rows_a * K, rows_b * K);
          // (waves walk the bricks past the first of each)
          check(ea.nbricks >= (rows_a + 31) / 32 * ((K + 63) / 64) && eb.nbricks >= (rows_b + 31) / 32 * ((K + 63) / 64),
                "bricks", rows_a, K);
        }
}

// The kernel whose waves split the reduction counts tiles and the bytes of a side's row blocks in 32
// bits: whatever chooses it, a variant is only taken where they fit.
static void slice_tiles() {
  const int cus = 256;
  for (const char* forced : {"", "1", "2", "3", "4", "5", "6"}) {
    if (*forced)
      setenv("AWE_GEMM_SLICE", forced, 1);
    else
      unsetenv("AWE_GEMM_SLICE");
    read_tuning();
    int taken = 0;
    for (int64_t M : {1ll, 300ll, 8192ll, 1ll << 20, 1ll << 24, 1ll << 27, 0x7fffff00ll})
      for (int64_t N : {1ll, 300ll, 8192ll, 1ll << 20, 1ll << 24, 0x7fffff00ll}) {
        GemmLaunch L{};
        L.M = M;
        L.N = N;
        L.K = 512;
        L.k_end = 512;
        L.r = L.flat.r = 6;
        L.flat.k_seg = 512;
        L.modulus = 89;
        const Slice s = choose_slice(L, cus, 1e30);
        const int group = choose_slice_group(&L, 1, cus, 1e30);
        for (int v : {s.variant, group}) {
          if (v == 0) continue;
          ++taken;
          const VariantCost& c = kVariants[v - 1];
          const int64_t tiles = ((M + c.bm - 1) / c.bm) * ((N + c.bn - 1) / c.bn) * s.split;
          check(tiles * kMaxModuli <= 0x7fffffff, "tiles", M, N);
          check(((M > N ? M : N) + 31) / 32 * 3 * kBrickBytes < (int64_t)1 << 32, "row blocks", M, N);
        }
      }
    check(taken >= 8, "variants taken where they fit", atoi(forced), taken);
  }
}

int main() {
  encoder_grids();
  slice_tiles();
  std::printf("failures %d\n", fails);
  return fails ? 1 : 0;
}
