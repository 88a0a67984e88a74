// Host-side checks of the encoder's and the small-output kernels' launch shapes (no GPU needed).
#include <cstdint>
#include <cstdio>
#include <initializer_list>

#include "encode_device.h"

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

int main() {
  encoder_grids();
  std::printf("failures %d\n", fails);
  return fails ? 1 : 0;
}
