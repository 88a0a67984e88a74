// What the product launches of awe_gemm_exact, awe_gemm_exact_noalloc and awe_gemm_mod may do, as the
// launcher sees it: which of them brings the operands, and which may multiply straight from them.
// Built by tests/test_host_sanitizers.py; the device launchers are stubs.
#include <cstdio>
#include <vector>

#include "awe_internal.h"

namespace awe {
extern void (*g_on_gemm)(const GemmLaunch&);
}

static int failures = 0;
static void check(bool ok, const char* what, int enc, long long k) {
  if (ok) return;
  std::printf("FAIL %s (encoding %d, K %lld)\n", what, enc, k);
  ++failures;
}

struct Seen {
  bool operands, from_operands;
};
static std::vector<Seen> seen;
static void on_gemm(const awe::GemmLaunch& L) { seen.push_back(Seen{L.operands != nullptr, L.from_operands}); }

int main() {
  awe::g_on_gemm = on_gemm;
  auto at = [](size_t a) { return reinterpret_cast<void*>(a); };  // never dereferenced
  void *A = at(0x10000000), *B = at(0x20000000), *C = at(0x30000000), *ws = at(0x1000000000);
  const size_t ws_n = (size_t)1 << 40;
  int calls = 0;

  // The operands come with the first launch alone, and a product of several launches (launch groups,
  // reduction ranges) never multiplies straight from them: its later launches read the planes.
  for (int enc = 0; enc <= 12; ++enc)
    for (int64_t K : {1, 64, 300, 512, 300000}) {
      if (enc == AWE_ENC_MOD) continue;
      seen.clear();
      if (awe_gemm_exact((awe_encoding)enc, 40, 50, K, A, K, B, 50, C, 50, AWE_I64, ws, ws_n, nullptr, nullptr) != AWE_OK)
        continue;
      ++calls;
      check(!seen.empty(), "a product without launches", enc, K);
      for (size_t i = 0; i < seen.size(); ++i) {
        check(seen[i].operands == (i == 0), "operands with the first launch", enc, K);
        check(seen[i].from_operands == (seen.size() == 1), "planes left out only by a whole product", enc, K);
      }
    }

  // Nor does a product whose C shares memory with an operand: its tiles would be stored while others
  // still read.  A: 100 x 40 bytes, rows 48 apart, [0, 4792); B: 40 x 100, rows 112 apart, [0, 4468); C:
  // 100 x 100 int32, rows 400 apart, [0, 40000), int64 twice that.
  for (int64_t d : {-90000, -80000, -79999, -40000, -39999, -4792, -4468, -4467, -1, 0, 1, 4467, 4468, 4791, 4792, 90000})
    for (int side = 0; side < 2; ++side)
      for (awe_dtype t : {AWE_I32, AWE_I64}) {
        void* X = at(0x30000000 + d);  // that operand's distance from C
        const int64_t c_end = t == AWE_I64 ? 80000 : 40000, x_len = side ? 39 * 112 + 100 : 99 * 48 + 40;
        const bool apart = d >= c_end || d + x_len <= 0;
        seen.clear();
        if (awe_gemm_exact(AWE_ENC_AWE6, 100, 100, 40, side ? A : X, 48, side ? X : B, 112, C, 100, t, ws, ws_n, nullptr,
                           nullptr) != AWE_OK)
          return 1;
        ++calls;
        check(seen.size() == 1 && seen[0].operands && seen[0].from_operands == apart, "operand and C in one memory",
              side, d);
      }
  // residues (bytes and int32), and the last byte of a leading dimension past the row
  for (int64_t d : {-99 * 48 - 41, -99 * 48 - 40, -99 * 48 - 39, 39999, 40000}) {
    seen.clear();
    if (awe_gemm_mod(89, 100, 100, 40, (const uint8_t*)at(0x30000000 + d), 48, (const uint8_t*)B, 112, (int32_t*)C, 100, ws,
                     ws_n, nullptr, nullptr) != AWE_OK)
      return 1;
    ++calls;
    check(seen.size() == 1 && seen[0].from_operands == (d >= 40000 || d + 99 * 48 + 40 <= 0), "residues and C in one memory",
          AWE_ENC_MOD, d);
  }
  std::printf("calls %d failures %d\n", calls, failures);
  return failures ? 1 : 0;
}
