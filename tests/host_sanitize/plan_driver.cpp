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
  std::printf("calls %d failures %d\n", calls, failures);
  return failures ? 1 : 0;
}
