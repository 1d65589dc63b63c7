// The library's corrected quotient against the division, over random bit patterns
// of both operands and the edges of their ranges; prints the first difference that
// is not allowed.
#define __host__
#define __device__
#define __forceinline__ inline
#include "../paper_1811_04141_amd/csrc/mkf_quotient.hpp"

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <limits>

static uint32_t bits(float v) { uint32_t u; std::memcpy(&u, &v, 4); return u; }
static float value(uint32_t u) { float v; std::memcpy(&v, &u, 4); return v; }

static long n_ulp = 0, n_equal = 0;

static bool same(float a, float v) {
  const float d = sqrtf(v), want = a / d, got = mkf::over(a, d, 1.f / d);
  if (bits(got) == bits(want) || (std::isnan(got) && std::isnan(want))) return ++n_equal, true;
  if (got == 0.f && want == 0.f && bits(a) == 0x80000000u) return true;
  if (std::fabs(a) < 1e-30f && std::llabs((long long)bits(got) - (long long)bits(want)) == 1)
    return ++n_ulp, true;
  std::printf("a %a d %a: %a, division %a\n", a, d, got, want);
  return false;
}

int main(int argc, char **argv) {
  const long n = argc > 1 ? std::atol(argv[1]) : 1000000;
  const float inf = std::numeric_limits<float>::infinity();
  const float as[] = {0.f, -0.f, 0x1p-149f, -0x1p-149f, 0x1.fffffcp-127f, 0x1p-126f, 9.99e-31f, 1e-30f,
                      0x1.fffffep-1f, 1.f, -1.f, 0x1.000002p0f, 3.f, 0x1.fffffep127f,
                      -0x1.fffffep127f, inf, -inf, std::numeric_limits<float>::quiet_NaN()};
  const float vs[] = {0x1p-149f, 0x1.fffffcp-127f, 0x1p-126f, 0x1.fffffep-126f, 0x1.fffffep-1f, 1.f,
                      0x1.000002p0f, 2.f, 3.f, 0x1.fffffep127f, inf};
  for (float a : as)
    for (float v : vs)
      if (!same(a, v)) return 1;
  uint64_t s = 88172645463325252ull;
  auto next = [&]() {  // xorshift64
    s ^= s << 13;
    s ^= s >> 7;
    s ^= s << 17;
    return (uint32_t)(s >> 32);
  };
  for (long i = 0; i < n; ++i) {
    // any float; any positive float, every fourth near a power of two
    const float a = value(next());
    uint32_t v = next() & 0x7FFFFFFFu;
    if (i % 4 == 0) v = (v & 0x7F800000u) | (v & 0xFu) | (i % 8 ? 0x7FFFF0u : 0u);
    if (v == 0u || v > 0x7F800000u) continue;
    if (!same(a, value(v))) return 1;
  }
  std::printf("equal %ld, one ulp %ld\n", n_equal, n_ulp);
  return 0;
}
