// Compares the closed-form pair tests (csrc/closed.h) with the definition:
// every thread of every block of two random access points.  Prints the number
// of comparisons and of differences; args: seed, rounds.
#include <cstdio>
#include <cstdlib>
#include <random>

#include "../paper_2011_08373_amd/csrc/closed.h"

using namespace rp;

struct Pt {
  int32_t a, b, c;
  uint32_t m, r, bm, br;
};

int main(int argc, char** argv) {
  if (argc < 3) return 2;
  std::mt19937_64 g(std::strtoull(argv[1], nullptr, 10));
  const long rounds = std::atol(argv[2]);
  long compared = 0, conflicts = 0, wrong = 0;
  auto pick = [&](int64_t lo, int64_t hi) { return lo + (int64_t)(g() % (uint64_t)(hi - lo + 1)); };
  for (long it = 0; it < rounds; it++) {
    // array sizes of every kind: powers of two, odd ones, 1, the largest
    uint32_t W = pick(0, 3) == 0 ? 1u << pick(0, 7) : (uint32_t)pick(1, 90);
    if (pick(0, 30) == 0) W = 0xFFFFFFFFu - (uint32_t)pick(0, 3);
    const uint32_t T = (uint32_t)pick(1, 14), B = (uint32_t)pick(1, 9);
    auto point = [&]() {
      Pt p;
      const int64_t kind = pick(0, 5);
      auto step = [&]() -> int32_t {
        switch (kind) {
          case 0: return (int32_t)pick(-2, 2);
          case 1: return (int32_t)pick(-6, 6);
          case 2: return (int32_t)g();
          case 3: return (int32_t)(pick(0, 1) * T);
          case 4: return (int32_t)pick(-40, 40);
          default: return (int32_t)pick(-1, 2);
        }
      };
      p.a = step();
      p.b = step();
      p.c = pick(0, 4) ? (int32_t)pick(-5, 5) : (int32_t)g();
      if (pick(0, 20) == 0) p.a = INT32_MIN;
      if (pick(0, 20) == 0) p.b = INT32_MAX;
      p.m = pick(0, 2) ? 1 : (uint32_t)pick(1, 5);
      p.r = (uint32_t)pick(0, p.m - 1);
      p.bm = pick(0, 1) ? 1 : (uint32_t)pick(1, 5);
      p.br = (uint32_t)pick(0, p.bm - 1);
      return p;
    };
    const Pt p = point();
    Pt q = pick(0, 4) == 0 ? p : point();
    if (pick(0, 2) == 0) q.b = p.b;
    if (pick(0, 3) == 0) q.a = p.a;
    auto count = [](uint32_t n, uint32_t m, uint32_t r) { return r < n ? (n - 1 - r) / m + 1 : 0u; };
    const uint32_t xp = count(T, p.m, p.r), xq = count(T, q.m, q.r);
    if (!xp || !xq || !count(B, p.bm, p.br) || !count(B, q.bm, q.br)) continue;
    auto word = [&](const Pt& s, uint32_t t, uint32_t k) {
      const __int128 v = (__int128)s.a * t + (__int128)s.b * k + s.c, w = v % (__int128)W;
      return (uint32_t)(w < 0 ? w + W : w);
    };
    bool self = false, same = false, cross = false;
    for (uint32_t k = p.br; k < B; k += p.bm)
      for (uint32_t t = p.r; t < T; t += p.m) {
        for (uint32_t u = p.r; u < t; u += p.m) self |= word(p, t, k) == word(p, u, k);
        for (uint32_t l = q.br; l < B; l += q.bm)
          for (uint32_t u = q.r; u < T; u += q.m)
            if (word(p, t, k) == word(q, u, l)) {
              cross |= k != l;
              same |= k == l && t != u;
            }
      }
    const Access x = make_access(p.a, p.b, p.c, W, p.m, p.r, xp, p.bm, p.br, B);
    const Access y = make_access(q.a, q.b, q.c, W, q.m, q.r, xq, q.bm, q.br, B);
    auto check = [&](const char* what, bool got, bool want) {
      compared++;
      conflicts += want;
      if (got == want) return;
      if (wrong++ < 10)
        std::printf("%s: %d, by enumeration %d: W=%u T=%u B=%u p=(%d,%d,%d m%u r%u bm%u br%u) "
                    "q=(%d,%d,%d m%u r%u bm%u br%u)\n", what, got, want, W, T, B, p.a, p.b, p.c, p.m,
                    p.r, p.bm, p.br, q.a, q.b, q.c, q.m, q.r, q.bm, q.br);
    };
    check("self", self_same_block(x), self);
    check("same block", pair_same_block<int64_t>(x, y, B), same);
    check("different blocks", pair_cross_block<int64_t>(x, y), cross);
    bool small = W <= SMALL_SIZE;
    for (const Access* s : {&x, &y}) {
      small = small && std::llabs(s->A) * (int64_t)(s->X - 1) < SMALL_SPAN;
      small = small && std::llabs(s->S) * (int64_t)(s->Z - 1) < SMALL_SPAN;
    }
    if (!small) continue;
    check("same block, 32 bits", pair_same_block<int32_t>(x, y, B), same);
    check("different blocks, 32 bits", pair_cross_block<int32_t>(x, y), cross);
  }
  std::printf("%ld comparisons, %ld conflicts, %ld wrong\n", compared, conflicts, wrong);
  return wrong != 0;
}
