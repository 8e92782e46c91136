// The closed-form pair tests (csrc/closed.h) up to the limits of their 32-bit
// form: array sizes over the whole range, spans up to SMALL_SPAN, thousands of
// threads and blocks.  Where the accesses are few enough they are enumerated,
// sorted by word and joined; elsewhere the 32-bit form and the one for few terms
// are compared with the 64-bit form.  Prints the number of comparisons and of
// differences; args: seed, rounds.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "../paper_2011_08373_amd/csrc/closed.h"

using namespace rp;

struct Pt {
  int32_t a, b, c;
  uint32_t m, r, bm, br;
};
struct Hit {
  uint32_t word, t, k;
};

int main(int argc, char** argv) {
  if (argc < 3) return 2;
  std::mt19937_64 g(std::strtoull(argv[1], nullptr, 10));
  const long rounds = std::atol(argv[2]);
  long compared = 0, conflicts = 0, wrong = 0, joined = 0, few = 0, at_span = 0;
  auto pick = [&](int64_t lo, int64_t hi) { return lo + (int64_t)(g() % (uint64_t)(hi - lo + 1)); };
  auto log_pick = [&](double lo, double hi) {
    const double u = (double)(g() >> 11) / 9007199254740992.0;
    return (int64_t)std::llround(lo * std::pow(hi / lo, u));
  };
  // the device's reduction: values of every size, near multiples and at the ends
  for (long it = 0; it < 4 * rounds; it++) {
    const uint32_t W = (uint32_t)log_pick(3, 4294967295.0);
    int64_t v = (int64_t)g() >> pick(0, 62);
    if (pick(0, 1)) v -= v % (int64_t)W + pick(-2, 2);
    if (pick(0, 999) == 0) v = pick(0, 1) ? INT64_MAX - pick(0, 9) : INT64_MIN + pick(0, 9);
    const int64_t r = v % (int64_t)W, want = r < 0 ? r + (int64_t)W : r;
    if ((int64_t)mod_by_doubles(v, W) != want && wrong++ < 10)
      std::printf("mod_by_doubles(%lld, %u) = %u\n", (long long)v, W, mod_by_doubles(v, W));
  }
  for (long it = 0; it < rounds; it++) {
    uint32_t W = (uint32_t)log_pick(2, (double)SMALL_SIZE);
    if (pick(0, 3) == 0) W = 1u << pick(1, 30);
    const bool join = pick(0, 1);
    const uint32_t T = (uint32_t)log_pick(1, join ? 400 : 1 << 20);
    const uint32_t B = (uint32_t)log_pick(1, join ? 12 : 1 << 14);
    // steps near the largest that SMALL_SPAN takes, or of any size below it
    auto step = [&](uint32_t n, uint32_t m) -> int32_t {
      const int64_t most = std::min<int64_t>((SMALL_SPAN - 1) / std::max<int64_t>(1, (int64_t)n - 1) / m,
                                             W / 2);
      if (most < 1) return 0;
      int64_t s = pick(0, 2) ? log_pick(1, (double)most) : most - pick(0, std::min<int64_t>(most - 1, 3));
      if (pick(0, 7) == 0) s = 0;
      return (int32_t)(pick(0, 1) ? s : -s);
    };
    auto count = [](uint32_t n, uint32_t m, uint32_t r) { return r < n ? (n - 1 - r) / m + 1 : 0u; };
    auto point = [&]() {
      Pt p;
      p.m = pick(0, 2) ? 1 : (uint32_t)pick(1, 5);
      p.r = (uint32_t)pick(0, p.m - 1);
      p.bm = pick(0, 1) ? 1 : (uint32_t)pick(1, 5);
      p.br = (uint32_t)pick(0, p.bm - 1);
      p.a = step(count(T, p.m, p.r), p.m);
      p.b = step(count(B, p.bm, p.br), p.bm);
      p.c = pick(0, 2) ? (int32_t)pick(-9, 9) : (int32_t)g();
      return p;
    };
    const Pt p = point();
    Pt q = pick(0, 5) == 0 ? p : point();
    if (pick(0, 2) == 0) { q.b = p.b; q.bm = p.bm; q.br = p.br; }
    if (pick(0, 3) == 0) { q.a = p.a; q.m = p.m; q.r = p.r; }
    const uint32_t xp = count(T, p.m, p.r), xq = count(T, q.m, q.r);
    if (!xp || !xq || !count(B, p.bm, p.br) || !count(B, q.bm, q.br)) continue;
    const Access x = make_access(p.a, p.b, p.c, W, p.m, p.r, xp, p.bm, p.br, B);
    const Access y = make_access(q.a, q.b, q.c, W, q.m, q.r, xq, q.bm, q.br, B);
    bool small = true;
    for (const Access* s : {&x, &y}) {
      const int64_t sp = std::llabs(s->A) * (int64_t)(s->X - 1);
      small = small && sp < SMALL_SPAN && std::llabs(s->S) * (int64_t)(s->Z - 1) < SMALL_SPAN;
      at_span += sp > SMALL_SPAN / 2;
    }
    if (!small) continue;
    // (walks of many values take too long)
    const PairEq<int64_t> bl(blocks_of(y), blocks_of(x), true), eq(threads_of(x), threads_of(y), true);
    const uint64_t n = bl.g == 0 ? 1 : (uint64_t)(bl.w / bl.g) + 1, wraps = (uint64_t)eq.w / W + 1;
    const bool by_g = n <= (uint64_t)x.Z * y.Z;
    if (std::max<uint64_t>(B, by_g ? n : (uint64_t)x.Z * y.Z) * wraps > 20000) continue;
    auto check = [&](const char* what, bool got, bool want) {
      compared++;
      conflicts += want;
      if (got == want) return;
      if (wrong++ < 10)
        std::printf("%s: %d instead of %d: W=%u T=%u B=%u p=(%d,%d,%d m%u r%u bm%u br%u) "
                    "q=(%d,%d,%d m%u r%u bm%u br%u)\n", what, got, want, W, T, B, p.a, p.b, p.c, p.m,
                    p.r, p.bm, p.br, q.a, q.b, q.c, q.m, q.r, q.bm, q.br);
    };
    bool same = pair_same_block<int64_t>(x, y, B), cross = pair_cross_block<int64_t>(x, y);
    if (join) {
      joined++;
      auto hits = [&](const Pt& s) {
        std::vector<Hit> v;
        for (uint32_t k = s.br; k < B; k += s.bm)
          for (uint32_t t = s.r; t < T; t += s.m) {
            const __int128 e = (__int128)s.a * t + (__int128)s.b * k + s.c, w = e % (__int128)W;
            v.push_back(Hit{(uint32_t)(w < 0 ? w + W : w), t, k});
          }
        std::sort(v.begin(), v.end(), [](const Hit& f, const Hit& h) { return f.word < h.word; });
        return v;
      };
      const std::vector<Hit> u = hits(p), v = hits(q);
      bool es = false, ec = false, self = false;
      size_t b = 0;
      for (size_t a = 0; a < u.size() && !(es && ec); a++) {
        while (b < v.size() && v[b].word < u[a].word) b++;
        for (size_t e = b; e < v.size() && v[e].word == u[a].word && !(es && ec); e++) {
          ec |= u[a].k != v[e].k;
          es |= u[a].k == v[e].k && u[a].t != v[e].t;
        }
      }
      std::vector<std::pair<uint64_t, uint32_t>> w;
      for (const Hit& h : u) w.push_back({(uint64_t)h.word << 32 | h.k, h.t});
      std::sort(w.begin(), w.end());
      for (size_t a = 1; a < w.size(); a++) self |= w[a].first == w[a - 1].first;
      check("self", self_same_block(x), self);
      check("same block, 64 bits", same, es);
      check("different blocks, 64 bits", cross, ec);
      same = es;
      cross = ec;
    }
    check("same block, 32 bits", pair_same_block<int32_t>(x, y, B), same);
    check("different blocks, 32 bits", pair_cross_block<int32_t>(x, y), cross);
    if (by_g) {
      few++;
      check("different blocks, few terms", pair_cross_block<int32_t, true>(x, y), cross);
    }
  }
  std::printf("%ld comparisons, %ld conflicts, %ld wrong, %ld joined, %ld few terms, %ld near the span\n",
              compared, conflicts, wrong, joined, few, at_span);
  return wrong != 0;
}
