// Whether two access points conflict, decided from their affine addresses
// alone (plain C++, used by the device kernels and the host plan).
//
// A point's accesses are the words (a*t + b*k + c) mod W over its executing
// threads t = r + m*x, x in [0, X), and executing blocks k = br + bm*z,
// z in [0, Z).  Points p and q touch one word from thread x of p and thread
// y of q exactly when
//     A_p*x - A_q*y  =  D  (mod W),        A = a*m,
// where D depends on the two blocks only.  Two races are asked about:
//   same block       the blocks are equal and the two threads differ;
//   different blocks the blocks differ and the threads are free.
// With steps taken as signed residues, A_p*x - A_q*y runs over an interval
// [lo, hi] of integers around 0, so the congruence is one linear equation
// A_p*x - A_q*y = e over a box for each integer e = D mod W inside it
// (usually one or none).  The solutions of such an equation lie on a line
// of the box whose end points come from one modular inverse and two
// divisions; along the line the difference of the two thread ids is affine,
// so a solution with different threads exists exactly when one of the two end
// points has different threads.  Over the blocks (for different blocks, over
// the multiples of the gcd of the two block steps), D is an arithmetic
// progression mod W, walked from one value inside the interval to the next
// (closed_scan).  Every step is exact: no thread or block is left out, whatever
// the strides, guards and array sizes.
#pragma once
#include <stdint.h>

#if defined(__HIPCC__)
#include <hip/hip_runtime.h>
#define RP_HD __host__ __device__ __forceinline__
#else
#define RP_HD inline
#endif

namespace rp {

// One access point over its executing threads and blocks.  Steps are signed
// residues in (-W/2, W/2]; X and Z are at least 1.
struct Access {
  int32_t A, S, b;         // word step per executing thread, per executing block, per block
  uint32_t W;              // words of the array
  uint32_t X, m, r;        // executing threads r + m*x, x < X
  uint32_t Z, bm, br;      // executing blocks br + bm*z, z < Z
  uint32_t base;           // word of the first executing thread, without the block's term
};

// v mod W (W >= 3) with the quotient in double precision, twice: the first leaves
// a few thousand W at most (|v| < 2^63 and the quotient is right to 52 bits), the
// second one W too many or too few.  (A 64-bit integer division is 100
// instructions and a dozen registers on the device, at every place that reduces;
// on the host it is the faster one: planning and filling 1,022 points of arrays
// of 65,537 words 39 us with doubles, 24 without.)
RP_HD uint32_t mod_by_doubles(int64_t v, uint32_t W) {
  const double inv = 1.0 / (double)W;
  int64_t r = (int64_t)((uint64_t)v - (uint64_t)(int64_t)((double)v * inv) * (uint64_t)W);
  r -= (int64_t)((double)r * inv) * (int64_t)W;
  if (r < 0) r += (int64_t)W;
  if (r >= (int64_t)W) r -= (int64_t)W;
  return (uint32_t)r;
}
RP_HD uint32_t word_mod(int64_t v, uint32_t W) {
  if ((W & (W - 1)) == 0) return (uint32_t)(uint64_t)v & (W - 1);
  if (v >= 0 && v < (int64_t)W) return (uint32_t)v;
  if (v < 0 && v >= -(int64_t)W) return (uint32_t)(v + (int64_t)W);
#if defined(__HIP_DEVICE_COMPILE__)
  return mod_by_doubles(v, W);
#else
  const int64_t r = v % (int64_t)W;
  return (uint32_t)(r < 0 ? r + (int64_t)W : r);
#endif
}
RP_HD int32_t step_mod(int64_t v, uint32_t W) {
  const uint32_t r = word_mod(v, W);
  return r > W / 2 ? (int32_t)((int64_t)r - (int64_t)W) : (int32_t)r;
}

// Blocks and threads: t % m == r over t < T (cnt of them, at least one), k %
// bm == br over k < B (at least one).
RP_HD Access make_access(int32_t a, int32_t b, int32_t c, uint32_t W, uint32_t m, uint32_t r,
                         uint32_t cnt, uint32_t bm, uint32_t br, uint32_t B) {
  Access s;
  const int32_t as = step_mod(a, W);
  s.W = W;
  s.b = step_mod(b, W);
  s.A = step_mod((int64_t)as * (int64_t)m, W);
  s.S = step_mod((int64_t)s.b * (int64_t)bm, W);
  s.X = cnt;
  s.m = m;
  s.r = r;
  s.bm = bm;
  s.br = br;
  s.Z = bm == 1 ? B : (B - 1 - br) / bm + 1;
  s.base = word_mod((int64_t)as * (int64_t)r + (int64_t)c, W);
  return s;
}

template <class I>
RP_HD I abs_of(I v) { return v < 0 ? -v : v; }

template <class I>
struct Unsigned;
template <>
struct Unsigned<int32_t> { using type = uint32_t; };
template <>
struct Unsigned<int64_t> { using type = uint64_t; };

// Division by a fixed d > 0, rounded down.  In 32 bits by a reciprocal in
// double precision: for a numerator |x| < 2^31, x + 1/2 is at least 1/2 from
// every multiple of d, 2^-32 of x, and the reciprocal is right to 48 bits (for
// every d on the device: |1 - d * inv| is at most 2^-48.6).
// (An integer division is 25 instructions, five of them quarter rate; this is
// four, and four for the reciprocal.)
template <class I>
struct Divisor;
template <>
struct Divisor<int32_t> {
  double inv;
  RP_HD explicit Divisor(int32_t d) {
#if defined(__HIP_DEVICE_COMPILE__)
    const double r = __builtin_amdgcn_rcp((double)d);
    inv = r + r * (1.0 - (double)d * r);
#else
    inv = 1.0 / (double)d;
#endif
  }
  RP_HD int32_t floor(int32_t x) const { return (int32_t)__builtin_floor(((double)x + 0.5) * inv); }
};
template <>
struct Divisor<int64_t> {
  int64_t d;
  RP_HD explicit Divisor(int64_t by) : d(by) {}
  RP_HD int64_t floor(int64_t x) const { return x >= 0 ? x / d : -((d - 1 - x) / d); }
};

template <class I>
RP_HD I gcd_of(I x, I y) {     // x, y >= 0
  while (y != 0) {
    const I t = x % y;
    x = y;
    y = t;
  }
  return x;
}
template <>
RP_HD int32_t gcd_of<int32_t>(int32_t x, int32_t y) {
  while (y != 0) {
    const int32_t t = x - Divisor<int32_t>(y).floor(x) * y;
    x = y;
    y = t;
  }
  return x;
}

// Inverse of p mod n (n >= 2, gcd(p, n) = 1), in [1, n).
template <class I>
RP_HD I inverse_of(I p, I n) {
  I r0 = n, r1 = p - Divisor<I>(n).floor(p) * n;
  I t0 = 0, t1 = 1;
  while (r1 > 1) {
    const I q = Divisor<I>(r1).floor(r0);
    const I r2 = r0 - q * r1, t2 = t0 - q * t1;
    r0 = r1;
    r1 = r2;
    t0 = t1;
    t1 = t2;
  }
  return t1 < 0 ? t1 + n : t1;
}

// a * b mod n for a, b in [0, n)
RP_HD int32_t mul_mod(int32_t a, int32_t b, int32_t n, const Divisor<int32_t>& by) {
  if (n <= 46340) return a * b - by.floor(a * b) * n;
  return (int32_t)((uint64_t)a * (uint64_t)b % (uint64_t)n);
}
RP_HD int64_t mul_mod(int64_t a, int64_t b, int64_t n, const Divisor<int64_t>&) {   // n < 2^32
  return (int64_t)((uint64_t)a * (uint64_t)b % (uint64_t)n);
}

// One side of a two-variable equation: a step, a count and the ids r + m*x of
// the values x in [0, n).
struct Axis {
  int32_t step;
  uint32_t n, m, r;
};
RP_HD Axis threads_of(const Access& s) { return Axis{s.A, s.X, s.m, s.r}; }
RP_HD Axis blocks_of(const Access& s) { return Axis{s.S, s.Z, s.bm, s.br}; }

// The equation A*x - B*y = e over 0 <= x < X, 0 <= y < Y of two axes.
// I = int32_t where the spans |step|*(n-1) of all axes are below 2^28
// (SMALL_SPAN) and the words, threads and blocks at most 2^30 (SMALL_SIZE),
// else int64_t (spans below 2^40).
constexpr int64_t SMALL_SPAN = 1ll << 28, SMALL_SIZE = 1ll << 30, MAX_SPAN = 1ll << 40;

template <class I>
struct PairEq {
  I A, B, X, Y;
  I p, q, g, inv;          // A/g, B/g, g = gcd(A, B) (0 if both are); inverse of p mod |q|
  I m1, r1, m2, r2;        // ids r1 + m1*x and r2 + m2*y
  I lo, w;                 // A_p*x - A_q*y takes values in [lo, lo + w]
  bool off, neg;           // only solutions with different ids; x and y exchanged

  RP_HD PairEq(const Axis& P, const Axis& Q, bool off_diagonal) {
    off = off_diagonal;
    const I Ap = (I)P.step, Aq = (I)Q.step, sp = Ap * (I)(P.n - 1), sq = Aq * (I)(Q.n - 1);
    lo = (sp < 0 ? sp : 0) - (sq > 0 ? sq : 0);
    w = (sp > 0 ? sp : 0) - (sq < 0 ? sq : 0) - lo;
    // the unknown with the smaller step last: its inverse is the cheap one
    neg = abs_of(Ap) < abs_of(Aq);
    A = neg ? Aq : Ap;
    B = neg ? Ap : Aq;
    X = (I)(neg ? Q.n : P.n);
    Y = (I)(neg ? P.n : Q.n);
    m1 = (I)(neg ? Q.m : P.m);
    r1 = (I)(neg ? Q.r : P.r);
    m2 = (I)(neg ? P.m : Q.m);
    r2 = (I)(neg ? P.r : Q.r);
    p = A;
    q = B;
    inv = 0;
    if (B == 0) {
      g = abs_of(A);
    } else {
      g = 1;
      if (abs_of(B) > 1) {
        g = gcd_of(abs_of(A), abs_of(B));
        const Divisor<I> by(g);
        p = by.floor(A);
        q = by.floor(B);
      }
      const I n = abs_of(q);
      inv = n == 1 ? 0 : n == 2 ? 1 : inverse_of(p, n);
    }
  }

  RP_HD bool differ(I x, I y) const { return r1 + m1 * x != r2 + m2 * y; }

  // some solution of A_p*x - A_q*y = e (with different ids if off)
  RP_HD bool hit(I e) const {
    if (neg) e = -e;
    if (B == 0) {
      if (A == 0) return e == 0 && (!off || X > 1 || Y > 1 || differ(0, 0));
      I x = Divisor<I>(abs_of(A)).floor(e);
      if (x * abs_of(A) != e) return false;
      if (A < 0) x = -x;
      return x >= 0 && x < X && (!off || Y > 1 || differ(x, 0));
    }
    I f = e;
    if (g > 1) {
      f = Divisor<I>(g).floor(e);
      if (f * g != e) return false;
    }
    // x = x0 + n*t, y = y0 + s*t
    const I n = abs_of(q), s = q < 0 ? -p : p;
    I x0 = 0, y0 = -f, t0 = 0, t1 = X - 1;
    if (n > 1) {
      const Divisor<I> by(n);
      const I fm = f - by.floor(f) * n;
      x0 = n == 2 ? fm : mul_mod(fm, inv, n, by);
      if (x0 >= X) return false;
      y0 = by.floor(p * x0 - f);
      t1 = by.floor(X - 1 - x0);
    }
    if (q < 0) y0 = -y0;
    const I d = abs_of(s);
    I lo_y, hi_y;                          // steps to the ends of [0, Y) in s's direction
    if (s > 0) {
      if (y0 >= Y) return false;
      lo_y = -y0;
      hi_y = Y - 1 - y0;
    } else {
      if (y0 < 0) return false;
      lo_y = y0 - Y + 1;
      hi_y = y0;
    }
    if (d == 1) {
      if (lo_y > 0) t0 = lo_y;
      if (hi_y < t1) t1 = hi_y;
    } else {
      const Divisor<I> by(d);
      if (lo_y > 0) t0 = by.floor(lo_y - 1) + 1;
      const I ty = by.floor(hi_y);
      if (ty < t1) t1 = ty;
    }
    if (t0 > t1) return false;
    if (!off) return true;
    return differ(x0 + n * t0, y0 + s * t0) || differ(x0 + n * t1, y0 + s * t1);
  }
};

RP_HD uint32_t quotient(int32_t x, int32_t d) { return (uint32_t)Divisor<int32_t>(d).floor(x); }
RP_HD uint32_t quotient(int64_t x, int64_t d) { return (uint32_t)x / (uint32_t)d; }   // (below 2^32)

// Some z in [0, n) with ok(z) and a solution for D = D0 + beta*z mod W, where
// v0 = (D0 - lo) mod W.  Values of D outside the interval are stepped over.
template <class I, class F>
RP_HD bool closed_scan(const PairEq<I>& q, uint32_t W, uint32_t v0, int32_t beta, uint64_t terms,
                       F ok) {
  using U = typename Unsigned<I>::type;
  const I w = q.w, Wl = (I)W;
  const U n = (U)terms;
  I v = (I)v0;
  U z = 0;
  if (beta == 0 && v > w) return false;
  while (z < n) {
    if (v <= w) {
      if (ok(z))
        for (I e = v; e <= w; e += Wl)
          if (q.hit(q.lo + e)) return true;
      z++;
      v += (I)beta;
      if (v >= Wl) v -= Wl;
      if (v < 0) v += Wl;
    } else if (beta > 0) {
      // to the first value past the top of the range
      const uint32_t s = quotient((I)(Wl - v - 1), (I)beta) + 1;
      z += s;
      v = (I)((U)v + (U)s * (U)beta - (U)Wl);       // in [0, beta)
    } else {
      const uint32_t d = (uint32_t)(-(int64_t)beta);
      const uint32_t s = quotient((I)(v - w - 1), (I)d) + 1;
      z += s;
      v = (I)((U)v - (U)s * (U)d);                  // in (w - d, w]
      if (v < 0) v += Wl;
    }
  }
  return false;
}

// A point racing with itself inside a block: two of its threads share a word.
RP_HD bool self_same_block(const Access& p) {
  if (p.X < 2) return false;
  if (p.A == 0) return true;
  const uint32_t a = (uint32_t)(p.A < 0 ? -(int64_t)p.A : (int64_t)p.A);
  if ((uint64_t)a * (p.X - 1) < p.W) return false;     // (nothing wraps)
  return p.W / gcd_of<uint32_t>(p.W, a) < p.X;
}

// Common blocks of two block conditions: first, first + step, ... below B;
// their number (0: none).
RP_HD uint64_t common_blocks(const Access& p, const Access& q, uint32_t B, uint32_t& first,
                             uint64_t& step) {
  uint64_t k;
  if (p.bm == 1 || q.bm == 1 || p.bm == q.bm) {
    if (p.bm == q.bm && p.br != q.br) return 0;
    step = p.bm > q.bm ? p.bm : q.bm;
    k = p.bm > q.bm ? p.br : q.br;
  } else {
    const uint64_t g = gcd_of<uint64_t>(p.bm, q.bm);
    const int64_t d = (int64_t)q.br - (int64_t)p.br;
    if (d % (int64_t)g != 0) return 0;
    const int64_t n = (int64_t)(q.bm / g);          // k = br_p + bm_p*u, u mod n
    int64_t u = 0;
    if (n > 1) {
      u = (d / (int64_t)g) % n;
      if (u < 0) u += n;
      u = mul_mod(u, inverse_of<int64_t>((int64_t)(p.bm / g), n), n, Divisor<int64_t>(n));
    }
    step = (uint64_t)p.bm * (uint64_t)n;
    k = (uint64_t)p.br + (uint64_t)p.bm * (uint64_t)u;
  }
  if (k >= B) return 0;
  first = (uint32_t)k;
  return (B - 1 - k) / step + 1;
}

// Two threads of one block, one at p and one at q (different points), share a
// word.
template <class I>
RP_HD bool pair_same_block(const Access& p, const Access& q, uint32_t B) {
  uint32_t k;
  uint64_t step;
  const uint64_t n = common_blocks(p, q, B, k, step);
  if (n == 0) return false;
  const uint32_t W = p.W;
  const int64_t db = (int64_t)q.b - (int64_t)p.b;
  const PairEq<I> eq(threads_of(p), threads_of(q), true);
  int32_t dw = 0, beta = 0;
  if (db != 0) {
    const int32_t d = step_mod(db, W);
    if (k != 0) dw = step_mod((int64_t)d * (int64_t)k, W);
    if (n > 1) beta = step_mod((int64_t)d * (int64_t)step, W);
  }
  const uint32_t v0 =
      word_mod((int64_t)q.base - (int64_t)p.base + dw - (int64_t)eq.lo, W);
  return closed_scan(eq, W, v0, beta, beta == 0 ? 1 : n, [](uint64_t) { return true; });
}

// Threads of two different blocks, one at p and one at q (or both at p when
// the points are the same), share a word.  The blocks' part of the word
// difference is itself such an equation, S_q*z - S_p*y = u over the executing
// blocks with different block ids: u runs over the multiples of its gcd, or,
// where those are more than the pairs of blocks, the pairs are taken one by
// one (a few blocks with unrelated strides; FEW_TERMS: never so).
template <class I, bool FEW_TERMS = false>
RP_HD bool pair_cross_block(const Access& p, const Access& q) {
  const uint32_t W = p.W;
  const PairEq<I> eq(threads_of(p), threads_of(q), false);
  const PairEq<I> bl(blocks_of(q), blocks_of(p), true);
  // word difference of the first executing blocks' first threads
  const int64_t d0 = (int64_t)q.base - (int64_t)p.base +
                     (q.br ? (int64_t)step_mod((int64_t)q.b * (int64_t)q.br, W) : 0) -
                     (p.br ? (int64_t)step_mod((int64_t)p.b * (int64_t)p.br, W) : 0);
  const uint64_t n = bl.g == 0 ? 1 : (uint64_t)(bl.w / bl.g) + 1;
  if (FEW_TERMS || n <= (uint64_t)p.Z * q.Z)
    return closed_scan(eq, W, word_mod(d0 + (int64_t)bl.lo - (int64_t)eq.lo, W),
                       bl.g == 0 ? 0 : step_mod((int64_t)bl.g, W), n,
                       [&](uint64_t u) { return bl.hit(bl.lo + bl.g * (I)u); });
  // every block of the point with fewer, against the other's (here neither
  // step is 0: the multiples of the other's would be no more than its blocks)
  const bool few = p.Z <= q.Z;
  const Axis o = few ? blocks_of(p) : blocks_of(q), i = few ? blocks_of(q) : blocks_of(p);
  const int32_t so = few ? step_mod(-(int64_t)o.step, W) : o.step;
  const int32_t si = few ? i.step : step_mod(-(int64_t)i.step, W);
  uint32_t v = word_mod(d0 - (int64_t)eq.lo, W);
  for (uint32_t z = 0; z < o.n; z++) {
    const uint64_t k = (uint64_t)o.r + (uint64_t)o.m * z;
    if (closed_scan(eq, W, v, si, i.n,
                    [&](uint64_t u) { return (uint64_t)i.r + (uint64_t)i.m * u != k; }))
      return true;
    v = word_mod((int64_t)v + so, W);
  }
  return false;
}

}  // namespace rp
