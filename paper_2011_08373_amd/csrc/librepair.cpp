// librepair host side: descriptor validation and the per-kernel plan (field
// widths of the packed records, executing-thread counts, barrier tables).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cmath>
#include <cstring>
#include <vector>

#include "closed.h"
#include "common.h"
#include "launch.h"
#include "plan.h"

namespace rp {

static int g_digit_bits = 0;          // 0 = automatic
static int g_timing = 1;              // RP_TUNE_TIMING

int timing_level(int v, bool set) {
  const int old = g_timing;
  if (set) g_timing = v;
  return old;
}

static int g_digit_order = 1;         // RP_TUNE_DIGIT_ORDER

int digit_order(int v, bool set) {
  const int old = g_digit_order;
  if (set) g_digit_order = v;
  return old;
}

static int g_race_route = 0;          // RP_TUNE_RACE_ROUTE

int race_route(int v, bool set) {
  const int old = g_race_route;
  if (set) g_race_route = v;
  return old;
}

static int g_nodes_log2 = 28;         // RP_TUNE_SOLVER_NODES

int solver_nodes_log2(int v, bool set) {
  const int old = g_nodes_log2;
  if (set) g_nodes_log2 = v;
  return old;
}

int job_error_status(const JobState& st) {
  if (st.err == ERR_PHI_CAP || st.err == ERR_SCRATCH) return RP_ERR_CAPACITY;
  if (st.err == ERR_NODES) return RP_ERR_SEARCH;
  return RP_ERR_DEVICE;
}

int g_digit_bits_ref(int v, bool set) {
  const int old = g_digit_bits;
  if (set) g_digit_bits = v;
  return old;
}

static uint32_t bits_for(uint64_t maxval) {   // bits to hold 0..maxval
  return maxval == 0 ? 0u : (uint32_t)(64 - __builtin_clzll(maxval));
}

int validate_kernel(const rp_kernel* k) {
  if (!k) return RP_ERR_INVALID;
  if (k->blocks < 1 || k->threads < 1) return RP_ERR_INVALID;
  if (k->n_slots > 64 || k->n_points > (uint32_t)MAX_POINTS) return RP_ERR_INVALID;
  if ((k->n_arrays && !k->arrays) || (k->n_guards && !k->guards) ||
      (k->n_points && !k->points) || (k->n_slots && !k->slots))
    return RP_ERR_INVALID;
  uint64_t maxw = 1;
  for (uint32_t a = 0; a < k->n_arrays; a++) {
    if (k->arrays[a].words < 1 || k->arrays[a].space > 1) return RP_ERR_INVALID;
    maxw = std::max<uint64_t>(maxw, k->arrays[a].words);
  }
  bool bguard = false;
  for (uint32_t g = 0; g < k->n_guards; g++) {
    if (k->guards[g].m < 1 || k->guards[g].r >= k->guards[g].m) return RP_ERR_INVALID;
    if (k->block_guards) {
      if (k->block_guards[g].m < 1 || k->block_guards[g].r >= k->block_guards[g].m)
        return RP_ERR_INVALID;
      bguard |= k->block_guards[g].m > 1;
    }
  }
  for (uint32_t s = 0; s < k->n_slots; s++)
    if (k->slots[s].level > 1 || k->slots[s].preexisting > 1 || k->slots[s].weight < 1)
      return RP_ERR_INVALID;
  int32_t slot_guard[64];
  for (int s = 0; s < 64; s++) slot_guard[s] = -1;
  uint32_t next = 0;
  for (uint32_t i = 0; i < k->n_points; i++) {
    const rp_point& p = k->points[i];
    if (p.kind > RP_NOP) return RP_ERR_INVALID;
    if (p.kind == RP_ACCESS) {
      if (p.array >= k->n_arrays || p.guard >= k->n_guards || p.is_write > 1)
        return RP_ERR_INVALID;
    } else if (p.kind == RP_BARRIER) {
      if (p.slot >= k->n_slots || p.guard >= k->n_guards) return RP_ERR_INVALID;
      if (slot_guard[p.slot] < 0) {
        if (p.slot != next) return RP_ERR_INVALID;   // numbered by first occurrence
        next++;
        slot_guard[p.slot] = p.guard;
      } else if (slot_guard[p.slot] != (int32_t)p.guard) {
        return RP_ERR_INVALID;                         // one guard per slot
      }
    }
  }
  if (next != k->n_slots) return RP_ERR_INVALID;     // every slot occurs
  // (block conditions add one array id: the location of the padding records)
  const uint32_t total = bits_for(k->n_arrays ? k->n_arrays - 1 + bguard : 0) + bits_for(maxw - 1) +
                         bits_for(k->blocks - 1) + bits_for(k->n_points ? k->n_points - 1 : 0) +
                         bits_for(k->threads - 1);
  if (total > 64) return RP_ERR_INVALID;
  return RP_OK;
}

// The plan of a kernel is one pass over its points.  The points of one array,
// guard and pair of strides differ in the offset c only, so what depends on
// the rest (executing threads and blocks, records, the arc of words, the
// closed form's steps and spans) is worked out once per such combination and
// looked up by the following points (a small direct-mapped table; programs
// unrolled from loops repeat few combinations).
//
// Word compaction.  The sort only has to group records by location: the
// order of the locations themselves is free.  So each array's words are
// rotated (w -> (w + off) mod words) so that every word its accesses can
// touch lands in [0, span), and the word field of the records is only as
// wide as the largest span: fewer key bits, fewer or narrower radix passes.
// The touched words of a point lie in the arc of the circle of residues from
// the smallest to the largest value of a*t + b*k + c over its executing
// threads and blocks.  The circle is cut into CW_BINS bins, one bit each;
// every bin an arc meets is marked, and the rotation moves the longest run of
// unmarked bins (words no access can touch) to the top of the range.  The
// rotation is folded into each point's c, so record generation is unchanged.
//
// Which arrays are decided in closed form.  The closed form tests pairs of
// points of one array, each over the values of an arithmetic progression that
// fall into an interval (closed_scan); the log sorts every access.  For an
// array with n points, pairs <= n(n+1)/2, and the tests of a pair are bounded
// by how often the progression can enter the interval and how long it can
// stay there: trips = (terms * |step| / W + 1) * (width / |step| + 2), at most
// one per term.  Measured on pairs that never conflict: a test 5 to 11 ps with
// the chip full (2,800 points of 32 threads, one block; 64 such kernels and one)
// and 0.26 to 0.54 us one after another in one lane (0.85 us in 64 bits); a
// record of the log costs 16 ps (31.9 ms for the 2.0G records of the stress
// kernel) and the log's launches alone 0.1 ms, 0.3 ms where one block holds
// all records.  So the closed form is taken where its bound is no larger than
// the log's own work (RECORDS_FREE tests cost no more than the launches), and
// where the tests of one lane in sequence end before the log would (at the
// line, 250 points of 352 threads and 2,048 blocks: 3.2 ms, 3.9 by records).
// Where 64-bit steps share no divisor a test in one lane takes 2 us and a step of
// Euclid's algorithm 0.6 (SLOW_STEP, SLOW_EUCLID; six 64-bit divisions that
// others are spared): 120 points in rows of 289 such tests 0.63 ms, by records
// 0.31; 2,800 points of three related steps, 44 chunks a row, 0.18 ms and 0.34.
//
// A pair's gcd and inverse come on top: 6 ps per step of Euclid's algorithm in
// 32 bits and 8.5 ps in 64 (2,000 and 2,800 points of unrelated steps: 85 and
// 134 ps a pair), EUCLID tests each.  What the bounds of all arrays of a call
// cost with them beyond the arrays' own records has to end before a log's
// launches, which the call would make once (COST_FREE, 0.2 ms); the arrays of
// most cost are left to the records where it does not (choose_routes).  2,800
// points of steps up to 2^25 in 64 bits take 0.52 ms in closed form and 0.34 ms
// by records, 2,000 points of steps up to 2^22 0.17 and 0.3 ms; the 64 kernels
// above 1.28 and 0.33 ms (0.04 and 0.25 alone), 64 of 1,000 points 0.16 and
// 0.26 ms.  128 batched kernels come to 2 to 3M tests, 1,024 to 17M.
namespace {
constexpr uint32_t CW_BINS = 256;
constexpr double RECORDS_FREE = 4.0e6, SERIAL_FREE = 512, SERIAL_RECORDS = 16384;
constexpr double COST_FREE = 4.0e7, EUCLID = 1;
constexpr double SLOW_STEP = 4, SLOW_EUCLID = 1.5;
// for calls with a log, in ps
constexpr double RECORD_PS = 16, TEST_PS = 6, CHAIN_PS = 0.4e6, FIRST_LAUNCH = 10e6, CHAIN_GAIN = 10e6;

// [min, max] of x * (r + m*u) over u in [0, n) (n >= 1); false on overflow
bool lin_range(int64_t x, uint64_t r, uint64_t m, uint64_t n, int64_t& lo, int64_t& hi) {
  int64_t a, b;
  if (r > (uint64_t)INT64_MAX || m * (n - 1) > (uint64_t)INT64_MAX) return false;
  if (__builtin_mul_overflow(x, (int64_t)r, &a)) return false;
  if (__builtin_mul_overflow(x, (int64_t)(m * (n - 1)), &b)) return false;
  int64_t l = 0, h = 0;
  if (__builtin_add_overflow(a, b < 0 ? b : 0, &l)) return false;
  if (__builtin_add_overflow(a, b > 0 ? b : 0, &h)) return false;
  lo = l;
  hi = h;
  return true;
}

// The gcd of x and y, and the steps of Euclid's algorithm to it (n: the most so
// far); their mean where the two are not known.
uint32_t gcd_steps(uint32_t x, uint32_t y, double& n) {
  int k = 0;
  for (; y > 1; k++) {
    const uint32_t t = x % y;
    x = y;
    y = t;
  }
  if (k > n) n = k;
  return y ? 1 : x;
}
double mean_steps(int64_t largest) { return 0.584 * std::log2((double)largest + 1); }

double scan_trips(double n, double step, double w, double W) {
  step = step < 0 ? -step : step;
  if (step == 0 || n <= 1) return 1;
  return std::min(n, (n * step / W + 1) * (w / step + 2));
}

// Points of one array, guard and pair of strides.
struct Combo {
  uint32_t epoch = 0;                    // of the plan that filled it
  uint16_t array = 0, guard = 0;
  int32_t a = 0, b = 0;
  bool runs = false, arc = false;        // executed at all; lo and width are known
  uint64_t intra = 0, inter = 0;         // records per block, cross-block records
  int64_t lo = 0, hi = 0;                // range of a*t + b*k
};

// Its place in the table: the top bits of a product, so that strides that are
// multiples of the table's size (block strides commonly are) differ in it.
uint32_t combo_index(const rp_point& p) {
  return (((uint32_t)p.array * 31u + (uint32_t)p.guard * 7u + (uint32_t)p.a * 5u + (uint32_t)p.b) *
          0x9E3779B1u) >> 24;
}

struct ArrayScratch {
  uint64_t bw = 1;                       // words per bin; its shift where a power of two
  int32_t sh = -1;
  bool used = false, full = false;       // some access; an arc round the circle
  uint64_t bins[CW_BINS / 64] = {};
  // the closed form's bound
  // distinct (b, block condition) of its points that are told apart, and distinct
  // |A|: their pairs are gone through one by one (planning 64 points of one
  // array takes 0.65 us with one stride, 2.0 us with eight)
  static constexpr int MAXC = 8;
  struct Blocks { int32_t b, S; uint32_t bm, br, Z; } c[MAXC];
  int nc = 0;
  bool many = false;                     // more than MAXC of them
  uint32_t step[MAXC];
  int ns = 0;
  bool steps = false;                    // more than MAXC of them
  uint32_t step_max = 0;                 // the largest of all
  uint64_t n = 0, intra = 0, inter = 0;  // points, records per block, cross-block records
  int64_t span = 0, bspan = 0;           // largest |A| * (X - 1) and |S| * (Z - 1)
};

struct PlanScratch {
  uint32_t epoch = 0;
  Combo combos[256];
  std::vector<ArrayScratch> arrays;
};
thread_local PlanScratch t_scratch;

void mark_bins(ArrayScratch& a, uint64_t wa, uint64_t wb) {   // words [wa, wb] inside [0, N)
  uint32_t j = (uint32_t)(a.sh >= 0 ? wa >> a.sh : wa / a.bw);
  const uint32_t e = (uint32_t)(a.sh >= 0 ? wb >> a.sh : wb / a.bw);
  for (; j <= e; j = (j | 63) + 1) {
    uint64_t m = ~0ull << (j & 63);
    if ((j | 63) > e) m &= ~0ull >> (63 - (e & 63));
    a.bins[j >> 6] |= m;
  }
}

// The first bin at or after j that is marked (or not), nb if there is none.
uint32_t next_bin(const ArrayScratch& a, uint32_t j, uint32_t nb, bool marked) {
  while (j < nb) {
    const uint64_t w = (marked ? a.bins[j >> 6] : ~a.bins[j >> 6]) >> (j & 63);
    if (w) return std::min<uint32_t>(nb, j + (uint32_t)__builtin_ctzll(w));
    j = (j | 63) + 1;
  }
  return nb;
}

// Rotation and span of an array of N words whose marked bins are known.
void rotation_of(const ArrayScratch& a, uint64_t N, uint64_t& off, uint64_t& span) {
  off = 0;
  span = N;
  if (a.full) return;
  if (!a.used) {
    span = 1;                                        // no access touches this array
    return;
  }
  const uint64_t bw = a.bw;
  const uint32_t nb = (uint32_t)((N + bw - 1) / bw);     // bins inside [0, N)
  // longest circular run of unmarked bins: the runs inside [0, nb), and the
  // one that wraps (the unmarked tail joined to the unmarked head)
  const uint32_t head = next_bin(a, 0, nb, true);
  if (head == nb) {
    span = 1;
    return;
  }
  uint32_t best_len = 0, best_end = 0, tail = 0;
  for (uint32_t j = 0; j < nb;) {
    const uint32_t z = next_bin(a, j, nb, false);
    const uint32_t o = next_bin(a, z, nb, true);
    if (o - z > best_len) {
      best_len = o - z;
      best_end = o == nb ? 0 : o;                    // first bin after the run
    }
    if (o == nb) tail = o - z;
    j = o;
  }
  if (head + tail > best_len) {                      // the wrapping run
    best_len = head + tail;
    best_end = head;
  }
  if (best_len == 0) return;
  // words of the gap: bins best_end - best_len .. best_end - 1 (mod nb);
  // only the last bin of the circle can be narrower than bw
  const uint64_t last_w = N - (uint64_t)(nb - 1) * bw;
  const uint32_t first = best_end >= best_len ? best_end - best_len : best_end + nb - best_len;
  const bool has_last = first + best_len > nb || first + best_len == nb;
  const uint64_t gap = (uint64_t)(best_len - (has_last ? 1 : 0)) * bw + (has_last ? last_w : 0);
  const uint64_t next = (uint64_t)best_end * bw;     // first word after the gap
  off = (N - next % N) % N;
  span = N - gap;
}

// Whether the closed form's bound can take the array (see above): then the form
// it needs, the bound on its tests, and what that costs beyond its own records.
bool bound_closed(const ArrayScratch& a, uint32_t words, bool global, uint32_t B, uint32_t T,
                  PlanArray& o) {
  if (a.n == 0 || a.span >= MAX_SPAN || a.bspan >= MAX_SPAN) return false;
  const double W = words, w = 2.0 * (double)a.span, wraps = 1 + std::floor(w / W);
  const double bw = 2.0 * (double)a.bspan;
  const bool cross = global && B > 1;
  double t0 = 1, t1 = cross ? 1 : 0;   // tests of a pair: same block, different blocks
  double e0 = 0, e1 = 0;               // Euclid's steps on two threads' steps, on two blocks'
  bool plain = !a.many;
  if (a.many) {                        // whatever the steps are
    t0 = B;
    if (cross) t1 = std::min(bw + 1, (double)B * B);
    if (cross) e1 = mean_steps(words);
  }
  if (a.steps) e0 = mean_steps(a.step_max);
  for (int u = 0; u < a.ns && !a.steps; u++)
    for (int v = 0; v < u; v++) (void)gcd_steps(a.step[u], a.step[v], e0);
  for (int u = 0; u < a.nc && !a.many; u++) {
    for (int v = 0; v <= u; v++) {
      const auto &p = a.c[u], &q = a.c[v];
      plain = plain && p.bm == 1 && q.bm == 1;
      const double lcm = p.bm == q.bm ? p.bm : (double)p.bm * q.bm / gcd_of<uint32_t>(p.bm, q.bm);
      if (lcm < B) {
        const int64_t db = step_mod((int64_t)p.b - q.b, words);
        t0 = std::max(t0, scan_trips(std::floor(B / lcm) + 1,
                                     step_mod(db * (int64_t)lcm, words), w, W));
      }
      if (cross) {
        const double sp = std::abs((double)p.S), sq = std::abs((double)q.S);
        const double g = gcd_steps((uint32_t)sp, (uint32_t)sq, e1);
        const double n = g > 0 ? (sp * (p.Z - 1.0) + sq * (q.Z - 1.0)) / g + 1 : 1;
        if (n <= (double)p.Z * q.Z) t1 = std::max(t1, scan_trips(n, g, w, W));
        else t1 = std::max(t1, p.Z <= q.Z ? p.Z * scan_trips(q.Z, q.S, w, W)
                                          : q.Z * scan_trips(p.Z, p.S, w, W));
        plain = plain && n <= (double)p.Z * q.Z;
      }
    }
  }
  const double n = (double)a.n, rec = (double)a.intra * B + (double)a.inter;
  const double work = n * (n + 1) / 2 * (t0 + t1) * wraps;
  const bool wide = a.span >= SMALL_SPAN || a.bspan >= SMALL_SPAN || words > SMALL_SIZE ||
                    T > SMALL_SIZE || B > SMALL_SIZE;
  // one lane's chain of tests
  const bool slow = wide && e0 + e1 > 2;
  const double serial = std::ceil(n / 64) * (std::max(t0, t1) * wraps * (slow ? SLOW_STEP : 1) +
                                             (slow ? SLOW_EUCLID * (e0 + e1) : 0));
  const double cost = work + n * (n + 1) / 2 * EUCLID * (e0 * (cross ? 2 : 1) + e1);
  if (work > RECORDS_FREE + rec || serial > SERIAL_FREE + rec / SERIAL_RECORDS) return false;
  o.form = FORM_PLAIN;
  if (wide) o.form = FORM_WIDE;
  else if (!plain) o.form = FORM_SMALL;
  o.tests = work;
  o.cost = cost;
  o.serial = serial;
  o.over = std::max(0.0, cost - rec);
  return true;
}

bool divides(uint32_t words, int32_t a) {                // a = 0 mod words
  return (a < 0 ? 0u - (uint32_t)a : (uint32_t)a) % words == 0;
}

// Records of an access point (the reductions are listed in common.h): per
// block of the same-block log, and in the cross-block log.
void records_of(uint32_t cnt, uint64_t nblk, bool tconst, bool bconst, bool cross,
                uint64_t& intra, uint64_t& inter) {
  intra = tconst ? std::min<uint64_t>(cnt, 2) : cnt;
  inter = 0;
  if (cross)
    inter = (tconst ? std::min<uint64_t>(cnt, 1) : cnt) *
            (bconst ? std::min<uint64_t>(nblk, 2) : nblk);
}

}  // namespace

// The least cost beyond an array's own records that no longer fits into the
// plans' allowance, least cost first.
static double cost_line(Plan* const* plans, size_t n) {
  std::vector<double> over;
  for (size_t j = 0; j < n; j++)
    for (const PlanArray& a : plans[j]->arrays)
      if (a.over > 0) over.push_back(a.over);
  std::sort(over.begin(), over.end());
  double sum = 0;
  for (double v : over)
    if ((sum += v) > COST_FREE) return v;
  return INFINITY;
}

// Where a call makes a log anyway, for arrays that no bound can take, the closed
// form of the others saves no launches: the longest chain of tests that is worth
// it.  The arrays up to a chain cost a launch, the chain (rows run beside each
// other) and their tests, and save their records.  All that can are kept unless
// a shorter chain, or none, is better by CHAIN_GAIN, less than a tenth of any call
// with a log.  51 points of 71 threads and 5 blocks, two of their four arrays on
// the log: 396 us with the others' chains of 350 tests, 249 by records alone.
static double longest_chain(Plan* const* plans, size_t n) {
  std::vector<const PlanArray*> v;
  double time = FIRST_LAUNCH, best = 0, at = -1;
  for (size_t j = 0; j < n; j++)
    for (const PlanArray& a : plans[j]->arrays)
      if (a.bounded) {
        v.push_back(&a);
        best += a.rec * RECORD_PS;
      }
  std::sort(v.begin(), v.end(),
            [](const PlanArray* a, const PlanArray* b) { return a->serial < b->serial; });
  time += best;
  double all = best;
  for (size_t q = 0; q < v.size(); q++) {
    time += v[q]->cost * TEST_PS - v[q]->rec * RECORD_PS;
    if (q + 1 < v.size() && v[q + 1]->serial == v[q]->serial) continue;
    all = time + v[q]->serial * CHAIN_PS;
    if (all < best) {
      best = all;
      at = v[q]->serial;
    }
  }
  return all - best > CHAIN_GAIN ? at : INFINITY;
}

// The arrays below the lines in closed form, and what follows from it.
static void set_routes(Plan& pl, double line, double chain) {
  uint64_t intra = 0, inter = 0;
  double tests = 0;
  pl.any_closed = false;
  pl.closed_form = FORM_PLAIN;
  for (PlanArray& a : pl.arrays) {
    a.closed = a.bounded && a.over < line && a.serial <= chain;
    if (a.closed) {
      pl.any_closed = true;
      pl.closed_form = std::max(pl.closed_form, a.form);
      tests += a.tests;
    } else {
      intra += a.intra;
      inter += a.inter;
    }
  }
  pl.rblk = intra;
  pl.log_intra = intra * pl.B;
  pl.log_inter = inter;
  pl.packed = pl.P <= PACKED_POINTS && tests <= PACKED_TESTS && intra + inter == 0;
}

void make_plan(const rp_kernel* k, Plan& pl) {
  pl.k = k;
  pl.P = k->n_points;
  pl.S = k->n_slots;
  pl.B = k->blocks;
  pl.T = k->threads;
  bool bguard = false;
  pl.guards.resize(k->n_guards);
  for (uint32_t g = 0; g < k->n_guards; g++) {
    // threads t < T with t % m == r, blocks likewise
    const rp_guard& t = k->guards[g];
    PlanGuard& o = pl.guards[g];
    o.cnt = t.r < pl.T ? (pl.T - 1 - t.r) / t.m + 1 : 0;
    o.bm = 1;
    o.br = 0;
    o.nblk = pl.B;
    if (k->block_guards) {
      o.bm = k->block_guards[g].m;
      o.br = k->block_guards[g].r;
      bguard |= o.bm > 1;
      o.nblk = o.br < pl.B ? (pl.B - 1 - o.br) / o.bm + 1 : 0;
    }
  }
  // padding records of the same-block log (blocks that do not execute a
  // point) use array id n_arrays
  pl.pad_array = bguard ? k->n_arrays : 0;
  pl.abits = bits_for(k->n_arrays ? k->n_arrays - 1 + bguard : 0);
  pl.bbits = bits_for(pl.B - 1);
  pl.pbits = bits_for(pl.P ? pl.P - 1 : 0);
  pl.tbits = bits_for(pl.T - 1);
  pl.key_shift = pl.tbits + pl.bbits + pl.pbits;
  pl.div_if_enabled = 0;
  pl.accesses = 0;
  PlanScratch& sc = t_scratch;
  if (++sc.epoch == 0) {                     // (wrapped: forget every combination)
    for (Combo& c : sc.combos) c.epoch = 0;
    sc.epoch = 1;
  }
  sc.arrays.assign(k->n_arrays, ArrayScratch{});
  for (uint32_t arr = 0; arr < k->n_arrays; arr++) {
    // words per bin, as a shift when it is a power of two (the usual case: no
    // division per access)
    const uint64_t N = k->arrays[arr].words;
    ArrayScratch& a = sc.arrays[arr];
    a.bw = (N + CW_BINS - 1) / CW_BINS;
    if ((N & (N - 1)) == 0 && (a.bw & (a.bw - 1)) == 0) a.sh = __builtin_ctzll(a.bw);
  }
  for (uint32_t i = 0; i < pl.P; i++) {
    const rp_point& p = k->points[i];
    if (p.kind == RP_NOP) continue;
    const PlanGuard& g = pl.guards[p.guard];
    if (p.kind == RP_BARRIER) {
      // a block barrier must be reached by all threads of each block that
      // reaches it, a grid barrier by all threads of the grid
      const uint64_t reach = (uint64_t)g.cnt * g.nblk;
      const bool div = k->slots[p.slot].level == RP_GRID
                           ? reach > 0 && reach < (uint64_t)pl.B * pl.T
                           : g.nblk > 0 && g.cnt > 0 && g.cnt < pl.T;
      if (div) pl.div_if_enabled |= 1ull << p.slot;
      continue;
    }
    const rp_array& ar = k->arrays[p.array];
    ArrayScratch& a = sc.arrays[p.array];
    Combo& c = sc.combos[combo_index(p)];
    if (!(c.epoch == sc.epoch && c.array == p.array && c.guard == p.guard && c.a == p.a &&
          c.b == p.b)) {
      c.epoch = sc.epoch;
      c.array = p.array;
      c.guard = p.guard;
      c.a = p.a;
      c.b = p.b;
      records_of(g.cnt, g.nblk, divides(ar.words, p.a), divides(ar.words, p.b),
                 ar.space == RP_GLOBAL && pl.B > 1, c.intra, c.inter);
      c.runs = g.cnt != 0 && g.nblk != 0;
      c.arc = false;
      if (c.runs) {
        const rp_guard& t = k->guards[p.guard];
        int64_t tlo, thi, blo, bhi;
        c.arc = ar.words <= (1ull << 31) && lin_range(p.a, t.r, t.m, g.cnt, tlo, thi) &&
                lin_range(p.b, g.br, g.bm, g.nblk, blo, bhi) &&
                !__builtin_add_overflow(tlo, blo, &c.lo) && !__builtin_add_overflow(thi, bhi, &c.hi);
        const Access s = make_access(p.a, p.b, 0, ar.words, t.m, t.r, g.cnt, g.bm, g.br, pl.B);
        a.span = std::max<int64_t>(a.span, abs_of<int64_t>(s.A) * (int64_t)(s.X - 1));
        a.bspan = std::max<int64_t>(a.bspan, abs_of<int64_t>(s.S) * (int64_t)(s.Z - 1));
        const uint32_t as = (uint32_t)abs_of<int64_t>(s.A);
        a.step_max = std::max(a.step_max, as);
        int q = 0;
        if (!a.many) {
          while (q < a.nc && !(a.c[q].b == s.b && a.c[q].bm == s.bm && a.c[q].br == s.br)) q++;
          if (q == ArrayScratch::MAXC) a.many = true;
          else if (q == a.nc) a.c[a.nc++] = {s.b, s.S, s.bm, s.br, s.Z};
        }
        if (!a.steps) {
          for (q = 0; q < a.ns && a.step[q] != as;) q++;
          if (q == ArrayScratch::MAXC) a.steps = true;
          else if (q == a.ns) a.step[a.ns++] = as;
        }
      }
    }
    pl.accesses += (uint64_t)g.cnt * g.nblk;
    a.n++;
    a.intra += c.intra;
    a.inter += c.inter;
    if (!c.runs || a.full) continue;
    a.used = true;
    // the arc of the point's words (rotated offsets must fit the int32 c)
    int64_t lo, hi;
    const uint64_t N = ar.words;
    if (!c.arc || __builtin_add_overflow(c.lo, (int64_t)p.c, &lo) ||
        __builtin_add_overflow(c.hi, (int64_t)p.c, &hi) || (uint64_t)(hi - lo) + 1 >= N) {
      a.full = true;
      continue;
    }
    const uint64_t s0 = word_mod(lo, (uint32_t)N), e0 = s0 + (uint64_t)(hi - lo);   // may pass N
    if (e0 < N) {
      mark_bins(a, s0, e0);
    } else {
      mark_bins(a, s0, N - 1);
      mark_bins(a, 0, e0 - N);
    }
  }
  uint64_t span_max = 1, intra = 0, inter = 0;
  pl.arrays.assign(k->n_arrays, PlanArray{});
  pl.over = 0;
  pl.log = false;
  for (uint32_t arr = 0; arr < k->n_arrays; arr++) {
    const ArrayScratch& a = sc.arrays[arr];
    const uint32_t words = k->arrays[arr].words;
    PlanArray& o = pl.arrays[arr];
    uint64_t off, span;
    rotation_of(a, words, off, span);
    span_max = std::max(span_max, span);
    o.off = (uint32_t)off;
    o.bounded = g_race_route == 0 && bound_closed(a, words, k->arrays[arr].space == RP_GLOBAL,
                                                  pl.B, pl.T, o);
    o.rec = (double)a.intra * pl.B + (double)a.inter;
    pl.over += o.over;
    pl.log = pl.log || (!o.bounded && o.rec > 0);
    o.intra = a.intra;
    o.inter = a.inter;
    intra += a.intra;
    inter += a.inter;
  }
  pl.nbits = bits_for(span_max - 1);
  pl.key_bits = pl.abits + pl.nbits;
  pl.n_intra = intra * pl.B;
  pl.n_inter = inter;
  pl.grid_slots = pl.pre_slots = 0;
  for (uint32_t s = 0; s < pl.S; s++) {
    if (k->slots[s].level == RP_GRID) pl.grid_slots |= 1ull << s;
    if (k->slots[s].preexisting) pl.pre_slots |= 1ull << s;
  }
  Plan* const self = &pl;
  set_routes(pl, pl.over <= COST_FREE ? INFINITY : cost_line(&self, 1),
             pl.log ? longest_chain(&self, 1) : INFINITY);
}

void choose_routes(Plan* const* plans, size_t n) {
  double over = 0;
  bool log = false;
  for (size_t j = 0; j < n; j++) {
    over += plans[j]->over;
    log = log || plans[j]->log;
  }
  if (over <= COST_FREE && !log) return;     // (nor has any of them a line of its own)
  const double line = over <= COST_FREE ? INFINITY : cost_line(plans, n);
  const double chain = log ? longest_chain(plans, n) : INFINITY;
  for (size_t j = 0; j < n; j++) set_routes(*plans[j], line, chain);
}

void fill_points(const Plan& pl, DPoint* pts) {
  const rp_kernel* k = pl.k;
  for (uint32_t i = 0; i < pl.P; i++) {
    const rp_point& p = k->points[i];
    DPoint d{};
    d.kind = p.kind;
    d.bm = 1;
    if (p.kind == RP_BARRIER) {
      d.array = p.slot;
      if (k->slots[p.slot].level == RP_GRID) d.flags = PF_GRID;
    } else if (p.kind == RP_ACCESS) {
      const PlanGuard& g = pl.guards[p.guard];
      const PlanArray& pa = pl.arrays[p.array];
      const rp_array& a = k->arrays[p.array];
      d.a = p.a;
      d.b = p.b;
      d.c = p.c;
      d.words = a.words;
      d.m = k->guards[p.guard].m;
      d.r = k->guards[p.guard].r;
      d.cnt = g.cnt;
      d.bm = g.bm;
      d.br = g.br;
      d.array = p.array;
      uint8_t f = (p.is_write ? PF_WRITE : 0) | (a.space == RP_GLOBAL ? PF_GLOBAL : 0);
      if (pa.closed) {
        // the closed form's steps and first word, reduced (closed.h); a point
        // that executes nowhere is none
        f |= PF_CLOSED;
        if (g.cnt == 0 || g.nblk == 0) {
          d.kind = RP_NOP;
        } else {
          const Access s = make_access(p.a, p.b, p.c, a.words, d.m, d.r, g.cnt, g.bm, g.br, pl.B);
          d.a = s.A;
          d.b = s.b;
          d.c = (int32_t)s.base;
        }
      } else {
        if ((a.words & (a.words - 1)) == 0) f |= PF_POW2;
        if (divides(a.words, p.a)) f |= PF_TCONST;
        if (divides(a.words, p.b)) f |= PF_BCONST;
        if (pa.off != 0) {
          const uint64_t c = (uint64_t)word_mod(p.c, a.words) + pa.off;      // (off < words)
          d.c = (int32_t)(uint32_t)(c >= a.words ? c - a.words : c);
        }
      }
      d.flags = f;
    }
    pts[i] = d;
  }
}

void fill_prefixes(const Plan& pl, const DPoint* pts, uint64_t* cnt_pre, uint64_t* gcnt_pre) {
  uint64_t in = 0, ex = 0;
  for (uint32_t i = 0; i < pl.P; i++) {
    cnt_pre[i] = in;
    gcnt_pre[i] = ex;
    const DPoint& d = pts[i];
    if (d.kind != RP_ACCESS || (d.flags & PF_CLOSED)) continue;
    uint64_t a, b;
    records_of(d.cnt, pl.guards[pl.k->points[i].guard].nblk, d.flags & PF_TCONST,
               d.flags & PF_BCONST, (d.flags & PF_GLOBAL) && pl.B > 1, a, b);
    in += a;
    ex += b;
  }
  cnt_pre[pl.P] = in;
  gcnt_pre[pl.P] = ex;
}

// Automatic digit width: the fewest passes of at most 10 bits, each as
// narrow as that pass count allows (but at least 8 bits).
int pick_digit_bits(uint32_t key_bits) {
  if (g_digit_bits) return g_digit_bits;
  const uint32_t passes = std::max<uint32_t>(1, (key_bits + 9) / 10);
  const uint32_t rb = (key_bits + passes - 1) / passes;
  return (int)std::min<uint32_t>(10, std::max<uint32_t>(8, rb));
}

static int g_low_digit_bits = 6;      // RP_TUNE_LOW_DIGIT_BITS

int low_digit_bits(int v, bool set) {
  const int old = g_low_digit_bits;
  if (set) g_low_digit_bits = v;
  return old;
}

std::vector<DigitPass> digit_plan(uint32_t key_bits) {
  std::vector<DigitPass> v;     // lowest digit first
  if (key_bits == 0) return v;
  const uint32_t low = (uint32_t)g_low_digit_bits;
  // the rest of the key above a narrow lowest digit, in digits of at most
  // 10 bits but no fewer than 6 (the narrowest digit the kernels take)
  const uint32_t rest = key_bits > low ? key_bits - low : 0;
  const uint32_t n = (rest + 9) / 10;
  if (low != 0 && rest > 0 && rest >= 6 * n && g_digit_bits == 0) {
    v.push_back(DigitPass{0, low});
    uint32_t lo = low;
    for (uint32_t i = 0; i < n; i++) {
      const uint32_t w = rest / n + (i < rest % n ? 1u : 0u);
      v.push_back(DigitPass{lo, w});
      lo += w;
    }
  } else {
    const uint32_t rb = (uint32_t)pick_digit_bits(key_bits);
    for (uint32_t lo = 0; lo < key_bits; lo += rb) v.push_back(DigitPass{lo, rb});
  }
  if (g_digit_order != 0) std::reverse(v.begin(), v.end());
  return v;
}

}  // namespace rp
