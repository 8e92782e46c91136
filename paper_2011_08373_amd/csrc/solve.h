// Solve of Alg. 1: the minimum-weight barrier assignment satisfying phi
// (weighted partial MaxSAT with phi hard and {not b_s} soft, Sections 2.3-2.4),
// ties broken by (number of enabled barriers, mask as an unsigned integer).
// As one integer the key is the sum over enabled slots of
// w_s*2^71 + 2^64 + 2^s, so it is additive over slots and the optimum is
// unique.  It is carried as (hi, lo) = (sum of w_s*128+1, mask).
//
// Under the mhs strategy the rounds before the first SAFE take the greedy
// hitting set of greedy_solve instead, and the round after it the exact
// query (phase PH_FINAL) that confirms or replaces the greedy answer.
//
// One workgroup of SV_BLOCK threads (the round loop's) per job:
//   1. reduction to a fixpoint: positive units force a slot on, negative units
//      force it off, a clause with no literal left proves UNSAT; a slot that
//      is in no positive literal of an open clause is set off (it can only
//      add weight); and a slot s is set off when another slot t with a smaller
//      key is in every open clause that s is in (and in no negative literal):
//      an assignment with s would be improved by t in its place, so the
//      optimum has no s.  Subsumed open clauses are dropped in between;
//   2. if what is left is all positive and every clause is a contiguous run of
//      the slots left (a race's clause is the run of barriers between two
//      points), the optimum is a shortest path over the slots
//      (interval_optimum), one step per slot;
//   3. else the open clauses split into components over the free slots (the
//      key is additive, so components are solved independently): again a
//      path where one is made of runs;
//   4. a component of k <= 20 slots is enumerated bit-sliced: a 64-bit word
//      holds the six lowest slots' 64 assignments, every clause is evaluated
//      on whole words with AND/OR, and each word's cheapest feasible pattern
//      is found through the patterns pre-sorted by key;
//   5. a wider component is searched depth-first by all waves of the
//      workgroup: branch on the free positive literals of the open clause
//      with the fewest of them, prune on key and on a per-clause lower bound;
//      clause tests are spread over the 64 lanes and combined with
//      cross-lane reductions.  The tree's nodes at depth SPLIT_DEPTH are
//      dealt out to the waves in the order of the search (every wave walks
//      the levels above it alike, pruning there only dead nodes, so they all
//      number those nodes the same way); below it each wave searches its own
//      subtrees, pruning against the smallest weight any wave has found so
//      far (a shared word) as well as its own best key.  The optimum is
//      unique, so the smallest of the waves' best keys is the answer whatever
//      order the waves run in.
// Up to WV_CLAUSES clauses are held in the registers of a wave, one or two per
// lane: every wave then runs the greedy strategy and the reduction alike, with
// no barrier and no LDS.  More are staged in LDS (up to SV_CLAUSES; more again
// are read from memory until few enough are open) and reduced by the whole
// workgroup until they fit a wave.  Bound: latency, a chain of reductions: keys
// are compared in 32 bits where they fit, and what a wave does not need is out
// of line.  Measured: 300 runs over 56 slots of weights 1 to 10, 69 us by
// reduction and path (81 us with 64-bit keys and one clause read at a time), 1
// to 90 ms (over a second at 64 slots) by the search alone; the 35 greedy rounds
// of plain-large one trace at a time 0.25 ms, 0.36 ms with 64-bit keys, weights
// compared slot by slot and phi in memory, 0.85 ms with a barrier per pick, 2.5
// ms with LDS counters per slot and one thread comparing them; 512 instrumented
// programs to their verdicts 0.09 ms, 0.14 ms reduced with barriers, 0.47 ms by
// enumeration alone.
#pragma once
#include "common.h"

namespace rp {

constexpr int SV_BLOCK = 256;
constexpr int SV_WAVES = SV_BLOCK / 64;
constexpr uint32_t SV_CLAUSES = 1536;     // clauses of a component; clauses kept in LDS
constexpr int ENUM_MAX = 20;

struct Key { uint64_t hi, lo; };
__device__ __forceinline__ bool key_lt(Key a, Key b) { return a.hi != b.hi ? a.hi < b.hi : a.lo < b.lo; }

__device__ __forceinline__ uint32_t sv_uni(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ uint64_t sv_uni64(uint64_t v) {
  return ((uint64_t)sv_uni((uint32_t)(v >> 32)) << 32) | sv_uni((uint32_t)v);
}
__device__ __forceinline__ uint64_t lane_value(uint64_t v, uint32_t l) {   // v of lane l, uniform
  return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), l) << 32) |
         (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, l);
}

// Whether lane l's bit of the uniform mask m is set.
__device__ __forceinline__ bool lane_bit(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }

// OR over the wave (DPP row shifts and broadcasts; the result is uniform).
__device__ __forceinline__ uint32_t wave_or32(uint32_t v) {
  v |= __builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, false);   // row_shr 1, 2, 4, 8
  v |= __builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, false);
  v |= __builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, false);
  v |= __builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, false);
  v |= __builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xF, 0xF, false);   // row_bcast 15, 31
  v |= __builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xF, 0xF, false);
  return __builtin_amdgcn_readlane(v, 63);
}
__device__ __forceinline__ uint64_t wave_or(uint64_t v) {
  return ((uint64_t)wave_or32((uint32_t)(v >> 32)) << 32) | wave_or32((uint32_t)v);
}
// Sum over the wave (row prefixes by shifts, then the rows' totals).
__device__ __forceinline__ uint32_t wave_sum32(uint32_t v) {
  v += __builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false);
  return __builtin_amdgcn_readlane(v, 63);
}
// Minimum, maximum over the wave; a lane with no source keeps its own value.
template <int CTRL>
__device__ __forceinline__ uint64_t dpp64(uint64_t v) {
  const int lo = (int)(uint32_t)v, hi = (int)(uint32_t)(v >> 32);
  return ((uint64_t)(uint32_t)__builtin_amdgcn_update_dpp(hi, hi, CTRL, 0xF, 0xF, false) << 32) |
         (uint32_t)__builtin_amdgcn_update_dpp(lo, lo, CTRL, 0xF, 0xF, false);
}
__device__ __forceinline__ uint64_t wave_min_u64(uint64_t v) {
  auto mn = [](uint64_t a, uint64_t b) { return b < a ? b : a; };
  v = mn(v, dpp64<0x111>(v));
  v = mn(v, dpp64<0x112>(v));
  v = mn(v, dpp64<0x114>(v));
  v = mn(v, dpp64<0x118>(v));
  v = mn(v, dpp64<0x142>(v));
  v = mn(v, dpp64<0x143>(v));
  return lane_value(v, 63);
}
__device__ __forceinline__ uint32_t wave_min_u32(uint32_t v) {
  auto mn = [](uint32_t a, int b) { return (uint32_t)b < a ? (uint32_t)b : a; };
  v = mn(v, __builtin_amdgcn_update_dpp((int)v, (int)v, 0x111, 0xF, 0xF, false));
  v = mn(v, __builtin_amdgcn_update_dpp((int)v, (int)v, 0x112, 0xF, 0xF, false));
  v = mn(v, __builtin_amdgcn_update_dpp((int)v, (int)v, 0x114, 0xF, 0xF, false));
  v = mn(v, __builtin_amdgcn_update_dpp((int)v, (int)v, 0x118, 0xF, 0xF, false));
  v = mn(v, __builtin_amdgcn_update_dpp((int)v, (int)v, 0x142, 0xF, 0xF, false));
  v = mn(v, __builtin_amdgcn_update_dpp((int)v, (int)v, 0x143, 0xF, 0xF, false));
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}
__device__ __forceinline__ uint32_t wave_min(uint32_t v) { return wave_min_u32(v); }
__device__ __forceinline__ uint64_t wave_min(uint64_t v) { return wave_min_u64(v); }
__device__ __forceinline__ uint64_t wave_max_u64(uint64_t v) { return ~wave_min_u64(~v); }
// Total weight of the slots of x (the same in every lane).
__device__ __forceinline__ uint64_t weight_of(uint64_t x, const uint32_t* s_w) {
  const uint32_t w = (x >> __lane_id()) & 1 ? s_w[__lane_id()] : 0;
  return ((uint64_t)wave_sum32(w >> 16) << 16) + wave_sum32(w & 0xFFFFu);
}

__device__ __forceinline__ Key block_min_key(Key k, uint64_t* smh, uint64_t* sml) {
  for (int off = 32; off > 0; off >>= 1) {
    Key o;
    o.hi = __shfl_xor(k.hi, off);
    o.lo = __shfl_xor(k.lo, off);
    if (key_lt(o, k)) k = o;
  }
  const int w = threadIdx.x >> 6;
  if (__lane_id() == 0) { smh[w] = k.hi; sml[w] = k.lo; }
  __syncthreads();
  Key r = {smh[0], sml[0]};
  for (int q = 1; q < SV_WAVES; q++) {
    Key o = {smh[q], sml[q]};
    if (key_lt(o, r)) r = o;
  }
  __syncthreads();
  return r;
}

// pattern of local slot b (< 6) over the 64 assignments of a word
__device__ __forceinline__ uint64_t pat(int b) {
  const uint64_t P6[6] = {0xAAAAAAAAAAAAAAAAull, 0xCCCCCCCCCCCCCCCCull, 0xF0F0F0F0F0F0F0F0ull,
                          0xFF00FF00FF00FF00ull, 0xFFFF0000FFFF0000ull, 0xFFFFFFFF00000000ull};
  return P6[b];
}

struct DfsFrame { uint64_t ones, zeros, khi, klo, todo, tried; };
constexpr int SPLIT_DEPTH = 3;           // depth whose nodes are dealt out to the waves

constexpr uint32_t GREEDY_MAX = 16384;   // clauses the greedy step handles

// A job's weights and, per slot, the slots with a smaller key (LDS).
struct SlotKeys {
  uint32_t w[64];
  union {
    uint64_t less[64];
    uint16_t part[64][SV_WAVES];           // (a quarter by each wave)
  };
};
__device__ __forceinline__ void slot_keys(const Job& J, SlotKeys& K) {
  static_assert(64 / SV_WAVES == 16, "a wave's quarter");
  const uint32_t l = __lane_id(), wv = sv_uni(threadIdx.x >> 6), t0 = wv * 16;
  const uint32_t w = l < J.S ? J.weights[l] : 0;
  uint32_t m = 0;
  if (t0 < J.S)
#pragma unroll
    for (uint32_t k = 0; k < 16; k++) {    // (a slot past the last one is in no clause)
      const uint32_t o = (uint32_t)__builtin_amdgcn_readlane((int)w, t0 + k);
      m |= (o < w || (o == w && t0 + k < l) ? 1u : 0u) << k;
    }
  K.part[l][wv] = (uint16_t)m;
  if (wv == 0) K.w[l] = w;
}

// LDS of the solver.
struct SolveLds {
  rp_clause cl[SV_CLAUSES];                // phi, then the open clauses (restricted)
  union {
    rp_clause u[SV_CLAUSES];               // open clauses on their way through the reduction
    struct {                               // per component: local pos / neg
      uint64_t lp[SV_CLAUSES], ln[SV_CLAUSES];
    };
  };
  uint64_t la[SV_CLAUSES];                 // aux per component clause
  uint64_t kh[64], kl[64];                 // local slot key parts
  uint64_t lowh[64], lowl[64];             // key of each low pattern
  uint32_t order[64], gslot[64];
  int32_t first[64], last[64];             // per last (first) slot: the largest first (last) slot
  uint64_t smA[SV_WAVES], smB[SV_WAVES];
  uint64_t inch[SV_WAVES], incl[SV_WAVES];
  uint64_t red[2][SV_WAVES][5];            // reductions, two in turn (one barrier each)
  union {
    uint64_t dom[2][SV_WAVES][64];         // of the reduction, of the greedy set, of the search
    uint32_t c64[2][SV_WAVES][64];
    DfsFrame stack[SV_WAVES][65];
  };
  unsigned long long bound;                // smallest weight part found by any wave
  uint32_t cnt, overflow;
};

// OR of K values over the workgroup.  turn alternates between calls, so that a
// call's values are read by everyone before the call after next writes there.
template <int K>
__device__ __forceinline__ void block_or(uint64_t (&v)[K], SolveLds& L, uint32_t& turn) {
  const uint32_t w = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < K; k++) v[k] = wave_or(v[k]);
  if (__lane_id() == 0) {
#pragma unroll
    for (int k = 0; k < K; k++) L.red[turn][w][k] = v[k];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < K; k++) {
    uint64_t r = 0;
    for (int q = 0; q < SV_WAVES; q++) r |= L.red[turn][q][k];
    v[k] = sv_uni64(r);
  }
  turn ^= 1;
}

// The lane (slot) with the largest c / w, the lowest one of equals; some c is
// not 0.  From a first slot on, to the lowest slot that is better than it, as
// long as there is one (every best slot is, so the last step meets the lowest).
// NARROW: counts below 2^8 and weights below 2^24, a product in 32 bits.
template <bool NARROW>
__device__ __forceinline__ uint32_t best_slot(uint32_t c, uint32_t w) {
  auto of = [](uint32_t v, uint32_t l) { return (uint32_t)__builtin_amdgcn_readlane((int)v, l); };
  uint32_t best = (uint32_t)__builtin_ctzll(__ballot(c != 0));
  for (;;) {
    const uint32_t cb = of(c, best), wb = of(w, best);
    const uint64_t m = NARROW ? __ballot(__umul24(c, wb) > __umul24(cb, w))
                              : __ballot((uint64_t)c * wb > (uint64_t)cb * w);
    if (m == 0) return best;
    best = (uint32_t)__builtin_ctzll(m);
  }
}

// A greedy answer into the state (every thread of the workgroup calls it).
__device__ __forceinline__ void greedy_answer(JobState* st, const uint32_t* s_w, uint64_t x) {
  const uint64_t W = weight_of(x, s_w);
  if (threadIdx.x != 0) return;
  st->x = x;
  st->weight = W;
  if (st->max_rounds && st->rounds >= st->max_rounds) st->state = ST_ROUNDS;
}

// The mhs strategy's Solve (Section 2.4): the greedy minimal hitting set of
// the positive clauses of phi -- repeatedly the slot hitting the most clauses
// not yet hit per unit of weight (exact integer comparison, ties to the lower
// slot), then every pick whose removal leaves all positive clauses hit is
// dropped, last pick first.  Returns false (the caller solves exactly) when
// phi has an empty clause, is too long, or the set breaks a clause of phi.
// A lane is a slot: the waves share the clauses of a count (LDS: each clause
// read once by all lanes; from memory a clause per lane, counted with LDS
// adds), and every wave finds the best slot alike, so a pick costs one barrier.
template <bool LDS, class G>
__device__ bool greedy_solve(const Job& J, const uint32_t* s_w, JobState* st, uint32_t n, G get,
                             SolveLds& L, uint32_t& turn) {
  const uint32_t tid = threadIdx.x, lane = __lane_id(), wv = sv_uni(tid >> 6);
  if (n > GREEDY_MAX) return false;
  uint64_t bad[1] = {0};
  for (uint32_t q = tid; q < n; q += SV_BLOCK) {
    const rp_clause c = get(q);
    if (c.pos == 0 && c.neg == 0) bad[0] = 1;
  }
  block_or(bad, L, turn);
  if (bad[0]) return false;
  const uint32_t w = lane < J.S ? s_w[lane] : 1;
  uint64_t x = 0;
  uint32_t np = 0, mine = 0;               // picks; lane q keeps the q-th
  while (np < 64) {
    uint32_t c = 0;
    if constexpr (LDS) {
      for (uint32_t q = wv; q < n; q += SV_WAVES) {
        const rp_clause t = get(q);
        const uint64_t pos = sv_uni64(t.pos), neg = sv_uni64(t.neg);
        if (neg == 0 && (pos & x) == 0) c += (uint32_t)(pos >> lane) & 1u;
      }
      L.c64[turn][wv][lane] = c;
    } else {
      L.c64[turn][wv][lane] = 0;
      for (uint32_t q = tid; q < n; q += SV_BLOCK) {
        const rp_clause t = get(q);
        if (t.neg != 0 || (t.pos & x) != 0) continue;
        for (uint64_t p = t.pos; p; p &= p - 1) atomicAdd(&L.c64[turn][wv][__builtin_ctzll(p)], 1u);
      }
    }
    __syncthreads();
    c = 0;
    for (int q = 0; q < SV_WAVES; q++) c += L.c64[turn][q][lane];
    turn ^= 1;
    if (__ballot(c != 0) == 0) break;
    const uint32_t best = best_slot<false>(c, w);
    x |= 1ull << best;
    if (lane == np) mine = best;
    np++;
  }
  // every wave tests every clause, alike
  for (uint32_t k = np; k-- > 0;) {
    const uint64_t y = x & ~(1ull << __builtin_amdgcn_readlane(mine, k));
    bool miss = false;
    for (uint32_t q = lane; q < n && !miss; q += 64) {
      const rp_clause c = get(q);
      miss = c.pos && !c.neg && !(c.pos & y);
    }
    if (__ballot(miss) == 0) x = y;
  }
  bool viol = false;
  for (uint32_t q = lane; q < n && !viol; q += 64) {
    const rp_clause c = get(q);
    viol = !((c.pos & x) || (c.neg & ~x));
  }
  if (__ballot(viol)) return false;
  greedy_answer(st, s_w, x);
  return true;
}

// Clauses held by a wave: clause 64 g + l in lane l.
constexpr uint32_t WV_CLAUSES = 128;
template <int G>
struct WaveClauses {
  uint64_t pos[G], neg[G];
  bool on[G];                              // there is (still) such a clause
};
template <int G>
__device__ __forceinline__ WaveClauses<G> wave_clauses(const rp_clause* C, uint32_t n) {
  WaveClauses<G> c;
#pragma unroll
  for (int g = 0; g < G; g++) {
    const uint32_t q = 64 * g + __lane_id();
    c.on[g] = q < n;
    const rp_clause v = c.on[g] ? C[q] : rp_clause{0, 0};
    c.pos[g] = v.pos;
    c.neg[g] = v.neg;
  }
  return c;
}

// greedy_solve on clauses held by every wave alike.  A lane is a slot too: it
// keeps the set of clauses its slot hits, one bit each.
template <int G>
__device__ __forceinline__ bool greedy_wave(uint32_t S, const uint32_t* s_w, JobState* st,
                                            const WaveClauses<G>& c) {
  const uint32_t lane = __lane_id();
  bool empty = false;
  uint64_t hits[G], todo[G];
#pragma unroll
  for (int g = 0; g < G; g++) {
    empty = empty || (c.on[g] && c.pos[g] == 0 && c.neg[g] == 0);
    const uint64_t p = c.on[g] && c.neg[g] == 0 ? c.pos[g] : 0;     // a positive clause
    todo[g] = __ballot(p != 0);
    hits[g] = 0;
    uint32_t lo = 0, hi = 0;
    for (uint32_t m = (uint32_t)todo[g]; m; m &= m - 1) {
      const uint32_t r = (uint32_t)__builtin_ctz(m);
      if (lane_bit(lane_value(p, r))) lo |= 1u << r;
    }
    for (uint32_t m = (uint32_t)(todo[g] >> 32); m; m &= m - 1) {
      const uint32_t r = (uint32_t)__builtin_ctz(m);
      if (lane_bit(lane_value(p, 32 + r))) hi |= 1u << r;
    }
    hits[g] = (uint64_t)hi << 32 | lo;
  }
  if (__ballot(empty)) return false;
  const uint32_t w = lane < S ? s_w[lane] : 1;
  const bool narrow = __ballot(w >= 1u << 24) == 0;
  uint64_t x = 0;
  uint32_t np = 0, mine = 0;               // picks; lane q keeps the q-th
  for (;;) {
    uint32_t k = 0;
#pragma unroll
    for (int g = 0; g < G; g++) k += (uint32_t)__popcll(hits[g] & todo[g]);
    if (__ballot(k != 0) == 0) break;
    const uint32_t best = narrow ? best_slot<true>(k, w) : best_slot<false>(k, w);
    x |= 1ull << best;
    if (lane == np) mine = best;
    np++;
#pragma unroll
    for (int g = 0; g < G; g++) todo[g] &= ~lane_value(hits[g], best);
  }
  for (uint32_t k = np; k-- > 0;) {
    const uint64_t y = x & ~(1ull << __builtin_amdgcn_readlane(mine, k));
    bool miss = false;
#pragma unroll
    for (int g = 0; g < G; g++)
      miss = miss || (c.on[g] && c.pos[g] && !c.neg[g] && !(c.pos[g] & y));
    if (__ballot(miss) == 0) x = y;
  }
  bool viol = false;
#pragma unroll
  for (int g = 0; g < G; g++)
    viol = viol || (c.on[g] && !((c.pos[g] & x) || (c.neg[g] & ~x)));
  if (__ballot(viol)) return false;
  greedy_answer(st, s_w, x);
  return true;
}

// The slots of core that another one makes needless: d has the slots in every
// open clause of the lane's slot, negs those in a negative literal.
__device__ __forceinline__ uint64_t needless(uint64_t d, uint64_t core, uint64_t negs,
                                             const uint64_t* less) {
  return core & __ballot((d & core & ~negs & less[__lane_id()]) != 0);
}

// The reduction on clauses held by every wave alike, to its fixpoint: on and
// off grow, satisfied and subsumed clauses go, the others are restricted to
// the free slots.  Returns false when they cannot be satisfied.
template <int G>
__device__ __forceinline__ bool reduce_wave(WaveClauses<G>& c, uint64_t all, const uint64_t* less,
                                            uint64_t& on, uint64_t& off) {
  const uint32_t lane = __lane_id();
  for (;;) {
    uint64_t vp = 0, vn = 0, up = 0, un = 0;
    bool bad = false;
#pragma unroll
    for (int g = 0; g < G; g++) {
      if (!c.on[g] || (c.pos[g] & on) || (c.neg[g] & off)) {
        c.on[g] = false;
        continue;
      }
      const uint64_t p = c.pos[g] &= ~off, m = c.neg[g] &= ~on;
      vp |= p;
      vn |= m;
      if (p == 0 && m == 0) bad = true;
      else if (p == 0 && (m & (m - 1)) == 0) un |= m;
      else if (m == 0 && (p & (p - 1)) == 0) up |= p;
    }
    if (__ballot(bad)) return false;
    const uint64_t core = wave_or(vp), negs = __ballot(vn != 0) ? wave_or(vn) : 0;
    uint64_t non = 0, noff = 0;
    if (__ballot((up | un) != 0)) {
      non = wave_or(up);
      noff = wave_or(un);
      if ((non & (off | noff)) || (noff & (on | non))) return false;
    }
    const uint64_t nz = all & ~on & ~off & ~non & ~noff & ~core;
    on |= non;
    off |= noff | nz;
    if (non | noff | (nz & negs)) continue;
    if (core == 0) return true;
    // every clause past every lane: as a slot, the lane keeps what is in all
    // clauses of its slot; as a clause, it is dropped for a subset
    uint64_t d = ~0ull;
    bool dead[G] = {};
#pragma unroll
    for (int h = 0; h < G; h++) {
      if (negs == 0) {
        for (uint64_t m = __ballot(c.on[h]); m; m &= m - 1) {
          const uint32_t r = (uint32_t)__builtin_ctzll(m);
          const uint64_t p = lane_value(c.pos[h], r);
          if (lane_bit(p)) d &= p;
#pragma unroll
          for (int g = 0; g < G; g++)
            dead[g] = dead[g] || ((p & ~c.pos[g]) == 0 && (p != c.pos[g] || 64 * h + r < 64 * g + lane));
        }
      } else {
        for (uint64_t m = __ballot(c.on[h]); m; m &= m - 1) {
          const uint32_t r = (uint32_t)__builtin_ctzll(m);
          const uint64_t p = lane_value(c.pos[h], r), q = lane_value(c.neg[h], r);
          if (lane_bit(p)) d &= p;
#pragma unroll
          for (int g = 0; g < G; g++)
            dead[g] = dead[g] || ((p & ~c.pos[g]) == 0 && (q & ~c.neg[g]) == 0 &&
                                  (p != c.pos[g] || q != c.neg[g] || 64 * h + r < 64 * g + lane));
        }
      }
    }
    bool died = false;
#pragma unroll
    for (int g = 0; g < G; g++) {
      died = died || (c.on[g] && dead[g]);
      c.on[g] = c.on[g] && !dead[g];
    }
    const uint64_t drop = needless(d, core, negs, less);
    off |= drop;
    if (drop == 0 && __ballot(died) == 0) return true;
  }
}

// Reduction of the n clauses get(q): on and off grow to the fixpoint, by units
// and, with DOM (clauses in LDS), by slots another one makes needless.
// Returns false when the clauses cannot be satisfied.
template <bool DOM, class G>
__device__ bool propagate(G get, uint32_t n, uint64_t all, const uint64_t* less, uint64_t& on,
                          uint64_t& off, SolveLds& L, uint32_t& turn) {
  const uint32_t tid = threadIdx.x, lane = __lane_id(), wv = sv_uni(tid >> 6);
  for (;;) {
    uint64_t v[5] = {0, 0, 0, 0, 0};       // new units on, off, positive, negative literals, empty
    for (uint32_t q = tid; q < n; q += SV_BLOCK) {
      const rp_clause c = get(q);
      if ((c.pos & on) || (c.neg & off)) continue;
      const uint64_t p = c.pos & ~off, m = c.neg & ~on;
      if (p == 0 && m == 0) v[4] = 1;
      else if (p == 0 && (m & (m - 1)) == 0) v[1] |= m;
      else if (m == 0 && (p & (p - 1)) == 0) v[0] |= p;
      v[2] |= p;
      v[3] |= m;
    }
    block_or(v, L, turn);
    const uint64_t non = v[0], noff = v[1], core = v[2];
    if (v[4] || (non & (off | noff)) || (noff & (on | non))) return false;
    const uint64_t nz = all & ~on & ~off & ~non & ~noff & ~core;
    on |= non;
    off |= noff | nz;
    if (non | noff | nz) continue;
    if (!DOM || core == 0) return true;
    // slots in every open clause of the lane's slot
    uint64_t d = ~0ull;
    for (uint32_t q = wv; q < n; q += SV_WAVES) {
      const rp_clause c = get(q);
      const uint64_t pos = sv_uni64(c.pos), neg = sv_uni64(c.neg);
      if ((pos & on) || (neg & off)) continue;
      if ((pos >> lane) & 1) d &= pos;
    }
    L.dom[turn][wv][lane] = d;
    __syncthreads();
    for (int q = 0; q < SV_WAVES; q++) d &= L.dom[turn][q][lane];
    turn ^= 1;
    const uint64_t drop = needless(d, core, v[3], less);
    if (drop == 0) return true;
    off |= drop;
  }
}

// The optimum over the slots of M when every clause is positive and a
// contiguous run of them; fl: the largest first slot of the clauses whose last
// slot is this lane (-1: none), ll: the largest last slot of those whose first
// is this lane.  Slots are taken in ascending order: a chosen slot s may
// follow a chosen slot p exactly when no clause lies wholly between them,
// that is when p >= the largest first slot of the clauses that end before s.
// Every wave computes the same; lane p keeps the best key of a choice that
// ends with p, its first part in an H.  The budget counts one node per slot of
// a run of linked slots longer than ENUM_MAX (returns false when it is spent):
// a caller that sets a budget of fewer nodes than there are slots gets the
// status that the search gave it, which takes more nodes than slots there.
template <class H>
__device__ __forceinline__ bool interval_path(uint64_t M, const uint32_t* s_w, uint64_t budget,
                                              int32_t fl, int32_t ll, uint64_t& answer) {
  const uint32_t lane = __lane_id();
  const bool slot = lane_bit(M);
  const H w = slot ? (H)s_w[lane] * 128u + 1u : 0;
  H bh = (H)~(H)0;                         // this lane's best key
  uint64_t bl = 0;
  int32_t need = -1, reach = -1;           // largest first slot that ended; last slot reached
  uint32_t run = 0;
  // the least key of the lanes in
  auto least = [&](bool in, H& h) {
    h = wave_min(in ? bh : (H)~(H)0);
    uint64_t tie = __ballot(in && bh == h);
    uint64_t l = lane_value(bl, (uint32_t)__builtin_ctzll(tie));
    for (tie &= tie - 1; tie; tie &= tie - 1) {
      const uint64_t o = lane_value(bl, (uint32_t)__builtin_ctzll(tie));
      l = o < l ? o : l;
    }
    return l;
  };
  for (uint64_t m = M; m; m &= m - 1) {
    const uint32_t s = (uint32_t)__builtin_ctzll(m);
    run = reach >= (int32_t)s ? run + 1 : 1;
    if (run > (uint32_t)ENUM_MAX && run > budget) return false;
    H h = 0;                               // nothing before s has to be hit
    uint64_t l = 0;
    if (need >= 0) l = least(slot && lane < s && (int32_t)lane >= need, h);
    if (lane == s) {
      bh = h + w;
      bl = l | 1ull << s;
    }
    const int32_t f = __builtin_amdgcn_readlane(fl, s), e = __builtin_amdgcn_readlane(ll, s);
    need = f > need ? f : need;
    reach = e > reach ? e : reach;
  }
  H h;
  answer = least(slot && (int32_t)lane >= need, h);
  return true;
}
__device__ __forceinline__ bool interval_optimum(uint64_t M, const uint32_t* s_w, uint64_t budget,
                                                 int32_t fl, int32_t ll, uint64_t& answer) {
  // (a key's first part is at most 128 times the total weight and 64)
  return weight_of(M, s_w) < (1u << 25) - 1 ? interval_path<uint32_t>(M, s_w, budget, fl, ll, answer)
                                            : interval_path<uint64_t>(M, s_w, budget, fl, ll, answer);
}

// Whether the clauses U[0..n) inside the slots M are all positive contiguous
// runs of M; then first and last are filled for interval_optimum.
__device__ bool intervals_of(const rp_clause* U, uint32_t n, uint64_t M, SolveLds& L,
                             uint32_t& turn) {
  const uint32_t tid = threadIdx.x;
  if (tid < 64) L.first[tid] = L.last[tid] = -1;
  __syncthreads();
  uint64_t other[1] = {0};
  for (uint32_t q = tid; q < n; q += SV_BLOCK) {
    const rp_clause c = U[q];
    if (!((c.pos | c.neg) & M)) continue;
    if (c.pos == 0 || c.neg != 0) {
      other[0] = 1;
      continue;
    }
    const uint32_t lo = (uint32_t)__builtin_ctzll(c.pos), hi = 63u - (uint32_t)__builtin_clzll(c.pos);
    const uint64_t span = (~0ull >> (63 - hi)) & (~0ull << lo);
    if ((M & span) != c.pos) other[0] = 1;
    atomicMax(&L.first[hi], (int32_t)lo);
    atomicMax(&L.last[lo], (int32_t)hi);
  }
  block_or(other, L, turn);
  return other[0] == 0;
}

// The same for clauses held by a wave: fl and ll by passing every clause by
// every lane.  False when some clause is no run of M.
template <int G>
__device__ __forceinline__ bool wave_intervals(const WaveClauses<G>& c, uint64_t M, int32_t& fl,
                                               int32_t& ll) {
  const int32_t lane = (int32_t)__lane_id();
  fl = ll = -1;
#pragma unroll
  for (int g = 0; g < G; g++) {
    uint32_t lo = 0, hi = 0;
    bool other = false;
    if (c.on[g]) {
      other = c.pos[g] == 0 || c.neg[g] != 0;
      if (!other) {
        lo = (uint32_t)__builtin_ctzll(c.pos[g]);
        hi = 63u - (uint32_t)__builtin_clzll(c.pos[g]);
        other = (M & (~0ull >> (63 - hi)) & (~0ull << lo)) != c.pos[g];
      }
    }
    if (__ballot(other)) return false;
    for (uint64_t m = __ballot(c.on[g]); m; m &= m - 1) {
      const uint32_t r = (uint32_t)__builtin_ctzll(m);
      const int32_t l = __builtin_amdgcn_readlane(lo, r), h = __builtin_amdgcn_readlane(hi, r);
      if (h == lane) fl = l > fl ? l : fl;
      if (l == lane) ll = h > ll ? h : ll;
    }
  }
  return true;
}

// The reduction in the waves (of W[0..n), every wave alike) and, where that
// leaves runs of slots, the path: result.  Else left has the slots left, and
// L.cl[0..n) their clauses.  sat: they can be satisfied.  Returns false when
// the job has failed.
template <int G>
__device__ bool solve_wave(const Job& J, JobState* st, const rp_clause* W, uint32_t& n, uint64_t all,
                           const SlotKeys& K, SolveLds& L, int wv, uint64_t& on, uint64_t& off,
                           bool& sat, uint64_t& result, uint64_t& left) {
  WaveClauses<G> c = wave_clauses<G>(W, n);
  sat = reduce_wave(c, all, K.less, on, off);
  left = sat ? all & ~on & ~off : 0;
  if (left == 0) return true;
  int32_t fl, ll;
  if (wave_intervals(c, left, fl, ll)) {
    if (!interval_optimum(left, K.w, J.node_limit, fl, ll, result)) {
      if (threadIdx.x == 0) { st->err = ERR_NODES; st->state = ST_ERROR; }
      return false;
    }
    left = 0;
    return true;
  }
  // (the waves hold the same clauses: the first writes them out)
  n = 0;
  __syncthreads();                         // (everyone has read W)
#pragma unroll
  for (int g = 0; g < G; g++) {
    const uint64_t m = __ballot(c.on[g]);
    if (wv == 0 && c.on[g])
      L.cl[n + (uint32_t)__popcll(m & lanemask_lt())] = rp_clause{c.pos[g], c.neg[g]};
    n += (uint32_t)__popcll(m);
  }
  __syncthreads();
  return true;
}

// The rest of Solve, by the whole workgroup and out of line: the rounds' code is
// what is left of solve_body.
//
// Clauses too many for a wave: the greedy strategy (answered), the reduction
// and, over all that is left, the path.
struct Reduced {
  uint64_t on, off, result, left;
  rp_clause* U;                            // open clauses
  uint32_t nu;
  bool sat, answered;
};
__device__ __noinline__ Reduced reduce_many(const Job& J, JobState* st, const rp_clause* C, uint32_t n,
                                            uint64_t all, uint32_t phase, const SlotKeys& K,
                                            SolveLds& L) {
  const uint32_t tid = threadIdx.x, lane = __lane_id();
  uint32_t turn = 0;
  Reduced R{0, 0, 0, 0, L.cl, n, true, true};
  const bool lds = n <= SV_CLAUSES;
  if (lds)
    for (uint32_t q = tid; q < n; q += SV_BLOCK) L.cl[q] = C[q];
  __syncthreads();
  auto in_lds = [&](uint32_t q) { return L.cl[q]; };
  auto in_memory = [&](uint32_t q) { return C[q]; };
  if (phase == PH_GREEDY && (lds ? greedy_solve<true>(J, K.w, st, n, in_lds, L, turn)
                                 : greedy_solve<false>(J, K.w, st, n, in_memory, L, turn)))
    return R;
  R.sat = lds ? propagate<false>(in_lds, n, all, K.less, R.on, R.off, L, turn)
              : propagate<false>(in_memory, n, all, K.less, R.on, R.off, L, turn);
  if (R.sat && !lds) {
    // the open clauses alone, restricted, into LDS if they fit, else into the
    // first phi_cap clauses of scratch (which hold at least n)
    uint64_t open = 0;
    if (tid == 0) L.cnt = 0;
    __syncthreads();
    for (uint32_t q = tid; q < n; q += SV_BLOCK) {
      const rp_clause c = C[q];
      if (!(c.pos & R.on) && !(c.neg & R.off)) open++;
    }
    if (open) atomicAdd(&L.cnt, (uint32_t)open);
    __syncthreads();
    if (L.cnt > SV_CLAUSES) R.U = J.scratch;
    __syncthreads();
    if (tid == 0) L.cnt = 0;
    __syncthreads();
    for (uint32_t q = tid; q < n; q += SV_BLOCK) {
      const rp_clause c = C[q];
      if ((c.pos & R.on) || (c.neg & R.off)) continue;
      R.U[atomicAdd(&L.cnt, 1u)] = rp_clause{c.pos & ~R.off, c.neg & ~R.on};
    }
    __syncthreads();
    R.nu = L.cnt;
  }
  // restrict, drop the satisfied and the subsumed; reduce again until that
  // changes nothing, or until a wave can hold them
  while (R.sat && R.nu && R.U == L.cl) {
    for (uint32_t q = tid; q < R.nu; q += SV_BLOCK) {
      const rp_clause c = L.cl[q];
      L.cl[q] = (c.pos & R.on) || (c.neg & R.off) ? rp_clause{~0ull, ~0ull}     // (a tautology)
                                                  : rp_clause{c.pos & ~R.off, c.neg & ~R.on};
    }
    if (tid == 0) L.cnt = 0;
    __syncthreads();
    for (uint32_t q = tid; q < R.nu; q += SV_BLOCK) {
      const rp_clause c = L.cl[q];
      bool dead = (c.pos & c.neg) != 0;
      for (uint32_t r = 0; r < R.nu && !dead; r += 8) {      // (eight reads in flight)
#pragma unroll
        for (uint32_t k = 0; k < 8; k++) {
          const rp_clause d = L.cl[r + k];
          dead = dead || (r + k < R.nu && (d.pos & ~c.pos) == 0 && (d.neg & ~c.neg) == 0 &&
                          (d.pos != c.pos || d.neg != c.neg || r + k < q));
        }
      }
      if (!dead) L.u[atomicAdd(&L.cnt, 1u)] = c;
    }
    __syncthreads();
    R.nu = L.cnt;
    const uint64_t fixed = R.on | R.off;
    const bool few = R.nu <= WV_CLAUSES;
    if (!few)
      R.sat = propagate<true>([&](uint32_t q) { return L.u[q]; }, R.nu, all, K.less, R.on, R.off, L, turn);
    __syncthreads();
    for (uint32_t q = tid; q < R.nu; q += SV_BLOCK) L.cl[q] = L.u[q];
    __syncthreads();
    if (few || fixed == (R.on | R.off)) break;
  }
  R.answered = false;
  if (!R.sat || R.nu <= WV_CLAUSES) return R;
  R.left = all & ~R.on & ~R.off;
  if (R.left && R.U == L.cl && intervals_of(R.U, R.nu, R.left, L, turn)) {
    if (!interval_optimum(R.left, K.w, J.node_limit, L.first[lane], L.last[lane], R.result)) {
      if (tid == 0) { st->err = ERR_NODES; st->state = ST_ERROR; }
      R.answered = true;
    }
    R.left = 0;
  }
  return R;
}

// The components of the slots left, with their nu open clauses U: the result,
// or none (a final state).
struct Found {
  uint64_t result;
  bool ok;
};
__device__ __noinline__ Found solve_components(const Job& J, JobState* st, const rp_clause* U,
                                               uint32_t nu, uint64_t left, const SlotKeys& K,
                                               SolveLds& L) {
  uint64_t *smA = L.smA, *smB = L.smB;
  const int tid = threadIdx.x, lane = __lane_id(), wv = tid >> 6;
  const bool paths = U == L.cl;            // (a component over more clauses is refused below)
  uint32_t turn = 0;
  uint64_t result = 0;
  while (left) {
    // ---- 3. component of the lowest free slot
    uint64_t comp = left & (~left + 1);
    for (;;) {
      uint64_t add[1] = {0};
      for (uint32_t q = tid; q < nu; q += SV_BLOCK) {
        const uint64_t l = U[q].pos | U[q].neg;
        if ((l & comp) && (l & ~comp)) add[0] |= l;
      }
      block_or(add, L, turn);
      if ((add[0] & ~comp) == 0) break;
      comp |= add[0];
    }
    left &= ~comp;
    const int k = __popcll(comp);
    if (paths && intervals_of(U, nu, comp, L, turn)) {
      uint64_t x;
      if (!interval_optimum(comp, K.w, J.node_limit, L.first[lane], L.last[lane], x)) {
        if (tid == 0) { st->err = ERR_NODES; st->state = ST_ERROR; }
        return Found{0, false};
      }
      result |= x;
      continue;
    }
    // local slot numbering
    if (tid < 64 && ((comp >> lane) & 1)) {
      const uint32_t b = (uint32_t)__popcll(comp & lanemask_lt());
      L.gslot[b] = lane;
      L.kh[b] = (uint64_t)K.w[lane] * 128u + 1u;
      L.kl[b] = 1ull << lane;
    }
    if (tid == 0) L.cnt = 0;
    __syncthreads();
    // component clauses in local numbering (lp / ln); aux = the low slots'
    // pattern of a clause to enumerate, the lower bound of one to search
    const bool enumerate = k <= ENUM_MAX;
    const int low = k < 6 ? k : 6;
    const uint64_t lowmask = (1ull << low) - 1;
    for (uint32_t q = tid; q < nu; q += SV_BLOCK) {
      const rp_clause c = U[q];
      if (!((c.pos | c.neg) & comp)) continue;
      uint64_t lp = 0, ln = 0, lb = ~0ull;
      for (int b = 0; b < k; b++) {
        const uint64_t g = 1ull << L.gslot[b];
        if (c.pos & g) { lp |= 1ull << b; lb = L.kh[b] < lb ? L.kh[b] : lb; }
        if (c.neg & g) ln |= 1ull << b;
      }
      if (enumerate) {
        lb = 0;
        for (uint64_t m = lp & lowmask; m; m &= m - 1) lb |= pat(__builtin_ctzll(m));
      } else if (lp == 0) {
        lb = 0;
      }
      const uint32_t slot = atomicAdd(&L.cnt, 1u);
      if (slot < SV_CLAUSES) { L.lp[slot] = lp; L.ln[slot] = ln; L.la[slot] = lb; }
    }
    __syncthreads();
    const uint32_t nc = L.cnt;
    if (nc > SV_CLAUSES) {
      if (tid == 0) { st->err = ERR_SCRATCH; st->state = ST_ERROR; }
      return Found{0, false};
    }
    Key best = {~0ull, ~0ull};
    if (enumerate) {
      // ---- 4. bit-sliced enumeration
      if (tid < 64) {
        uint64_t h = 0, l = 0;
        for (int b = 0; b < low; b++)
          if ((tid >> b) & 1) { h += L.kh[b]; l |= L.kl[b]; }
        L.lowh[tid] = h;
        L.lowl[tid] = l;
      }
      __syncthreads();
      if (tid < 64) {   // rank of pattern tid by key
        uint32_t rk = 0;
        const Key me = {L.lowh[tid], L.lowl[tid]};
        for (int o = 0; o < 64; o++) {
          const Key ot = {L.lowh[o], L.lowl[o]};
          if (key_lt(ot, me) || (ot.hi == me.hi && ot.lo == me.lo && o < tid)) rk++;
        }
        L.order[rk] = tid;
      }
      __syncthreads();
      const uint64_t valid = low == 6 ? ~0ull : ((1ull << (1u << low)) - 1);
      const uint32_t nwords = 1u << (k - low);
      for (uint32_t H = tid; H < nwords; H += SV_BLOCK) {
        uint64_t feas = valid;
        const uint64_t hbits = (uint64_t)H << low;
        for (uint32_t q = 0; q < nc && feas; q++) {
          if (L.lp[q] & hbits) continue;
          uint64_t s = L.la[q];
          const uint64_t ln = L.ln[q];
          if (ln) {
            if (ln & ~hbits & ~lowmask) continue;
            for (uint64_t m = ln & lowmask; m; m &= m - 1) s |= ~pat(__builtin_ctzll(m));
          }
          feas &= s;
        }
        if (!feas) continue;
        Key kh = {0, 0};
        uint64_t m = hbits;
        while (m) {
          const int b = __ffsll((unsigned long long)m) - 1;
          m &= m - 1;
          kh.hi += L.kh[b];
          kh.lo |= L.kl[b];
        }
        for (int o = 0; o < 64; o++) {
          const uint32_t pt = L.order[o];
          if ((feas >> pt) & 1) {
            const Key cand = {kh.hi + L.lowh[pt], kh.lo | L.lowl[pt]};
            if (key_lt(cand, best)) best = cand;
            break;
          }
        }
      }
      best = block_min_key(best, smA, smB);
    } else {
      // ---- 5. depth-first branch and bound by every wave
      if (tid == 0) {
        L.bound = ~0ull;
        L.overflow = 0;
      }
      __syncthreads();
      {
        DfsFrame* stk = L.stack[wv];
        Key inc = {~0ull, ~0ull};
        bool found = false;
        uint64_t nodes = 0;
        uint32_t split_idx = 0;      // nodes met at SPLIT_DEPTH so far
        int depth = 0;
        // a frame is pushed only after its node was evaluated: todo holds
        // the free literals of the chosen open clause
        uint64_t ones = 0, zeros = 0;
        Key key = {0, 0};
        bool eval_pending = true;
        bool overflow = false;
        while (true) {
          if (eval_pending) {
            eval_pending = false;
            bool mine = true;
            if (depth == SPLIT_DEPTH) mine = (split_idx++ % SV_WAVES) == (uint32_t)wv;
            // above the split every wave evaluates every node alike (no
            // bound pruning there, so the numbering agrees); below it a node
            // no better than a known weight is skipped
            const uint64_t bound = depth >= SPLIT_DEPTH
                                       ? (uint64_t)__hip_atomic_load(&L.bound, __ATOMIC_RELAXED,
                                                                     __HIP_MEMORY_SCOPE_WORKGROUP)
                                       : ~0ull;
            if (mine) nodes++;
            if (nodes > J.node_limit) { overflow = true; break; }
            const bool skip = !mine || (depth >= SPLIT_DEPTH &&
                                        ((found && !key_lt(key, inc)) || key.hi > bound));
            if (!skip) {
              uint64_t dead = 0, pick = ~0ull, lbmax = 0;
              for (uint32_t q = lane; q < nc; q += 64) {
                const uint64_t lp = L.lp[q], ln = L.ln[q];
                if ((lp & ones) || (ln & ~ones)) continue;   // satisfied with undecided = 0
                const uint64_t fr = lp & ~zeros;
                if (fr == 0) { dead = 1; continue; }
                const uint64_t cand = ((uint64_t)__popcll(fr) << 32) | q;
                pick = cand < pick ? cand : pick;
                lbmax = L.la[q] > lbmax ? L.la[q] : lbmax;
              }
              dead = wave_or(dead);
              pick = wave_min_u64(pick);
              lbmax = wave_max_u64(lbmax);
              if (!dead) {
                if (pick == ~0ull) {
                  // every clause holds: a solution
                  if (!found || key_lt(key, inc)) {
                    inc = key;
                    found = true;
                    if (lane == 0)
                      __hip_atomic_fetch_min(&L.bound, (unsigned long long)key.hi,
                                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                  }
                } else if (depth < SPLIT_DEPTH ||
                           !((found && key.hi + lbmax > inc.hi) || key.hi + lbmax > bound)) {
                  const uint32_t q = (uint32_t)(pick & 0xFFFFFFFFu);
                  // every lane writes the same frame, so each lane's later
                  // read follows its own write
                  DfsFrame f;
                  f.ones = ones; f.zeros = zeros; f.khi = key.hi; f.klo = key.lo;
                  f.todo = L.lp[q] & ~zeros; f.tried = 0;
                  stk[depth] = f;
                  __builtin_amdgcn_wave_barrier();
                  depth++;
                }
              }
            }
          }
          // next branch of the deepest frame with literals left
          if (depth == 0) break;
          __builtin_amdgcn_wave_barrier();
          DfsFrame f = stk[depth - 1];
          if (f.todo == 0) { depth--; continue; }
          const uint64_t sbit = f.todo & (~f.todo + 1);
          const int b = __ffsll((unsigned long long)sbit) - 1;
          __builtin_amdgcn_wave_barrier();
          stk[depth - 1].todo = f.todo & ~sbit;
          stk[depth - 1].tried = f.tried | sbit;
          __builtin_amdgcn_wave_barrier();
          ones = f.ones | sbit;
          zeros = f.zeros | f.tried;
          key.hi = f.khi + L.kh[b];
          key.lo = f.klo | L.kl[b];
          eval_pending = true;
        }
        if (lane == 0) {
          if (overflow) atomicOr(&L.overflow, 1u);
          L.inch[wv] = found ? inc.hi : ~0ull;
          L.incl[wv] = found ? inc.lo : ~0ull;
        }
      }
      __syncthreads();
      if (L.overflow) {
        if (tid == 0) { st->err = ERR_NODES; st->state = ST_ERROR; }
        return Found{0, false};
      }
      best.hi = L.inch[0];
      best.lo = L.incl[0];
      for (int q = 1; q < SV_WAVES; q++) {
        const Key o = {L.inch[q], L.incl[q]};
        if (key_lt(o, best)) best = o;
      }
      __syncthreads();
    }
    if (best.hi == ~0ull && best.lo == ~0ull) {
      if (tid == 0) st->state = ST_UNSAT;
      return Found{0, false};
    }
    result |= best.lo;   // lo is the global mask of the component's optimum
    __syncthreads();
  }
  return Found{result, true};
}

// Solve over phi = C[0..n) for the job state *st (in LDS; thread 0 writes it):
// x and weight, or a final state.  K: the job's keys (LDS).  Every
// thread of the workgroup calls it.
__device__ __forceinline__ void solve_body(const Job& J, JobState* st, const rp_clause* C, uint32_t n,
                                           const SlotKeys& K, SolveLds& L) {
  const int tid = threadIdx.x, wv = tid >> 6;
  const uint32_t S = J.S;
  const uint64_t all = S >= 64 ? ~0ull : ((1ull << S) - 1);
  const uint32_t phase = st->phase;
  uint64_t on = 0, off = 0, result = 0, left = 0;
  bool sat = true;
  const rp_clause* U = C;                  // the clauses to reduce further
  uint32_t nu = n;
  __syncthreads();          // (every thread has the phase before thread 0 may change it)
  // ---- 1. reduction
  if (n <= WV_CLAUSES) {
    if (phase == PH_GREEDY && (n <= 64 ? greedy_wave(S, K.w, st, wave_clauses<1>(C, n))
                                       : greedy_wave(S, K.w, st, wave_clauses<2>(C, n))))
      return;
  } else {
    const Reduced R = reduce_many(J, st, C, n, all, phase, K, L);
    if (R.answered) return;
    on = R.on;
    off = R.off;
    result = R.result;
    left = R.left;
    sat = R.sat;
    U = R.U;
    nu = R.nu;
  }
  if (sat && nu <= WV_CLAUSES) {
    // ---- 2. in the waves; one path over all that is left
    const bool done = nu <= 64 ? solve_wave<1>(J, st, U, nu, all, K, L, wv, on, off, sat, result, left)
                               : solve_wave<2>(J, st, U, nu, all, K, L, wv, on, off, sat, result, left);
    if (!done) return;
    U = L.cl;
  }
  if (!sat) {
    if (tid == 0) st->state = ST_UNSAT;
    return;
  }
  result |= on;
  if (left) {
    const Found f = solve_components(J, st, U, nu, left, K, L);
    if (!f.ok) return;
    result |= f.result;
  }
  const uint64_t weight = weight_of(result, K.w);
  if (tid == 0) {
    if (phase == PH_FINAL) {
      // the exact query after the greedy answer was verified SAFE
      st->phase = PH_EXACT;
      if (result == st->x) {
        st->weight = weight;
        st->state = ST_SAFE;
        return;
      }
    }
    st->x = result;
    st->weight = weight;
    if (st->max_rounds && st->rounds >= st->max_rounds) st->state = ST_ROUNDS;
  }
}

}  // namespace rp
