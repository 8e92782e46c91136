// The rounds of Alg. 1 (Verify, GenerateClause, Solve until a verdict), one
// workgroup per job, in one launch.
//
// What a round needs of the accesses does not depend on the assignment.  A row
// (point i, view) whose first partner with no barrier enabled is j races under
// x exactly when no enabled occurrence lies between i and j, that is, when x
// meets none of the slots with an occurrence between them (grid-level ones
// for the cross-block view): when x & mask = 0 for the row's slot mask, which
// is also its clause.  A row whose occurrences include another's races only if
// that one does, with a weaker clause.  So the tables are built once per job
// (build_tables): for each view the inclusion-minimal occurrence intervals,
// as slot masks, reduced over both views (sorted, no duplicate, no superset):
// the reduced set F of every race clause the kernel can ever give.  Then
//   Verify          tests x against the masks of F and the divergent slots;
//   GenerateClause  appends the violated masks and the units of the divergent
//                   slots to phi.  x satisfies phi, so what it violates is
//                   neither in phi nor a superset of a clause there; and F has
//                   no proper subsets in it, so phi stays reduced.  An empty
//                   mask (two racing points with no slot between them) makes
//                   phi = {empty};
//   one trace per call (policy 1) takes the smallest divergent slot, else the
//                   smallest racing row with its own mask, which need not be
//                   in F: phi drops its supersets;
//   Solve           solve.h.
// Bound: latency of a chain of small steps of one workgroup (tens to hundreds
// of masks and clauses).  With four launches per round (interval scan, clause
// sort and subsumption, Solve, count of running jobs) and a host wait, the
// rounds of the small planted kernel took 84 us with their waits, of 512
// instrumented programs 1.9 ms; in one launch, with the small kernel's first
// partners, 12 us, and 0.09 ms.
#include "closed_rows.h"
#include "common.h"
#include "launch.h"
#include "solve.h"

namespace rp {

constexpr int RD_BLOCK = SV_BLOCK;
constexpr int RD_WAVES = RD_BLOCK / 64;
constexpr uint32_t RD_MASKS = 1536;        // masks reduced in LDS; more in the job's scratch
constexpr uint32_t ROUNDS_MAX = 100000;    // a job still running after that many has failed

struct BuildLds {
  uint8_t occ[2][MAX_POINTS];              // slot of each barrier occurrence (any, grid level)
  uint16_t next[2][MAX_POINTS + 1];        // occurrences before each point
  uint32_t end[MAX_POINTS + 1];            // shortest interval from each occurrence
  uint64_t raw[RD_MASKS];
  uint32_t dead[2 * MAX_POINTS / 32];
};

union RoundLds {
  PackedLds<RD_WAVES> p;
  BuildLds b;
  SolveLds s;
};

// The job's tables behind the first phi_cap clauses of its scratch (which has
// at least 2 P + 64 clauses of 16 bytes more): F, at most 2 P masks, and the
// masks of the racing rows.
__device__ __forceinline__ uint64_t* full_of(const Job& J) { return (uint64_t*)(J.scratch + J.phi_cap); }
__device__ __forceinline__ uint64_t* rows_of(const Job& J) { return full_of(J) + 2 * (uint64_t)J.P; }

__device__ __forceinline__ uint64_t block_excl_scan(uint64_t v, uint64_t* sm, uint64_t* total) {
  const uint32_t lane = __lane_id(), w = threadIdx.x >> 6;
  uint64_t inc = v;
  for (int o = 1; o < 64; o <<= 1) {
    const uint64_t y = __shfl_up(inc, o);
    if (lane >= (uint32_t)o) inc += y;
  }
  if (lane == 63) sm[w] = inc;
  __syncthreads();
  uint64_t pre = 0, tot = 0;
  for (uint32_t q = 0; q < (uint32_t)RD_WAVES; q++) {
    if (q < w) pre += sm[q];
    tot += sm[q];
  }
  __syncthreads();
  *total = tot;
  return pre + inc - v;
}

// Rank of this thread among those of the workgroup with hit, and their number.
__device__ __forceinline__ uint32_t block_rank(bool hit, uint64_t* sm, uint32_t* total) {
  const uint32_t w = threadIdx.x >> 6;
  const uint64_t m = __ballot(hit);
  if (__lane_id() == 0) sm[w] = (uint64_t)__popcll(m);
  __syncthreads();
  uint32_t pre = 0, tot = 0;
  for (uint32_t q = 0; q < (uint32_t)RD_WAVES; q++) {
    if (q < w) pre += (uint32_t)sm[q];
    tot += (uint32_t)sm[q];
  }
  __syncthreads();
  *total = tot;
  return pre + (uint32_t)__popcll(m & lanemask_lt());
}

// Builds F and, if rows, the masks of the racing rows (their sizes into
// st->n_full, low and high half).
__device__ void build_tables(const Job& J, JobState* st, bool rows, BuildLds& L, uint64_t* sm) {
  const uint32_t tid = threadIdx.x, lane = __lane_id(), wv = tid >> 6, P = J.P;
  const uint32_t per = (P + RD_BLOCK - 1) / RD_BLOCK;
  // ---- occurrences in program order
  uint64_t cnt = 0;
  for (uint32_t q = 0; q < per; q++) {
    const uint32_t i = tid * per + q;
    if (i < P) cnt += (slot_any(J.pts[i]) ? 1ull : 0ull) + (slot_grid(J.pts[i]) ? 1ull << 32 : 0ull);
  }
  uint64_t nocc;
  uint64_t at = block_excl_scan(cnt, sm, &nocc);
  for (uint32_t q = 0; q < per; q++) {
    const uint32_t i = tid * per + q;
    if (i >= P) break;
    const uint64_t a = slot_any(J.pts[i]), g = slot_grid(J.pts[i]);
    const uint32_t ta = (uint32_t)at, tg = (uint32_t)(at >> 32);
    L.next[0][i] = (uint16_t)ta;
    L.next[1][i] = (uint16_t)tg;
    if (a) L.occ[0][ta] = (uint8_t)__builtin_ctzll(a);
    if (g) L.occ[1][tg] = (uint8_t)__builtin_ctzll(g);
    at += (a ? 1ull : 0ull) + (g ? 1ull << 32 : 0ull);
  }
  __syncthreads();
  // slots of the occurrences [a, b) of a view
  auto mask_of = [&](uint32_t lv, uint32_t a, uint32_t b) {
    uint64_t m = 0;
    for (uint32_t t = a; t < b; t++) m |= 1ull << L.occ[lv][t];
    return m;
  };
  // ---- minimal intervals of each view: an interval is one unless another
  // with a later start ends no later
  uint32_t m = 0;                          // masks so far
  bool empty = false;
  uint32_t n_rows = 0;
  uint64_t* const big = (uint64_t*)J.scratch;      // (free until the first Solve)
  for (uint32_t lv = 0; lv < 2; lv++) {
    const uint32_t n = lv ? (uint32_t)(nocc >> 32) : (uint32_t)nocc;
    for (uint32_t t = tid; t <= n; t += RD_BLOCK) L.end[t] = NONE32;
    __syncthreads();
    for (uint32_t i = tid; i < P; i += RD_BLOCK) {
      const uint32_t j = J.j0[(uint64_t)lv * P + i];
      if (j >= P) continue;
      const uint32_t a = L.next[lv][i], b = L.next[lv][j];
      atomicMin(&L.end[a], b);
    }
    // the racing rows' masks, in the order of their points
    for (uint32_t b0 = 0; rows && b0 < P; b0 += RD_BLOCK) {
      const uint32_t i = b0 + tid;
      const uint32_t j = i < P ? J.j0[(uint64_t)lv * P + i] : NONE32;
      uint32_t total;
      const uint32_t at = block_rank(j < P, sm, &total);
      if (j < P) rows_of(J)[n_rows + at] = mask_of(lv, L.next[lv][i], L.next[lv][j]);
      n_rows += total;
    }
    __syncthreads();
    const uint32_t pt = n / RD_BLOCK + 1;  // starts of this thread, [t0, t1)
    const uint32_t t0 = tid * pt < n + 1 ? tid * pt : n + 1, t1 = t0 + pt < n + 1 ? t0 + pt : n + 1;
    uint32_t low = NONE32;                 // least end of this thread's starts
    for (uint32_t t = t0; t < t1; t++) low = L.end[t] < low ? L.end[t] : low;
    // least end of all later threads' starts
    uint32_t suf = low;
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t y = __shfl_down(suf, o);
      if (lane + (uint32_t)o < 64 && y < suf) suf = y;
    }
    if (lane == 0) sm[wv] = suf;
    uint32_t after = __shfl_down(suf, 1);
    if (lane == 63) after = NONE32;
    __syncthreads();
    for (uint32_t w = wv + 1; w < (uint32_t)RD_WAVES; w++) after = (uint32_t)sm[w] < after ? (uint32_t)sm[w] : after;
    __syncthreads();
    uint32_t keep = 0;
    {
      uint32_t least = after;
      for (uint32_t t = t1; t-- > t0;) {
        const uint32_t e = L.end[t];
        if (e < least) {
          least = e;
          keep++;
        }
      }
    }
    uint64_t total;
    uint32_t pos = m + (uint32_t)block_excl_scan(keep, sm, &total);
    uint32_t least = after;
    for (uint32_t t = t1; t-- > t0;) {
      const uint32_t e = L.end[t];
      if (e >= least) continue;
      least = e;
      const uint64_t mk = mask_of(lv, t, e);
      if (mk == 0) empty = true;
      if (pos < RD_MASKS) L.raw[pos] = mk;
      big[pos] = mk;                       // (all of them, for when there are many)
      pos++;
    }
    m += (uint32_t)total;
    __syncthreads();
  }
  // ---- F: duplicates and supersets dropped, ascending
  uint32_t any_empty;
  (void)block_rank(empty, sm, &any_empty);
  uint64_t* const F = full_of(J);
  if (any_empty) {
    if (tid == 0) {
      F[0] = 0;
      st->n_full = 1 | n_rows << 16;
    }
    __syncthreads();
    return;
  }
  const uint64_t* raw = m <= RD_MASKS ? L.raw : big;
  for (uint32_t q = tid; q < (m + 31) / 32; q += RD_BLOCK) L.dead[q] = 0;
  __syncthreads();
  for (uint32_t q = tid; q < m; q += RD_BLOCK) {
    const uint64_t c = raw[q];
    bool dead = false;
    for (uint32_t r = 0; r < m && !dead; r++) {
      const uint64_t d = raw[r];
      dead = (d & ~c) == 0 && (d != c || r < q);
    }
    if (dead) atomicOr(&L.dead[q >> 5], 1u << (q & 31));
  }
  __syncthreads();
  uint64_t alive = 0;
  for (uint32_t q = tid; q < m; q += RD_BLOCK) {
    if ((L.dead[q >> 5] >> (q & 31)) & 1) continue;
    const uint64_t c = raw[q];
    uint32_t rank = 0;
    for (uint32_t r = 0; r < m; r++)
      rank += raw[r] < c && !((L.dead[r >> 5] >> (r & 31)) & 1);
    F[rank] = c;
    alive++;
  }
  uint64_t total;
  (void)block_excl_scan(alive, sm, &total);
  if (tid == 0) st->n_full = (uint32_t)total | n_rows << 16;
  __syncthreads();
}

// GenerateClause over every trace under x: the divergent slots' units and the
// masks of F that x misses, behind the n clauses of phi.  Returns the number
// of clauses of phi (the caller has checked that something is learned).
__device__ __forceinline__ uint32_t learn_all(rp_clause* phi, uint32_t cap, uint64_t x, uint64_t div, uint32_t n,
                              const uint64_t* F, uint32_t n_full, uint64_t* sm) {
  const uint32_t tid = threadIdx.x;
  if (n_full == 1 && F[0] == 0) {
    __syncthreads();
    if (tid == 0) phi[0] = rp_clause{0, 0};
    return 1;
  }
  if (tid < 64 && ((div >> tid) & 1)) {
    const uint32_t at = n + (uint32_t)__popcll(div & ((1ull << tid) - 1));
    if (at < cap) phi[at] = rp_clause{0, 1ull << tid};
  }
  n += (uint32_t)__popcll(div);
  for (uint32_t b = 0; b < n_full; b += RD_BLOCK) {
    const uint32_t q = b + tid;
    const uint64_t mk = q < n_full ? F[q] : ~0ull;
    const bool hit = q < n_full && (mk & x) == 0;
    uint32_t total;
    const uint32_t at = n + block_rank(hit, sm, &total);
    if (hit && at < cap) phi[at] = rp_clause{mk, 0};
    n += total;
  }
  return n;
}

// One trace: clause c joins phi, whose supersets of it leave.
__device__ __forceinline__ uint32_t learn_one(rp_clause* phi, uint32_t cap, rp_clause c, uint32_t n, uint32_t* s_n) {
  if (threadIdx.x < 64) {
    const uint32_t lane = threadIdx.x;
    uint32_t k = 0;
    for (uint32_t b = 0; b < n; b += 64) {
      const uint32_t q = b + lane;
      rp_clause p{0, 0};
      bool keep = false;
      if (q < n) {
        p = phi[q];
        keep = (c.pos & ~p.pos) != 0 || (c.neg & ~p.neg) != 0;
      }
      const uint64_t m = __ballot(keep);
      if (keep) phi[k + (uint32_t)__popcll(m & lanemask_lt())] = p;   // (never past q)
      k += (uint32_t)__popcll(m);
    }
    if (lane == 0) {
      if (k < cap) phi[k] = c;
      *s_n = k + 1;
    }
  }
  __syncthreads();
  return *s_n;
}

// What one-trace rounds (many, of small steps) read and write, in the parts of
// the solver's LDS that it leaves alone while phi has at most WV_CLAUSES
// clauses: the racing rows' masks, phi and the trajectory since it was last
// written out.  From memory each step waited for the one before it to reach L2
// and come back.  Other jobs end after a few rounds, which do not pay for the
// copy (1 us of a small kernel's 12).
constexpr uint32_t NEAR = SV_CLAUSES - WV_CLAUSES;
__device__ __forceinline__ rp_clause* near_phi(SolveLds& L) { return L.cl + WV_CLAUSES; }
__device__ __forceinline__ uint64_t* near_masks(SolveLds& L) { return L.la + WV_CLAUSES; }
__device__ __forceinline__ uint64_t* near_traj(SolveLds& L) { return L.ln + WV_CLAUSES; }

// Writes out the rounds [from, to) of the trajectory.
__device__ __forceinline__ void save_traj(const Job& J, SolveLds& L, uint32_t from, uint32_t to) {
  if (!J.traj) return;
  for (uint32_t q = from + threadIdx.x; q < to && q < J.traj_cap; q += RD_BLOCK)
    J.traj[q] = near_traj(L)[q - from];
}

// flags: RD_BUILD builds the tables (from j0, which a packed job works out
// itself first; RD_FIRST: all jobs are such); RD_SOLVE makes one Solve first (the option
// units); RD_LEARN generates the clauses under the job's assignment and stops.
// limit: rounds to run (0: until a verdict).
template <int FORM>
__global__ __launch_bounds__(RD_BLOCK) void rounds_kernel(const Job* __restrict__ jobs, int flags,
                                                          uint32_t limit, CallBlock call) {
  __shared__ RoundLds L;
  __shared__ JobState s_st;
  __shared__ uint64_t sm[RD_WAVES];
  __shared__ uint32_t s_hit[RD_WAVES], s_n;
  __shared__ SlotKeys s_keys;
  // (a call's first kernel, unless first_kernel has come before)
  const bool begins = !(flags & RD_BUILD) || (flags & RD_FIRST);
  stamp_if(call.stamps, begins ? STAMP_BEGIN : STAMP_FIRST);
  const Job& J = jobs[blockIdx.x];
  const uint32_t tid = threadIdx.x, lane = __lane_id(), wv = sv_uni(tid >> 6), P = J.P;
  JobState* st = &s_st;
  if (J.st->state != ST_RUN) return;
  if (tid < sizeof(JobState) / 4) ((uint32_t*)st)[tid] = ((const uint32_t*)J.st)[tid];
  __syncthreads();
  const bool one = J.policy == 1 && !(flags & RD_LEARN);
  if (flags & RD_BUILD)
    for (uint32_t q = tid; q < st->n_phi; q += RD_BLOCK) J.phi[q] = J.phi0[q];
  if ((flags & RD_BUILD) && J.packed) {
    packed_first<FORM, RD_WAVES>(J, L.p, begins && blockIdx.x == 0 ? call.stamps : nullptr);
    if (begins) stamp_if(call.stamps, STAMP_FIRST);
  }
  if (flags & RD_BUILD) build_tables(J, st, J.policy == 1, L.b, sm);
  const bool timed = flags & RD_TIMED;
  uint64_t t0 = timed ? wall_clock64() : 0;
  auto lap = [&](uint32_t& ticks) {        // (thread 0's clock)
    if (!timed) return;
    const uint64_t t = wall_clock64();
    if (tid == 0) ticks += (uint32_t)(t - t0);
    t0 = t;
  };
  const bool loop = flags & (RD_LOOP | RD_LEARN);
  const uint32_t n_full = st->n_full & 0xFFFFu, n_rows = st->n_full >> 16;
  const uint64_t* masks = one ? rows_of(J) : full_of(J);   // what Verify tests
  rp_clause* phi = J.phi;
  uint32_t saved = st->rounds;             // rounds of the trajectory that are written out
  bool near = one && loop && st->state == ST_RUN && st->n_phi <= WV_CLAUSES && n_rows <= NEAR;
  if (near) {
    __syncthreads();                       // (the tables' LDS is free)
    for (uint32_t q = tid; q < n_rows; q += RD_BLOCK) near_masks(L.s)[q] = masks[q];
    for (uint32_t q = tid; q < st->n_phi; q += RD_BLOCK) near_phi(L.s)[q] = phi[q];
    masks = near_masks(L.s);
    phi = near_phi(L.s);
    __syncthreads();
  }
  bool keyed = false;                      // s_keys is there (a job may end without a Solve)
  bool first = flags & RD_SOLVE;           // the Solve before the rounds
  for (uint32_t r = 0; first || (loop && st->state == ST_RUN); r++) {
    uint32_t n = st->n_phi;
    bool solve = true;
    if (!first) {
      // ---- Verify
      const uint64_t x = st->x, div = x & J.div_if_enabled;
      // (one trace: the smallest racing row, same-block rows first)
      const uint32_t nm = !one ? n_full : div == 0 ? n_rows : 0;
      uint32_t mine = NONE32;
      for (uint32_t b = wv * 64; b < nm && mine == NONE32; b += RD_BLOCK) {
        const uint64_t m = __ballot(b + lane < nm && (masks[b + lane] & x) == 0);
        if (m) mine = b + (uint32_t)__builtin_ctzll(m);
      }
      if (lane == 0) s_hit[wv] = mine;
      if (tid == 0) {
        if (near) near_traj(L.s)[st->rounds - saved] = x;
        else if (J.traj && st->rounds < J.traj_cap) J.traj[st->rounds] = x;
        st->rounds += 1;
        st->divergent = div;
      }
      __syncthreads();
      uint32_t row = NONE32;
      for (int q = 0; q < RD_WAVES; q++) row = s_hit[q] < row ? s_hit[q] : row;
      lap(st->t_check);
      if (row == NONE32 && div == 0) {
        // SAFE; under the mhs strategy the exact query still decides
        if (st->phase != PH_GREEDY || (flags & RD_LEARN)) solve = false;
        __syncthreads();
        if (tid == 0) {
          if (st->phase == PH_GREEDY) st->phase = PH_FINAL;
          else st->state = ST_SAFE;
        }
      } else {
        // ---- GenerateClause
        if (!one) {
          n = learn_all(phi, J.phi_cap, x, div, n, masks, n_full, sm);
        } else {
          rp_clause c{0, div & (~div + 1)};
          if (div == 0) c.pos = masks[row];
          n = learn_one(phi, near ? NEAR : J.phi_cap, c, n, &s_n);
        }
        __syncthreads();
        if (tid == 0) {
          st->n_phi = n;
          if (n > J.phi_cap) {
            st->err = ERR_PHI_CAP;
            st->state = ST_ERROR;
          }
        }
        if (n > J.phi_cap) solve = false;
      }
      __syncthreads();
      lap(st->t_clause);
      if (flags & RD_LEARN) break;
      if (near && (n > WV_CLAUSES || st->rounds - saved == NEAR)) {
        // written out; phi and the masks stay in memory once phi is long
        save_traj(J, L.s, saved, st->rounds);
        saved = st->rounds;
        if (n > WV_CLAUSES) {
          for (uint32_t q = tid; q < n && q < J.phi_cap; q += RD_BLOCK) J.phi[q] = phi[q];
          near = false;
          phi = J.phi;
          masks = rows_of(J);
        }
        __syncthreads();
      }
    }
    // (a lone Solve reads its clauses where they are)
    if (solve && !keyed) {
      slot_keys(J, s_keys);
      keyed = true;
      __syncthreads();
    }
    if (solve) solve_body(J, st, first && !(flags & RD_BUILD) ? J.phi0 : phi, n, s_keys, L.s);
    __syncthreads();
    if (first) {
      first = false;
      r--;
      if (timed) t0 = wall_clock64();
      continue;
    }
    lap(st->t_solve);
    if ((limit != 0 && r + 1 == limit) || r + 1 == ROUNDS_MAX) break;
  }
  __syncthreads();
  if (near) {
    save_traj(J, L.s, saved, st->rounds);
    for (uint32_t q = tid; q < st->n_phi && q < J.phi_cap; q += RD_BLOCK) J.phi[q] = phi[q];
    __syncthreads();
  }
  if (tid < sizeof(JobState) / 4) ((uint32_t*)J.st)[tid] = ((const uint32_t*)st)[tid];
  if (call.page) {
    // (a call over one job)
    const uint32_t nt = J.traj ? (st->rounds < J.traj_cap ? st->rounds : J.traj_cap) : 0;
    for (uint32_t q = tid; q < nt && q < PAGE_TRAJ; q += RD_BLOCK) call.page->traj[q] = J.traj[q];
    if (flags & RD_LEARN) {
      const uint32_t n = st->n_phi < J.phi_cap ? st->n_phi : J.phi_cap;
      for (uint32_t q = tid; q < n; q += RD_BLOCK) ((rp_clause*)call.page->tail())[q] = J.phi[q];
    }
  }
  finish_call(call, st);
}

hipError_t launch_rounds(const Job* jobs, uint32_t njobs, int form, int flags, uint32_t limit,
                         const CallBlock& call, hipStream_t s) {
  if (njobs == 0) return hipSuccess;
  if (form == FORM_WIDE) rounds_kernel<FORM_WIDE><<<njobs, RD_BLOCK, 0, s>>>(jobs, flags, limit, call);
  else rounds_kernel<FORM_SMALL><<<njobs, RD_BLOCK, 0, s>>>(jobs, flags, limit, call);
  return hipGetLastError();
}

}  // namespace rp
