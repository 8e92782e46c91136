// Host-side plan of a kernel model and the multi-job execution engine.
#pragma once
#include <algorithm>
#include <atomic>
#include <thread>
#include <vector>

#include "common.h"

namespace rp {

struct PlanGuard {                  // a guard over the kernel's threads and blocks
  uint32_t cnt;                     // executing threads of a block
  uint32_t bm, br, nblk;            // block condition, executing blocks
};
struct PlanArray {
  uint32_t off = 0;                 // rotation of its words in the log
  bool bounded = false;             // the closed form's bound can take it
  bool closed = false;              // decided in closed form: no records
  int form = FORM_PLAIN;            // the narrowest form it fits
  // the bound: tests, their cost with the gcds, the longest chain of tests in one
  // lane; the cost beyond the records' own (0 if it cannot)
  double tests = 0, cost = 0, serial = 0, over = 0;
  double rec = 0;                   // records of all its accesses
  uint64_t intra = 0, inter = 0;    // records per block, cross-block records
};

// What the host works out of a kernel model.  The kernel's descriptors have
// to stay where they are while the plan is used.
struct Plan {
  const rp_kernel* k = nullptr;     // NULL: a lone Solve (weights then)
  uint32_t P = 0, S = 0, B = 0, T = 0;
  uint32_t tbits = 0, bbits = 0, pbits = 0, nbits = 0, abits = 0, key_shift = 0, key_bits = 0;
  std::vector<PlanGuard> guards;
  std::vector<PlanArray> arrays;
  std::vector<uint32_t> weights;    // of a lone Solve
  uint64_t div_if_enabled = 0, grid_slots = 0, pre_slots = 0;
  uint32_t pad_array = 0;           // array id of padding records (block conditions)
  // records of a log of every access (workspace sizes follow these whether or
  // not the records are generated), and of the arrays outside the closed form
  uint64_t n_intra = 0, n_inter = 0, accesses = 0;
  uint64_t log_intra = 0, log_inter = 0;
  uint64_t rblk = 0;                // same-block records per block
  double over = 0;                  // of its arrays together
  bool log = false;                 // some array's accesses have to be records
  bool any_closed = false;          // some array is decided in closed form
  int closed_form = FORM_PLAIN;     // the narrowest form all of these fit
  bool packed = false;              // its first partners are the rounds kernel's
};

int validate_kernel(const rp_kernel* k);
void make_plan(const rp_kernel* k, Plan& pl);
// Which arrays of a call's kernels are decided in closed form.  make_plan has
// done it for its kernel alone; a call over several decides them together (its
// launches, which make room for work beyond the records' own, are shared).
void choose_routes(Plan* const* plans, size_t n);
// The device's point table, and the prefix tables of its records ([P + 1]).
void fill_points(const Plan& pl, DPoint* pts);
void fill_prefixes(const Plan& pl, const DPoint* pts, uint64_t* cnt_pre, uint64_t* gcnt_pre);

// Runs fn(first, last) over [0, n) on the calling thread and, where the work
// (in points) is worth the threads' start, a few more: planning takes 7 to 12
// ns per point (62 us for 16 kernels of 8,469 points, 773 us for 120 of
// 61,797), a thread's start and end about 8 us (1 to 15 at once 18 to 112
// us), so a thread gets at least 8K points.
template <class F>
void over_jobs(uint32_t n, uint64_t points, F fn) {
  unsigned nth = (unsigned)std::min<uint64_t>(
      std::min<unsigned>(16, std::max(1u, std::thread::hardware_concurrency())), points / 8192);
  nth = std::min<unsigned>(nth, n);
  if (nth < 2) {
    fn(0u, n);
    return;
  }
  std::atomic<uint32_t> next(0);
  const uint32_t step = std::max(1u, n / (nth * 8));
  auto work = [&]() {
    for (;;) {
      const uint32_t j = next.fetch_add(step);
      if (j >= n) break;
      fn(j, std::min(n, j + step));
    }
  };
  std::vector<std::thread> pool;
  pool.reserve(nth);
  try {
    for (unsigned t = 1; t < nth; t++) pool.emplace_back(work);
  } catch (...) {                   // no more threads to be had: the others do it all
  }
  work();
  for (std::thread& t : pool) t.join();
}

int pick_digit_bits(uint32_t key_bits);
// One radix pass: it sorts by key bits [lo, lo + bits) above the key shift.
struct DigitPass {
  uint32_t lo, bits;
};
// The radix passes of a key of key_bits bits, in execution order: digits of
// the automatic or set width (RP_TUNE_SORT_DIGIT_BITS), or with the lowest
// digit of RP_TUNE_LOW_DIGIT_BITS bits and the rest split evenly into
// digits of at most 10 bits; highest digit first or lowest first
// (RP_TUNE_DIGIT_ORDER).
std::vector<DigitPass> digit_plan(uint32_t key_bits);
// Width of the lowest digit (RP_TUNE_LOW_DIGIT_BITS, 0 = digits of one
// width); returns the old setting.
int low_digit_bits(int v, bool set);
// hipEvent timing level of engine calls (RP_TUNE_TIMING); returns the old one
int timing_level(int v, bool set);
// Order of the radix passes' digits (RP_TUNE_DIGIT_ORDER: 0 lowest first,
// 1 highest first); returns the old setting.
int digit_order(int v, bool set);
// First partners in closed form where the plan's rule takes it, or from the
// records always (RP_TUNE_RACE_ROUTE 0, 1); returns the old setting.
int race_route(int v, bool set);
// Node budget of the exact solver's branch and bound (RP_TUNE_SOLVER_NODES,
// as log2); returns the old log2.
int solver_nodes_log2(int v, bool set);
// Library status of a job that ended in ST_ERROR.
int job_error_status(const JobState& st);
// rp_repair_out of a repair job from its final state.
void fill_repair_out(const JobState& s, const Plan& pl, rp_repair_out& out);
// Unit clauses that the repair options impose before the first Solve.
std::vector<rp_clause> option_units(const Plan& pl, const rp_repair_opts& o);

enum Op { OP_CHECK = 0, OP_CLAUSES = 1, OP_REPAIR = 2, OP_SOLVE = 3, OP_FIRST = 4 };

struct JobInput {
  const Plan* plan;
  uint64_t x = 0;                   // assignment (check / clauses; a repair starts at 0)
  std::vector<rp_clause> phi0;      // initial constraint set (repair: option units)
  uint32_t policy = 0, max_rounds = 0;
  uint32_t solver = 0;              // 0 exact Solve, 1 greedy hitting set (mhs)
};

struct JobResult {
  JobState st;
  std::vector<rp_clause> phi;       // clauses mode: reduced learned clauses
  std::vector<uint32_t> first;      // first-partner mode: [2][P]
  uint64_t n_pairs = 0;
  std::vector<uint64_t> traj;
};

struct EngineOpts {
  Op op = OP_REPAIR;
  uint64_t pair_cap = 0;            // check: caller's capacity
  uint32_t traj_cap = 0;
  rp_pair* pair_out = nullptr;      // check of one job: the caller's list (at most pair_cap)
  bool no_alloc = false;            // stage through ordinary host memory, record no
                                    // timing events (no device or page-locked allocation)
};

// Bytes of workspace the engine needs for these jobs.
size_t engine_workspace(const std::vector<JobInput>& jobs, const EngineOpts& o);

// One job prepared in its own device region (serving): a host copy of its
// device job table entry, with absolute device pointers.
struct PreparedJob {
  Job job;
};
size_t engine_job_bytes(const JobInput& job);
// Bytes of one region holding a group of jobs prepared together.
size_t engine_group_bytes(const std::vector<JobInput>& jobs);
// Enqueues upload, record generation, sort, run logs, the first-partner
// tables and the first Solve of a group of jobs into one region, with one
// launch per phase for the whole group; out[j] is job j's device table
// entry.  staging must stay alive until the stream is synced.
int engine_prepare_group(const std::vector<JobInput>& jobs, void* region, size_t bytes,
                         hipStream_t s, std::vector<PreparedJob>& out,
                         std::vector<uint8_t>& staging);
// Enqueues one round (Verify, GenerateClause, Solve) over the device table of
// njobs prepared jobs.
int engine_round(const Job* djobs, uint32_t njobs, hipStream_t s);

// Runs the op over all jobs; returns RP_OK or an error status.
int engine_run(const std::vector<JobInput>& jobs, const EngineOpts& o, void* ws, size_t ws_bytes,
               hipStream_t s, std::vector<JobResult>& res, rp_stats* stats);

}  // namespace rp
