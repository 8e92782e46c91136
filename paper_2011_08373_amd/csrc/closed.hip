// Conflicts in closed form (closed.h), with no access records, for the points
// whose arrays the plan marks PF_CLOSED: the table j0 of first partners
// (first_kernel), or the rows of the racing-pair bitmap under an assignment
// (all_kernel).
//
// first_kernel: one wave per (point, view).  Lanes take the 64 points from the wave's own
// point on, a chunk at a time; a lane whose point touches the same array (one
// of the two writing) decides the pair, and the lowest lane that finds a
// conflict is the first partner, so most waves end in their first chunk.
//
// Bound: instruction latency (a pair costs two or three hundred integer
// instructions in one lane, a few of them divisions; a chunk reads 64 x 40 B
// of descriptors), so the kernel is spread over as many waves as there are
// rows and the rows' chunks are not split further.  Measured: 21 us for the
// stress kernel (512 accesses of 4.2M threads; generating, sorting and
// scanning their 2.0G records took 31 ms), 17 us for plain-large (0.56 ms),
// 4 us for a 16-point kernel, 0.32 ms for 128 kernels of the batched
// distribution (9.2 ms).
#include "closed.h"
#include "common.h"
#include "launch.h"

namespace rp {

constexpr int CF_WAVES = 4;      // two points, both views

__device__ __forceinline__ bool closed_point(const DPoint& d) {
  return d.kind == RP_ACCESS && (d.flags & PF_CLOSED);
}

__device__ __forceinline__ Access access_of(const DPoint& d, uint32_t B) {
  return make_access(d.a, d.b, d.c, d.words, d.m, d.r, d.cnt, d.bm, d.br, B);
}

// Whether this lane's point j (>= i, in range) races with point i of access a
// when no barrier separates them.
template <class I>
__device__ __forceinline__ bool lane_conflict(const Job& J, const DPoint& pi, const Access& a,
                                              uint32_t i, uint32_t j, uint32_t lv) {
  const DPoint& pj = J.pts[j];
  if (pj.kind != RP_ACCESS || pj.array != pi.array || !((pi.flags | pj.flags) & PF_WRITE) ||
      pj.cnt == 0 || pj.br >= J.B)
    return false;
  const Access q = access_of(pj, J.B);
  if (lv != 0) return pair_cross_block<I>(a, q);
  return j == i ? self_same_block(a) : pair_same_block<I>(a, q, J.B);
}

// Point i has conflicts to look for in view lv at all.
__device__ __forceinline__ bool row_runs(const DPoint& pi, uint32_t B, uint32_t lv) {
  return (lv == 0 || ((pi.flags & PF_GLOBAL) && B > 1)) && pi.cnt != 0 && pi.br < B;
}

// Stamps of the first wave: when it has its own point, and when it has picked
// the points of that point's array out of the first 64 (the closed form's
// counterparts of generating the records and of grouping them by location).
__device__ __forceinline__ void stamp_gather(uint64_t* stamps, const Job& J, const DPoint& pi) {
  if (!stamps || blockIdx.x != 0 || blockIdx.y != 0 || threadIdx.x >= 64) return;
  const uint32_t l = threadIdx.x;
  asm volatile("" ::"v"((uint32_t)pi.array));      // (waits for the value)
  stamp_if(stamps, STAMP_GEN);
  const bool same = l < J.P && J.pts[l].kind == RP_ACCESS && J.pts[l].array == pi.array;
  const uint64_t m = __ballot(same);
  asm volatile("" ::"s"(m));
  stamp_if(stamps, STAMP_SORT);
}

// The first point at or after base, among the chunk's 64, with an enabled
// barrier of the view (64: none): no pair reaches past it.
__device__ __forceinline__ uint32_t chunk_limit(const Job& J, uint32_t lv, uint64_t x, uint32_t i,
                                                uint32_t j) {
  bool on = false;
  if (j > i && j < J.P) on = ((lv ? slot_grid(J.pts[j]) : slot_any(J.pts[j])) & x) != 0;
  const uint64_t m = __ballot(on);
  return m ? (uint32_t)__builtin_ctzll(m) : 64u;
}

// X = false: the table j0, with no barrier enabled.  X = true: first partners
// under the job's assignment, into minj (and the page), of a job that has no
// records at all.
template <class I, bool X>
__global__ __launch_bounds__(CF_WAVES * 64) void first_kernel(const Job* __restrict__ jobs,
                                                              CallBlock call) {
  stamp_if(call.stamps, STAMP_BEGIN);
  const Job& J = jobs[blockIdx.y];
  const uint32_t wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = __lane_id();
  const uint32_t P = J.P, B = J.B, lv = wv & 1;
  const uint32_t i = blockIdx.x * (CF_WAVES / 2) + (wv >> 1);
  if (i < P) {
    const DPoint pi = J.pts[i];
    stamp_gather(call.stamps, J, pi);
    uint32_t best = NONE32;
    if (closed_point(pi) && row_runs(pi, B, lv)) {
      const Access a = access_of(pi, B);
      const uint64_t x = X ? J.st->x : 0;
      for (uint32_t base = i; base < P; base += 64) {
        const uint32_t j = base + lane;
        const uint32_t end = X ? chunk_limit(J, lv, x, i, j) : 64u;
        const uint64_t m = __ballot(j < P && lane < end && lane_conflict<I>(J, pi, a, i, j, lv));
        if (m) best = base + (uint32_t)__builtin_ctzll(m);
        if (m || end < 64) break;
      }
    }
    const uint32_t row = lv * P + i;
    if (lane == 0) {
      if constexpr (X) {
        J.minj[row] = best;
        if (call.page) ((uint32_t*)call.page->tail())[row] = best;
      } else if (closed_point(pi) || (J.nlog[0] == 0 && J.nlog[1] == 0)) {
        // (with a log its scan has set the rows of the other points)
        J.j0[row] = best;
      }
    }
  }
  if constexpr (X) finish_call(call, J.st);
}

// Every racing pair under the job's assignment, one wave per (point, view):
// the 64-point words of the row's bitmap are ballots, kept one per lane (at
// most 64 words) and stored together.  A row ends at the first enabled barrier
// after its point.  The row's pairs are counted into minj for the list.  Bound
// by latency as above: 31 us for plain-large under a quarter of its barriers, against 1.39 ms for
// the scan of its sorted records (and 0.45 ms to generate and sort them).
template <class I>
__global__ __launch_bounds__(CF_WAVES * 64) void all_kernel(const Job* __restrict__ jobs,
                                                            CallBlock call) {
  stamp_if(call.stamps, STAMP_BEGIN);
  static_assert(MAX_POINTS <= 64 * 64, "a row's words in one wave");
  const Job& J = jobs[blockIdx.y];
  const uint32_t wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = __lane_id();
  const uint32_t P = J.P, B = J.B, lv = wv & 1;
  const uint32_t i = blockIdx.x * (CF_WAVES / 2) + (wv >> 1);
  if (i >= P) return;
  const DPoint pi = J.pts[i];
  stamp_gather(call.stamps, J, pi);
  // (with no records at all the scan of the logs has not cleared the row)
  if (!closed_point(pi) && (J.nlog[0] != 0 || J.nlog[1] != 0)) return;
  uint64_t word = 0;
  if (closed_point(pi) && row_runs(pi, B, lv)) {
    const Access a = access_of(pi, B);
    const uint64_t x = J.st->x;
    for (uint32_t base = i & ~63u; base < P; base += 64) {
      const uint32_t j = base + lane;
      const uint32_t end = chunk_limit(J, lv, x, i, j);
      const uint64_t m = __ballot(j >= i && j < P && lane < end &&
                                  lane_conflict<I>(J, pi, a, i, j, lv));
      if (lane == base >> 6) word = m;
      if (end < 64) break;
    }
  }
  const uint64_t row = (uint64_t)lv * P + i;
  if (lane < J.wpr) J.bitmap[row * J.wpr + lane] = word;
  uint32_t c = (uint32_t)__popcll(word);
  for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o);
  if (lane == 0) J.minj[row] = c;
}

static dim3 row_grid(uint32_t max_points, uint32_t njobs) {
  return dim3((max_points + CF_WAVES / 2 - 1) / (CF_WAVES / 2), njobs);
}

hipError_t launch_all_closed(const Job* job, uint32_t points, bool small, const CallBlock& call,
                             hipStream_t s) {
  if (points == 0) return hipSuccess;
  const dim3 grid = row_grid(points, 1);
  if (small) all_kernel<int32_t><<<grid, CF_WAVES * 64, 0, s>>>(job, call);
  else all_kernel<int64_t><<<grid, CF_WAVES * 64, 0, s>>>(job, call);
  return hipGetLastError();
}

template <bool X>
static hipError_t first_go(const Job* jobs, uint32_t njobs, uint32_t max_points, bool small,
                           const CallBlock& call, hipStream_t s) {
  for (uint32_t j = 0; j < njobs; j += 65535) {      // (the grid's second dimension)
    const dim3 grid = row_grid(max_points, njobs - j < 65535 ? njobs - j : 65535);
    const CallBlock c = j == 0 ? call : CallBlock{};
    if (small) first_kernel<int32_t, X><<<grid, CF_WAVES * 64, 0, s>>>(jobs + j, c);
    else first_kernel<int64_t, X><<<grid, CF_WAVES * 64, 0, s>>>(jobs + j, c);
  }
  return hipGetLastError();
}

hipError_t launch_first_closed(const Job* jobs, uint32_t njobs, uint32_t max_points, bool small,
                               const CallBlock& call, hipStream_t s) {
  if (njobs == 0 || max_points == 0) return hipSuccess;
  return first_go<false>(jobs, njobs, max_points, small, call, s);
}

hipError_t launch_first_under(const Job* job, uint32_t points, bool small, const CallBlock& call,
                              hipStream_t s) {
  return first_go<true>(job, 1, points ? points : 1, small, call, s);
}

}  // namespace rp
