// Conflicts in closed form (closed.h), with no access records, for the points
// whose arrays the plan marks PF_CLOSED: the table j0 of first partners
// (first_kernel), or the rows of the racing-pair bitmap under an assignment
// (all_kernel).
//
// One wave per row (point, view).  It reads the 64 points from its own on, a
// chunk at a time, picks those of the same array (one of the two writing) and
// decides the pairs one per lane: the first chunk's at once (a racing point
// usually meets its partner there), later ones gathered in LDS until 64 are
// together, so that the lanes of a test are busy (with four arrays and 30%
// writes a chunk holds 5 to 16).  The lowest lane that finds a conflict is the
// first partner and ends the row.  A job's rows go round its waves; a batch
// gets ROW_GROUPS workgroups in all, since dispatching one costs as much as
// a short row.
//
// Bound: instruction latency for one kernel (a pair costs two or three hundred
// instructions in one lane, its divisions by reciprocals), instruction issue and
// waves in flight for a batch.  Measured: 22 us for the stress kernel (512
// accesses of 4.2M threads; generating, sorting and scanning their 2.0G records
// took 31 ms), 12 to 15 us for plain-large (a microsecond more with integer
// divisions, 17 us with every chunk tested at once, 0.56 ms by records), 113 to
// 116 us for 128 kernels of the batched distribution (154 us with integer
// divisions in workgroups of four waves, 338 us with a wave per row and every
// chunk tested at once, 9.2 ms by records); every pair of plain-large under a quarter of its barriers 13 us (14
// us; 31 us; 1.39 ms for the scan of its sorted records, and 0.45 ms to generate
// and sort them).
#include "closed_rows.h"
#include "common.h"
#include "launch.h"

namespace rp {

constexpr int CF_WAVES = 4;
constexpr uint32_t ROW_GROUPS = 16384;   // workgroups of a batch

// Workgroups of a batch are of two waves: rows differ in length, and a waiting
// workgroup needs room for all its waves at once (128 kernels: 123 us, 146 us
// with four waves, 145 us with one and its twice as many dispatches).  The form
// of most kernels is held to 96 registers there, five waves per SIMD and four
// spills (113 us); the other form spills more (512 programs 16 us instead of
// 12), and a lone kernel's rows all run at once (12 us instead of 13 without).
constexpr int BATCH_WAVES = 2;
template <int FORM, int WAVES>
constexpr int MIN_WAVES = FORM == FORM_PLAIN && WAVES == BATCH_WAVES ? 5 : 1;

// Walks row (i, lv): found(m, j) gets the lanes m that found a conflict and
// this lane's point j, in ascending order of points over lanes and calls, and
// ends the walk by returning true.  X: the row ends at the first enabled
// barrier of the view.  q: 128 entries of this wave.
template <int FORM, bool X, class F>
__device__ __forceinline__ void walk_row(const Job& J, const DPoint& pi, uint32_t i, uint32_t lv,
                                         uint64_t x, uint16_t* q, F found) {
  const uint32_t lane = __lane_id(), P = J.P, B = J.B;
  using I = FormInt<FORM>;
  const Access a = access_of<FORM>(pi, B);
  const bool wi = pi.flags & PF_WRITE;
  uint32_t n = 0;                          // gathered points
  for (uint32_t base = i;; base += 64) {
    const uint32_t j = base + lane;
    const PointTag t = j < P ? tag_of(J.pts[j]) : PointTag{(uint32_t)RP_NOP << 16};
    bool last = base + 64 >= P;
    uint64_t m = __ballot(t.kind() == RP_ACCESS && t.array() == pi.array &&
                          (wi || (t.flags() & PF_WRITE)));
    if constexpr (X) {
      const uint64_t e = __ballot(j > i && t.kind() == RP_BARRIER &&
                                  (lv == 0 || (t.flags() & PF_GRID)) && ((x >> t.array()) & 1));
      if (e) {
        m &= (e & (0ull - e)) - 1;
        last = true;
      }
    }
    if ((m >> lane) & 1) q[n + (uint32_t)__popcll(m & lanemask_lt())] = (uint16_t)j;
    n += (uint32_t)__popcll(m);
    __builtin_amdgcn_wave_barrier();
    while (n >= 64 || (n != 0 && (last || base == i))) {
      const uint32_t c = n < 64 ? n : 64;
      uint32_t jj = 0;
      bool hit = false;
      if (lane < c) {
        jj = q[lane];
        const Access b = access_of<FORM>(J.pts[jj], B);
        if (lv != 0) hit = pair_cross_block<I, FORM == FORM_PLAIN>(a, b);
        else hit = jj == i ? self_same_block(a) : pair_same_block<I>(a, b, B);
      }
      if (found(__ballot(hit), jj)) return;
      n -= c;
      if (lane < n) q[lane] = q[64 + lane];
      __builtin_amdgcn_wave_barrier();
    }
    if (last) return;
  }
}

// X = false: the table j0, with no barrier enabled.  X = true: first partners
// under the job's assignment, into minj (and the page), of a job that has no
// records at all.
template <int FORM, bool X, int WAVES>
__global__ __launch_bounds__(WAVES * 64, (MIN_WAVES<FORM, WAVES>))
void first_kernel(const Job* __restrict__ jobs, CallBlock call) {
  __shared__ uint16_t s_q[WAVES][128];
  stamp_if(call.stamps, STAMP_BEGIN);
  const Job& J = jobs[blockIdx.y];
  const uint32_t wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = __lane_id();
  const uint32_t P = J.P, B = J.B;
  const bool all_rows = J.nlog[0] == 0 && J.nlog[1] == 0;    // (else a scan has set the others)
  const uint64_t x = X ? J.st->x : 0;
  for (uint32_t r = blockIdx.x * WAVES + wv; r < 2 * P; r += gridDim.x * WAVES) {
    const uint32_t i = r >> 1, lv = r & 1;
    const DPoint pi = J.pts[i];
    if (r == 0) stamp_gather(call.stamps, J, pi);
    if (!X && J.packed) return;                          // (the rounds kernel's own)
    uint32_t best = NONE32;
    if (row_runs(pi, B, lv))
      walk_row<FORM, X>(J, pi, i, lv, x, s_q[wv], [&](uint64_t m, uint32_t j) {
        if (m) best = __builtin_amdgcn_readlane(j, (uint32_t)__builtin_ctzll(m));
        return m != 0;
      });
    const uint32_t row = lv * P + i;
    if (lane == 0) {
      if constexpr (X) {
        J.minj[row] = best;
        if (call.page) ((uint32_t*)call.page->tail())[row] = best;
      } else if (all_rows || closed_point(pi)) {
        J.j0[row] = best;
      }
    }
  }
  if constexpr (X) finish_call(call, J.st);
}

// Every racing pair under the job's assignment: the row's 64-point words are
// put together in LDS (at most 64 of them, one per lane at the end) and stored
// at once, and the row's pairs counted into minj for the list.
template <int FORM>
__global__ __launch_bounds__(CF_WAVES * 64) void all_kernel(const Job* __restrict__ jobs,
                                                            CallBlock call) {
  static_assert(MAX_POINTS <= 64 * 64, "a row's words in one wave");
  __shared__ uint16_t s_q[CF_WAVES][128];
  __shared__ unsigned long long s_row[CF_WAVES][64];
  stamp_if(call.stamps, STAMP_BEGIN);
  const Job& J = jobs[blockIdx.y];
  const uint32_t wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = __lane_id();
  const uint32_t P = J.P, B = J.B;
  const bool all_rows = J.nlog[0] == 0 && J.nlog[1] == 0;    // (else a scan has set the others)
  const uint64_t x = J.st->x;
  for (uint32_t r = blockIdx.x * CF_WAVES + wv; r < 2 * P; r += gridDim.x * CF_WAVES) {
    const uint32_t i = r >> 1, lv = r & 1;
    const DPoint pi = J.pts[i];
    if (r == 0) stamp_gather(call.stamps, J, pi);
    if (!all_rows && !closed_point(pi)) continue;
    s_row[wv][lane] = 0;
    __builtin_amdgcn_wave_barrier();
    if (row_runs(pi, B, lv))
      walk_row<FORM, true>(J, pi, i, lv, x, s_q[wv], [&](uint64_t m, uint32_t j) {
        if ((m >> lane) & 1) atomicOr(&s_row[wv][j >> 6], 1ull << (j & 63));
        return false;
      });
    __builtin_amdgcn_wave_barrier();
    const uint64_t word = s_row[wv][lane];
    const uint32_t row = lv * P + i;
    if (lane < J.wpr) J.bitmap[(uint64_t)row * J.wpr + lane] = word;
    uint32_t c = (uint32_t)__popcll(word);
    for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o);
    if (lane == 0) J.minj[row] = c;
  }
}

static dim3 row_grid(uint32_t max_points, uint32_t njobs, uint32_t waves) {
  const uint32_t all = (2 * max_points + waves - 1) / waves;
  const uint32_t most = ROW_GROUPS / njobs;
  return dim3(all < most ? all : (most ? most : 1), njobs);
}

hipError_t launch_all_closed(const Job* job, uint32_t points, int form, const CallBlock& call,
                             hipStream_t s) {
  if (points == 0) return hipSuccess;
  const dim3 grid = row_grid(points, 1, CF_WAVES);
  switch (form) {
    case FORM_PLAIN: all_kernel<FORM_PLAIN><<<grid, CF_WAVES * 64, 0, s>>>(job, call); break;
    case FORM_SMALL: all_kernel<FORM_SMALL><<<grid, CF_WAVES * 64, 0, s>>>(job, call); break;
    default: all_kernel<FORM_WIDE><<<grid, CF_WAVES * 64, 0, s>>>(job, call); break;
  }
  return hipGetLastError();
}

template <bool X, int WAVES>
static hipError_t first_go(const Job* jobs, uint32_t njobs, uint32_t max_points, int form,
                           const CallBlock& call, hipStream_t s) {
  for (uint32_t j = 0; j < njobs; j += 65535) {      // (the grid's second dimension)
    const dim3 grid = row_grid(max_points, njobs - j < 65535 ? njobs - j : 65535, WAVES);
    const CallBlock c = j == 0 ? call : CallBlock{};
    switch (form) {
      case FORM_PLAIN: first_kernel<FORM_PLAIN, X, WAVES><<<grid, WAVES * 64, 0, s>>>(jobs + j, c); break;
      case FORM_SMALL: first_kernel<FORM_SMALL, X, WAVES><<<grid, WAVES * 64, 0, s>>>(jobs + j, c); break;
      default: first_kernel<FORM_WIDE, X, WAVES><<<grid, WAVES * 64, 0, s>>>(jobs + j, c); break;
    }
  }
  return hipGetLastError();
}

hipError_t launch_first_closed(const Job* jobs, uint32_t njobs, uint32_t max_points, int form,
                               const CallBlock& call, hipStream_t s) {
  if (njobs == 0 || max_points == 0) return hipSuccess;
  return njobs > 1 ? first_go<false, BATCH_WAVES>(jobs, njobs, max_points, form, call, s)
                   : first_go<false, CF_WAVES>(jobs, njobs, max_points, form, call, s);
}

hipError_t launch_first_under(const Job* job, uint32_t points, int form, const CallBlock& call,
                              hipStream_t s) {
  return first_go<true, CF_WAVES>(job, 1, points ? points : 1, form, call, s);
}

}  // namespace rp
