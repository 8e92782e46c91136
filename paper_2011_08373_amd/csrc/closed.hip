// First partners in closed form (closed.h): the table j0 of the points whose
// arrays the plan marks PF_CLOSED, with no access records.
//
// One wave per (point, view).  Lanes take the 64 points from the wave's own
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

template <class I>
__global__ __launch_bounds__(CF_WAVES * 64) void first_kernel(const Job* __restrict__ jobs) {
  const Job& J = jobs[blockIdx.y];
  const uint32_t wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = __lane_id();
  const uint32_t P = J.P, B = J.B, lv = wv & 1;
  const uint32_t i = blockIdx.x * (CF_WAVES / 2) + (wv >> 1);
  if (i >= P) return;
  const DPoint pi = J.pts[i];
  uint32_t* out = J.j0 + (uint64_t)lv * P + i;
  if (!closed_point(pi)) {
    // with no records at all the scan of the logs has not cleared the row
    if (lane == 0 && J.nlog[0] == 0 && J.nlog[1] == 0) *out = NONE32;
    return;
  }
  uint32_t best = NONE32;
  if ((lv == 0 || ((pi.flags & PF_GLOBAL) && B > 1)) && pi.cnt != 0 && pi.br < B) {
    const Access a = access_of(pi, B);
    const bool wi = pi.flags & PF_WRITE;
    for (uint32_t base = i; base < P; base += 64) {
      const uint32_t j = base + lane;
      bool hit = false;
      if (j < P) {
        const DPoint& pj = J.pts[j];
        if (pj.kind == RP_ACCESS && pj.array == pi.array && (wi || (pj.flags & PF_WRITE)) &&
            pj.cnt != 0 && pj.br < B) {
          const Access q = access_of(pj, B);
          if (lv != 0) hit = pair_cross_block<I>(a, q);
          else hit = j == i ? self_same_block(a) : pair_same_block<I>(a, q, B);
        }
      }
      const uint64_t m = __ballot(hit);
      if (m) {
        best = base + (uint32_t)__builtin_ctzll(m);
        break;
      }
    }
  }
  if (lane == 0) *out = best;
}

hipError_t launch_first_closed(const Job* jobs, uint32_t njobs, uint32_t max_points, bool small,
                               hipStream_t s) {
  if (njobs == 0 || max_points == 0) return hipSuccess;
  for (uint32_t j = 0; j < njobs; j += 65535) {      // (the grid's second dimension)
    const dim3 grid((max_points + CF_WAVES / 2 - 1) / (CF_WAVES / 2),
                    njobs - j < 65535 ? njobs - j : 65535);
    if (small) first_kernel<int32_t><<<grid, CF_WAVES * 64, 0, s>>>(jobs + j);
    else first_kernel<int64_t><<<grid, CF_WAVES * 64, 0, s>>>(jobs + j);
  }
  return hipGetLastError();
}

}  // namespace rp
