// The closed form over the device's point table: what the row kernels and the
// rounds kernel share.
#pragma once
#include <stddef.h>

#include <type_traits>

#include "closed.h"
#include "common.h"
#include "launch.h"

namespace rp {

__device__ __forceinline__ bool closed_point(const DPoint& d) {
  return d.kind == RP_ACCESS && (d.flags & PF_CLOSED);
}

// The kernels' forms.  FORM_WIDE: any closed array; FORM_SMALL: 32-bit
// arithmetic; FORM_PLAIN: that, no block conditions, and the block strides of
// an array share a divisor that keeps their terms below the pairs of blocks
// (all but odd kernels): without the other cases' code the kernel keeps 105
// registers instead of 126.  (With integer divisions, 121 instead of 142 and so
// four waves per SIMD instead of three: 128 batched kernels 167 us from 231 us.)
template <int FORM>
using FormInt = std::conditional_t<FORM == FORM_WIDE, int64_t, int32_t>;

// (the plan stores the steps and the first word of a closed point reduced)
template <int FORM>
__device__ __forceinline__ Access access_of(const DPoint& d, uint32_t B) {
  Access s;
  s.A = d.a;
  s.b = d.b;
  s.W = d.words;
  s.X = d.cnt;
  s.m = d.m;
  s.r = d.r;
  s.base = (uint32_t)d.c;
  s.bm = 1;
  s.br = 0;
  s.S = d.b;
  s.Z = B;
  if (FORM != FORM_PLAIN && d.bm != 1) {
    s.bm = d.bm;
    s.br = d.br;
    s.S = step_mod((int64_t)d.b * (int64_t)d.bm, d.words);
    s.Z = (B - 1 - d.br) / d.bm + 1;
  }
  return s;
}

// The point's array, kind and flags in one word.
struct PointTag {
  uint32_t v;
  __device__ uint32_t array() const { return v & 0xFFFFu; }
  __device__ uint32_t kind() const { return (v >> 16) & 0xFFu; }
  __device__ uint32_t flags() const { return v >> 24; }
};
__device__ __forceinline__ PointTag tag_of(const DPoint& d) {
  static_assert(offsetof(DPoint, array) == 28 && offsetof(DPoint, kind) == 30 &&
                offsetof(DPoint, flags) == 31, "one word");
  return PointTag{*reinterpret_cast<const uint32_t*>(&d.array)};
}

// Row r of a job: its point and view.  (Points that execute nowhere are no
// accesses in a closed array's table.)
__device__ __forceinline__ bool row_runs(const DPoint& pi, uint32_t B, uint32_t lv) {
  return closed_point(pi) && (lv == 0 || ((pi.flags & PF_GLOBAL) && B > 1));
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

// First partners, with no barrier enabled, of a whole job of few points and few
// pair tests (Job::packed), by one workgroup of WAVES waves.  Such
// a job has many short rows, a handful of candidates each, so the pairs of
// several rows are gathered until 64 are together and tested one per lane;
// each row's least partner is kept in LDS.  A wave per row, most of its lanes
// idle, took 71 us for 512 programs of 41 points on average, before their
// rounds.
template <int WAVES>
struct PackedLds {
  uint32_t q[WAVES][128];                  // gathered pairs: view << 16 | i << 8 | j
  uint32_t best[2 * PACKED_POINTS];        // per row (view, point)
};
template <int FORM, int WAVES>
__device__ __forceinline__ void packed_first(const Job& J, PackedLds<WAVES>& L, uint64_t* stamps) {
  using I = FormInt<FORM>;
  const uint32_t tid = threadIdx.x, lane = __lane_id();
  const uint32_t wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t P = J.P, B = J.B;
  for (uint32_t r = tid; r < 2 * P; r += WAVES * 64) L.best[r] = NONE32;
  // this lane's points lane and lane + 64
  PointTag t[2];
#pragma unroll
  for (int h = 0; h < 2; h++)
    t[h] = lane + 64 * h < P ? tag_of(J.pts[lane + 64 * h]) : PointTag{(uint32_t)RP_NOP << 16};
  asm volatile("" ::"v"(t[0].v), "v"(t[1].v));       // (waits for the values)
  if (wv == 0) stamp_if(stamps, STAMP_GEN);
  __syncthreads();
  uint32_t* q = L.q[wv];
  uint32_t n = 0;
  bool first = true;
  auto test = [&](uint32_t c) {
    if (lane >= c) return;
    const uint32_t e = q[lane], lv = e >> 16, i = (e >> 8) & 0xFFu, j = e & 0xFFu;
    const Access a = access_of<FORM>(J.pts[i], B), b = access_of<FORM>(J.pts[j], B);
    bool hit;
    if (lv != 0) hit = pair_cross_block<I, FORM == FORM_PLAIN>(a, b);
    else hit = i == j ? self_same_block(a) : pair_same_block<I>(a, b, B);
    if (hit) atomicMin(&L.best[lv * P + i], j);
  };
  for (uint32_t i = wv; i < P; i += WAVES) {
    const uint32_t ti = i < 64 ? __builtin_amdgcn_readlane((int)t[0].v, i)
                               : __builtin_amdgcn_readlane((int)t[1].v, i - 64);
    const PointTag p{ti};
    // (an array outside the closed form has no records when none of its points
    // executes anywhere)
    if (p.kind() != RP_ACCESS || !(p.flags() & PF_CLOSED)) continue;
    const uint32_t views = (p.flags() & PF_GLOBAL) && B > 1 ? 2 : 1;
#pragma unroll
    for (int h = 0; h < 2; h++) {
      const uint32_t j = lane + 64 * h;
      const uint64_t m = __ballot(j >= i && t[h].kind() == RP_ACCESS && t[h].array() == p.array() &&
                                  ((p.flags() | t[h].flags()) & PF_WRITE));
      for (uint32_t lv = 0; m != 0 && lv < views; lv++) {
        if ((m >> lane) & 1) q[n + (uint32_t)__popcll(m & lanemask_lt())] = lv << 16 | i << 8 | j;
        n += (uint32_t)__popcll(m);
        __builtin_amdgcn_wave_barrier();
        if (n < 64) continue;
        if (wv == 0 && first) stamp_if(stamps, STAMP_SORT);
        first = false;
        test(64);
        n -= 64;
        const uint32_t rest = lane < n ? q[64 + lane] : 0;
        if (lane < n) q[lane] = rest;
        __builtin_amdgcn_wave_barrier();
      }
    }
  }
  if (wv == 0 && first) stamp_if(stamps, STAMP_SORT);
  test(n);
  __syncthreads();
  for (uint32_t r = tid; r < 2 * P; r += WAVES * 64) J.j0[r] = L.best[r];
  __syncthreads();
}

}  // namespace rp
