// What the host plan decides about kernels, for tests.
#include "../paper_2011_08373_amd/csrc/plan.h"

using namespace rp;

// per kernel: 1 when the rounds kernel works out its first partners itself
extern "C" int plan_packed(const rp_kernel* k) {
  Plan pl;
  if (validate_kernel(k) != RP_OK) return -1;
  make_plan(k, pl);
  return pl.packed;
}

// access records the kernel's log gets (0: every conflict in closed form)
extern "C" long long plan_records(const rp_kernel* k) {
  Plan pl;
  if (validate_kernel(k) != RP_OK) return -1;
  make_plan(k, pl);
  return (long long)(pl.log_intra + pl.log_inter);
}

// the same over the kernels of one call; over: what their arrays' bounds cost
// beyond their own records, together
extern "C" long long call_records(const rp_kernel* const* ks, int n, double* over) {
  std::vector<Plan> plans(n);
  std::vector<Plan*> call;
  *over = 0;
  for (int j = 0; j < n; j++) {
    if (validate_kernel(ks[j]) != RP_OK) return -1;
    make_plan(ks[j], plans[j]);
    for (const PlanArray& a : plans[j].arrays) *over += a.bounded ? a.over : 0;
    call.push_back(&plans[j]);
  }
  choose_routes(call.data(), call.size());
  long long sum = 0;
  for (const Plan& pl : plans) sum += (long long)(pl.log_intra + pl.log_inter);
  return sum;
}
