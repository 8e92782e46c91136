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
