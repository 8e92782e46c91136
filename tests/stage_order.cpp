// The page-locked buffers of a thread (csrc/stage.h) over a stand-in for the
// runtime that only notes its calls: prints them, one letter each.
#include <cstdio>
#include <cstdlib>

#include "../paper_2011_08373_amd/csrc/stage.h"

int main() {
  rp::PinnedStage st;
  auto step = [](const char* what) { std::printf("\n%s ", what); };
  step("first");
  if (!st.readback(100) || !st.get(100)) return 1;
  step("again");
  if (!st.readback(4096) || !st.get(4096)) return 1;
  // a call that ended early, then one that needs more room for its results
  step("early");
  st.in_flight(nullptr);
  step("results");
  if (!st.readback(5000)) return 1;
  step("upload");
  if (!st.get(5000)) return 1;
  step("early");
  st.in_flight(nullptr);
  step("upload");
  if (!st.get(6000) || !st.readback(100)) return 1;
  std::printf("\n");
  return 0;
}
