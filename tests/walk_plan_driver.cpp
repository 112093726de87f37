// The launch plan (csrc/plan.hpp) as a C call, built by tests/test_walk_plan.py
// for the CPU.
#include "plan.hpp"

using namespace mcmie;

extern "C" void walk_plan(const WalkRequest *q, WalkPlan *p) { *p = plan_walk(*q); }
extern "C" int walk_plan_sizes(int which) { return (int)(which ? sizeof(WalkPlan) : sizeof(WalkRequest)); }
extern "C" uint64_t words(const mc_detector_t *d, uint64_t n_inst) { return workspace_words(*d, n_inst); }
extern "C" int calm(int now, int stepped) { return calm_at_round(now, stepped != 0); }
