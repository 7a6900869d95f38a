// Global steps to queue (StepEstimate, paper_1408_3719_amd/csrc/host.h) in
// named situations, on the host: one line "<name> <steps>" each.
#include <cstdio>

#include "host.h"

using namespace aw;

static constexpr double N = double(MACRO_TICKS);

static Inst at(double T, double dt, bool open) {
  Inst in{};
  in.T = T;
  in.delta = dt / N;
  in.open = open;
  return in;
}

int main() {
  StepEstimate e;
  e.reset(2);
  Inst in[2] = {at(0.0, 0.0, true), at(0.0, 0.0, true)};
  std::printf("no_step_yet %d\n", e.steps(in, 1.0, 8));
  in[0] = at(0.25, 0.25, true);
  in[1] = at(0.125, 0.125, true);
  e.note(in);
  std::printf("furthest_behind %d\n", e.steps(in, 1.0, 8));
  std::printf("limited %d\n", e.steps(in, 100.0, 8));
  std::printf("inside_one_step %d\n", e.steps(in, 0.26, 8));
  // the first instance has reached its target, steps of it take no time
  in[0] = at(1.0, 0.0, false);
  in[1] = at(0.5, 0.125, true);
  e.note(in);
  e.note(in);
  std::printf("first_instance_done %d\n", e.steps(in, 1.0, 8));
  // a last step cut short by the target does not count, the one before does
  in[1] = at(1.0, 1e-6, false);
  e.note(in);
  std::printf("next_target %d\n", e.steps(in, 2.0, 8));
  std::printf("first_instance_again %d\n", e.steps(in, 1.5, 8));
  e.reset(2);
  std::printf("bound_anew %d\n", e.steps(in, 2.0, 8));
  in[0] = at(2.0, 0.0, false);
  in[1] = at(2.0, 0.0, false);
  std::printf("nothing_to_do %d\n", e.steps(in, 2.0, 8));
}
