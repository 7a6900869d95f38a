// Host-side pieces of the aderweno library: tables and topology.
#pragma once
#include <algorithm>
#include <cmath>
#include <string>
#include <vector>

#include "common.h"

namespace aw {

void gauss_legendre01(int n, double* x, double* w);
void build_tables(int M, Tables& T);

// Mesh topology built once on the host (paper Sec. 2.2: fixed stencils).
struct Topology {
  int NE = 0, NV = 0, NF = 0, ne = 0;
  std::vector<double> xy;                 // [NV][2] initial node positions
  std::vector<int> tri;                   // [NE][3]
  // edges in order of first appearance (elements by index, local edges 0,1,2)
  std::vector<int> e_a, e_b, e_L, e_R, e_el, e_er, e_bc;
  std::vector<int> elem_edges;            // [NE][3]
  std::vector<int> neigh;                 // [NE][3], -1 on the boundary
  std::vector<int> ring_ptr, ring_ent;    // node -> (element*4 + local vertex), by element
  std::vector<int> sten;                  // [NE][7][ne], -1 rows: dropped
  std::vector<int> sched_ptr, sched_idx;  // symmetric scheduling stencils (sorted)
  // for each element j, the stencil rows (c >= 1) that name it, as slots
  // ((i * ne + c) * 8 + s) of row c of stencil s of element i, ascending
  std::vector<int> tsten_ptr, tsten_idx;
  std::vector<double> wall_n;             // [NV][2] slip-wall unit normal or 0
  std::vector<int> wall_pin;              // [NV]
};

// Throws std::runtime_error with a message on an invalid mesh.
void build_topology(int M, int n_nodes, const double* xy, int n_elems, const int* tri,
                    int n_bedges, const int* bedge, Topology& t);

// Mean number of different elements that the stencils and face neighbours of
// `group` consecutive elements name, over at most 64 such groups spread over the mesh.
double named_elements(const Topology& t, int group);

// Is an instance at time T short of the target time (the test that the device
// applies too)?
inline bool short_of_target(double T, double t_target) {
  return !(t_target - T <= 1e-12 * std::fmax(1.0, std::fabs(t_target)));
}

// Global steps to queue before the next status read, estimated from the steps
// taken so far. Results do not depend on it: a step too many does nothing, one
// too few costs a status read. A new state's first steps are guessed from those of
// the state before, since a caller who uploads again mostly uploads a like state
// (1,064 triangles, M=1, 20 steps per upload: 1,245 us, 1,270 with a fresh start).
struct StepEstimate {
  // per instance the tick length of its last step that did not end at the
  // target (that one may be cut short), 0: none yet
  std::vector<double> delta;
  void reset(int K) { delta.assign(size_t(K), 0.0); }
  // the instances after the queued steps
  void note(const Inst* in) {
    for (size_t k = 0; k < delta.size(); ++k)
      if (in[k].open && in[k].delta > 0.0) delta[k] = in[k].delta;
  }
  // as many as the instance furthest behind needs, at most `limit`; one while an
  // instance short of the target has no step to go by. The others do not count.
  int steps(const Inst* in, double t_target, int limit) const {
    double need = 0.0;
    for (size_t k = 0; k < delta.size(); ++k) {
      if (!short_of_target(in[k].T, t_target)) continue;
      if (!(delta[k] > 0.0)) return 1;
      need = std::fmax(need, (t_target - in[k].T) / (double(MACRO_TICKS) * delta[k]));
    }
    return need >= double(limit) ? limit : std::max(1, int(std::ceil(need)));
  }
};

}  // namespace aw
