// Host-only check of the bounds under which FP32 phases are wrapped at the twists or
// at the ends of the sweeps (wrap_bound.cpp).
// Input on stdin: "n m C" then m lines "u v J colour"; arguments: alpha0 (degrees),
// twist ratio, period.  Prints "twists=.. dual=.. owner=.. sweeps=.. reach_dual=..
// reach_owner=.. reach_sweep=..": which forms leave the wrap, and the largest
// |x_u - x_v| in units of 2^-23 turn that an edge can meet before its update there
// (every step of both ends apart), over the edges whose difference may be taken from
// the v end.
#include <cstdio>
#include <cstdlib>

#include "internal.hpp"
int cosm::set_error(int st, const std::string &m) { fprintf(stderr, "err %s\n", m.c_str()); return st; }
void cosm::clear_error() {}

int main(int argc, char **argv) {
  if (argc < 4) return 1;
  const double alpha0 = atof(argv[1]), ratio = atof(argv[2]);
  const int period = atoi(argv[3]);
  int n; long m; int C;
  if (scanf("%d %ld %d", &n, &m, &C) != 3) return 1;
  cosm_state s; s.n = n; s.m = m; s.C = C;
  std::vector<long> wdeg(n, 0);
  for (long k = 0; k < m; k++) {
    int u, v, J, c;
    if (scanf("%d %d %d %d", &u, &v, &J, &c) != 4) return 1;
    s.h_eu.push_back(u); s.h_ev.push_back(v); s.h_J.push_back(J); s.h_colour.push_back(c);
    wdeg[u] += labs(J); wdeg[v] += labs(J);
  }
  for (long w : wdeg) s.wdeg_max = std::max<int64_t>(s.wdeg_max, w);
  s.p.storage = COSM_STORE_FP32;
  s.sched.grid = 1;
  s.sched.a0_units = (int64_t)(alpha0 / 360.0 * 4194304.0 + 0.5);
  s.sched.aunit = 1.0f / 4194304.0f;
  s.sched.tunit = 1.0f / 8388608.0f;
  s.sched.twist_num2 = (int)(2.0 * ratio + 0.5);
  s.sched.dwt_period = period;
  std::vector<int32_t> sizes(C, 0);
  for (int c : s.h_colour) sizes[c]++;
  s.class_begin.assign(C, 0);
  for (int c = 1; c < C; c++) s.class_begin[c] = s.class_begin[c - 1] + sizes[c - 1];
  cosm::find_wrap_bounds(&s);
  // edge by edge, by walking over the sweeps between two twists
  const long step = 2 * s.sched.a0_units, start = (1L << 23) - 1 + s.sched.twist_num2 * s.sched.a0_units;
  long reach[3] = {0, 0, 0};
  std::vector<long> moved(n, 0);
  for (int t = 0; t < std::max(1, period); t++)
    for (int c = 0; c < C; c++) {
      for (int pass = 0; pass < 2; pass++)
        for (long k = 0; k < m; k++) {
          if (s.h_colour[k] != c || s.h_J[k] == 0) continue;
          const int u = s.h_eu[k], v = s.h_ev[k];
          if (pass == 0) {
            const long d = start + moved[u] + moved[v];
            if (c % 2 == 0) reach[0] = std::max(reach[0], d);
            reach[1] = std::max(reach[1], d);
            if (t == 0 && c % 2 == 0) reach[2] = std::max(reach[2], d);
          } else {
            moved[u] += step * labs(s.h_J[k]);
            moved[v] += step * labs(s.h_J[k]);
          }
        }
    }
  printf("twists=%d dual=%d owner=%d sweeps=%d reach_dual=%ld reach_owner=%ld reach_sweep=%ld\n",
         cosm::wrap_at_twists(s), cosm::either_end_at_twists(s, true),
         cosm::either_end_at_twists(s, false), cosm::dual_wrap_at_sweeps(s), reach[0], reach[1],
         reach[2]);
  return 0;
}
