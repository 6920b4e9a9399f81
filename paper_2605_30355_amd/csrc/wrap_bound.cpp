// wrap_bound.cpp -- how far FP32 phases may drift between two wraps, and which
// sweep forms may leave the wrap to the twists or to the ends of the sweeps.
#include <algorithm>
#include <cstdlib>
#include <vector>

#include "internal.hpp"

namespace cosm {

namespace {
// The largest step and twist in turns (grid: exact products of small integers
// and powers of two).
double alpha_max_turns(const Schedule &sc) {
  return sc.grid ? (double)sc.a0_units * (double)sc.aunit : (double)sc.alpha0_turns;
}
double twist_max_turns(const Schedule &sc) {
  return sc.grid ? (double)sc.twist_num2 * (double)sc.a0_units * (double)sc.tunit
                 : (double)sc.dwt_ratio * alpha_max_turns(sc);
}
}  // namespace

double wrap_drift_turns(const cosm_state &s) {
  // the largest drift of one phase from its wrapped range between two twists:
  // the twist left unwrapped plus every step of `period` sweeps, J and h alike
  return twist_max_turns(s.sched) +
         (double)s.sched.dwt_period * alpha_max_turns(s.sched) * (double)s.wdeg_max;
}

bool exact_grid_fp32(const cosm_state &s) {
  return s.p.storage == COSM_STORE_FP32 && s.sched.grid && s.p.update == COSM_UPDATE_SCS;
}

// Between two twists a phase starts in [0, 1 + twist) and moves by at most
// period x alpha0 x (largest sum of |J| and |h| at one vertex); with that drift
// below one turn it stays in (-1, 2), where every multiple of 2^-23 turn is an
// FP32 number, so the phases and the updates stay exact without a wrap.  The
// difference x_u - x_v may then reach 3 turns in magnitude and round, but
// toward minus infinity, and halves of turns are FP32 numbers, so
// floor(2(x_u - x_v)) and with it the step's sign are still exact.  The twist
// wraps before it tests its windows.  (The forms without the parity step need
// the difference itself exact: half a turn, lds_lazy_wrap; and so do those with it
// that take the difference from the edge's v end: either_end_at_twists.)  Two of
// seven VALU per update fewer; whole trials, wrapping after every update -> at the
// twists: 20x20 torus, 64 replicas x 2000 sweeps 1057 -> 956 us (latency); 3-regular,
// N = 2000, 1024 x 10^4 10.79 -> 10.52 ms and 5-regular, N = 20000, 2048 x 1000
// 42.0 -> 41.0 ms (LDS).
bool wrap_at_twists(const cosm_state &s) {
  return exact_grid_fp32(s) && s.on_grid && s.sched.dwt_period > 0 && wrap_drift_turns(s) < 1.0;
}

// The same with a wrap at the end of every sweep.
bool grid_drift_below_turn(const cosm_state &s) {
  return s.p.storage == COSM_STORE_FP32 && s.sched.grid && s.on_grid &&
         twist_max_turns(s.sched) + alpha_max_turns(s.sched) * (double)s.wdeg_max < 1.0;
}
bool wrap_at_sweeps(const cosm_state &s) { return exact_grid_fp32(s) && grid_drift_below_turn(s); }

// x_u - x_v as the v end computes it, -(x_v - x_u) with x_v - x_u rounded toward
// minus infinity, is x_u - x_v rounded up: just below a half turn it would take the
// other sign.  So the forms that decide an edge's sign at either end (sweep_dual.hip,
// the owners of sweep_rstream.hip) need the difference exact, that is below two
// turns: two phases start in [0, 1 + twist) and part by the steps that both ends can
// have made before that edge's own update.  They are counted edge by edge, in units of
// the largest step (the two-class form's in the even classes only: it takes no other
// edge's difference from the v end).  Once per state: its schedule and couplings do not
// change.
// 20 x 20 torus at 14 degrees, period 3: 0.80 of the one turn there is; 141 x 141
// torus 0.88.
void find_wrap_bounds(cosm_state *s) {
  s->dual_twists = s->dual_sweeps = s->owner_twists = false;
  if (!wrap_at_sweeps(*s)) return;
  // edges class by class
  std::vector<int32_t> at(s->class_begin), order((size_t)s->m);
  for (int64_t k = 0; k < s->m; k++)
    order[(size_t)at[(size_t)s->h_colour[(size_t)k]]++] = (int32_t)k;
  // a vertex's steps in a whole sweep, and in the classes so far
  std::vector<int64_t> all((size_t)s->n, 0), done((size_t)s->n, 0);
  for (int64_t k = 0; k < s->m; k++) {
    const int64_t w = std::llabs((int64_t)s->h_J[(size_t)k]);
    all[(size_t)s->h_eu[(size_t)k]] += w;
    all[(size_t)s->h_ev[(size_t)k]] += w;
  }
  const double before = (double)(std::max(1, s->sched.dwt_period) - 1);
  double dual = 0.0, owner = 0.0, sweep = 0.0;
  for (int32_t k : order) {
    const size_t u = (size_t)s->h_eu[(size_t)k], v = (size_t)s->h_ev[(size_t)k];
    const int64_t w = std::llabs((int64_t)s->h_J[(size_t)k]);
    if (w == 0) continue;
    const double here = (double)(done[u] + done[v]), period = before * (double)(all[u] + all[v]);
    owner = std::max(owner, period + here);
    if (s->h_colour[(size_t)k] % 2 == 0) {
      dual = std::max(dual, period + here);
      sweep = std::max(sweep, here);
    }
    done[u] += w;
    done[v] += w;
  }
  auto exact = [&](double steps) {
    return twist_max_turns(s->sched) + alpha_max_turns(s->sched) * steps <= 1.0;
  };
  s->dual_sweeps = exact(sweep);
  s->dual_twists = exact(dual);
  s->owner_twists = exact(owner);
}
bool either_end_at_twists(const cosm_state &s, bool dual) {
  return wrap_at_twists(s) && (dual ? s.dual_twists : s.owner_twists);
}
bool dual_wrap_at_sweeps(const cosm_state &s) { return wrap_at_sweeps(s) && s.dual_sweeps; }

}  // namespace cosm
