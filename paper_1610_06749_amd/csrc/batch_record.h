// What the batched stepping kernels share: the instance of a tile, and the
// recording of the previous pass.
#pragma once

#include "reduce.h"

namespace it {

__device__ inline int find_instance(const BatchInstance* inst, int ninst, int L) {
  int lo = 0, hi = ninst - 1;
  while (lo < hi) {  // last instance with tile_begin <= L
    const int mid = (lo + hi + 1) >> 1;
    if (inst[mid].tile_begin <= L) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// Records the previous pass's T steps of instance q (its partials are in
// the buffer of the other parity), up to the instance's step limit: a pass
// may run past it, and those steps are not recorded.
//
// Pulse trains (a period of at least T steps, so at most one pulse in a
// pass): a pass computes steps c0 .. c0 + T - 1, and the pass in which a
// pulse falls due adds it to the outputs of the level that computes the
// step before it (pulse_add = j for a pulse at step c0 + j, j = 1..T; one
// at c0 + T is thus added by the pass before the one it precedes).  The
// recording block of a pass, which records the previous pass's steps
// r0 .. r0 + T - 1, books the release of a pulse deposited before one of
// them with that step (the first pulse's release, from the deposit, is
// kept when step 0 is recorded), then sets the flag of the next pass, which
// computes steps r0 + 2T .. r0 + 3T - 1.  The flags alternate by pass
// parity, so the tile blocks of a pass read a flag the previous pass wrote.
__device__ inline void record_previous(const BatchInstance& bi, int parity, int T) {
  const StepParams& p = bi.sp[parity ^ 1];
  __shared__ RunState now;
  snapshot_state(p.state, &now);
  __syncthreads();
  if (now.done) {
    if (threadIdx.x == 0 && threadIdx.y == 0) p.state->done = kStopAll;
    return;
  }
  // the previous pass's tile count, which its own recording block stored
  // (the host may have re-tiled the running instances since)
  __shared__ double totals[kAcc * kMaxT];
  reduce_partials(p.partials, now.rec_ntiles, kAcc * T, kAcc * T, totals);
  if (threadIdx.x == 0 && threadIdx.y == 0) {
    RunState* st = p.state;
    const int64_t step = now.steps;
    const int Te = (int)min((int64_t)T, bi.max_steps - step);
    const bool train = bi.npulses >= 2;
    int inject = -1;
    if (train) {
      if (step == 0) {
        now.pulse_q[0] = st->pulse_q[0] = now.released;
        now.pulse_q[1] = st->pulse_q[1] = now.released_neg;
      }
      const int k = now.pulses_counted;
      const int64_t s_k = (int64_t)k * bi.period_steps;
      if (k < bi.npulses && s_k >= step && s_k < step + Te) {
        inject = (int)(s_k - step);
        st->pulses_counted = k + 1;
      }
    }
    const int stopped = finalize_steps(st, &now, p.trace, totals, Te, step, p.cp, p.cn, p.dV, p.stop_tol,
                                       p.min_stop_step, inject, train ? now.pulse_q[0] : 0.0,
                                       train ? now.pulse_q[1] : 0.0);
    if (!stopped && step + Te >= bi.max_steps) {
      st->done = stop_after(parity);
      st->by_limit = 1;
    }
    st->rec_ntiles = bi.ntiles;  // this pass's tiles, for the next recording block
    if (train) {
      // the next pass computes steps c1 .. c1 + T - 1; a pulse at or past
      // the run's last step is never deposited
      const int64_t c1 = step + 2 * T;
      const int kf = now.pulses_flagged;
      const int64_t s_due = (int64_t)kf * bi.period_steps;
      const bool due = kf < bi.npulses && s_due > c1 && s_due <= c1 + T && s_due < bi.max_steps;
      st->pulse_add[parity ^ 1] = due ? (int)(s_due - c1) : 0;
      if (due) st->pulses_flagged = kf + 1;
    }
  }
}

}  // namespace it
