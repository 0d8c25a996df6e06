// The stop flag of a run whose launches record the launch before them.
//
// A recording block sets the flag while the tile blocks of its own launch look
// at it, and the waves of a tile block meet at barriers: they have to decide
// alike.  So there are two flags, one for launches of each parity, and a
// recording block sets only the other parity's, which no block of its launch
// reads; the next launch's recording block passes it on.  (One flag read by one
// thread for the whole block, as the blocked passes do, costs the one-step
// kernels a barrier per launch.)
#pragma once

#include <stdint.h>

#ifndef IT_HD
#ifdef __HIPCC__
#define IT_HD __host__ __device__
#else
#define IT_HD
#endif
#endif

namespace it {

struct StopFlags {
  int32_t skip[2];  // [parity of the launch]
};

// Whether the tile blocks of a launch of this parity compute nothing.
IT_HD inline bool launch_skips(const StopFlags& f, int parity) { return f.skip[parity] != 0; }

// By the recording block of a launch of this parity, once the run has stopped.
IT_HD inline void stop_after(StopFlags& f, int parity) { f.skip[parity ^ 1] = 1; }

// By a launch without tile blocks.
IT_HD inline void stop_now(StopFlags& f) { f.skip[0] = f.skip[1] = 1; }

}  // namespace it
