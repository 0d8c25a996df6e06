// The stop flag of a run whose launches record the launch before them.
//
// A recording block sets the flag while the tile blocks of its own launch look
// at it, and the waves of a tile block meet at barriers: they have to decide
// alike.  So the flag (0 while the run goes on) has a bit for launches of each
// parity, and a recording block sets only the other parity's, which no block of
// its launch looks at; the next launch sets both.  (The passes of several steps
// read the flag, whichever bit, by one thread for the whole block; that costs the
// one-step kernels a barrier per launch.  Two words instead of two bits made the
// run state larger: the read-back of 48 chambers' states then exceeded 16 KB,
// from which it takes another way, and pulse trains took 1.3 % longer.)
#pragma once

#ifdef __HIPCC__
#define IT_HD __host__ __device__
#else
#define IT_HD
#endif

namespace it {

// Whether the tile blocks of a launch of this parity compute nothing.
IT_HD inline bool launch_skips(int flag, int parity) { return (flag >> parity) & 1; }

// The flag that the recording block of a launch of this parity leaves when it
// finds the run stopped, and the one that a launch leaves which finds that an
// earlier one did (or that has no tile blocks).
IT_HD inline int stop_after(int parity) { return 1 << (parity ^ 1); }
constexpr int kStopAll = 3;

}  // namespace it
