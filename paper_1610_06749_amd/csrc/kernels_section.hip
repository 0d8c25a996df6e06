// Batched stepping of narrow periodic chambers: T steps per launch, a block
// per chunk of planes of one chamber's whole cross-section (section_pass),
// and one recording block per instance as in kernels_batch.hip.
#include <algorithm>

#include "batch_record.h"
#include "stencil_section.h"

namespace it {

namespace {

// CROWDED: as many waves per SIMD as the registers allow with level 0's
// planes loaded one iteration ahead (three with two or three rows per
// thread), so that three or four blocks share a CU; otherwise two waves per
// SIMD and planes loaded two iterations ahead, for batches that leave a CU
// only a block or two (one ahead, an iteration is then as long as a load).
template <int R, int NTP, bool PU, bool CROWDED>
__global__ __launch_bounds__(NTP) __attribute__((amdgpu_waves_per_eu(CROWDED ? 3 : 2, CROWDED ? 3 : 2)))
void batch_section_kernel(const BatchInstance* __restrict__ inst, int ninst, int total_tiles, int per_xcd,
                          int parity) {
  const int b = blockIdx.x;
  if (b >= 8 * per_xcd) {
    record_previous(inst[b - 8 * per_xcd], parity, kSectionT);
    return;
  }
  const int L = (b & 7) * per_xcd + (b >> 3);
  if (L >= total_tiles) return;
  const int q = find_instance(inst, ninst, L);
  const StepParams& p = inst[q].sp[parity];
  // the recording block of this launch may set the flag: one read for the block
  __shared__ int stopped;
  if (threadIdx.x == 0) stopped = p.state->done;
  __syncthreads();
  if (stopped) return;
  const int l = L - inst[q].tile_begin;
  double* out = p.partials + (size_t)l * kAcc * kSectionT;
  if (PU) {
    const BatchInstance& bi = inst[q];
    // written by the previous pass's recording block; one value for the block
    const int j = bi.npulses >= 2 ? __builtin_amdgcn_readfirstlane(p.state->pulse_add[parity]) : 0;
    section_pass<kSectionT, R, NTP, true, CROWDED ? 1 : 2>(p, l, out, j, bi.pulse_pos, bi.pulse_neg);
  } else {
    section_pass<kSectionT, R, NTP, false, CROWDED ? 1 : 2>(p, l, out, 0, nullptr, nullptr);
  }
}

template <int R, int NTP, bool CROWDED>
const void* section_ptr(bool pu) {
  return pu ? reinterpret_cast<const void*>(&batch_section_kernel<R, NTP, true, CROWDED>)
            : reinterpret_cast<const void*>(&batch_section_kernel<R, NTP, false, CROWDED>);
}

template <int R, bool CROWDED>
const void* section_threads(int threads, bool pu) {
  if (threads <= 192) return section_ptr<R, 192, CROWDED>(pu);
  if (threads <= 256) return section_ptr<R, 256, CROWDED>(pu);
  if constexpr (CROWDED) {
    return nullptr;  // a larger block has the CU to itself in either form
  } else {
    if (threads <= 384) return section_ptr<R, 384, false>(pu);
    return section_ptr<R, 512, false>(pu);
  }
}

}  // namespace

// The kernel for blocks of `threads` threads with R rows each (null if not
// offered).
const void* batch_section(int R, int threads, bool crowded, bool pu) {
  if (threads < 1 || threads > kSectionMaxThreads) return nullptr;
  switch (R) {
    case 2: return crowded ? section_threads<2, true>(threads, pu) : section_threads<2, false>(threads, pu);
    case 3: return crowded ? section_threads<3, true>(threads, pu) : section_threads<3, false>(threads, pu);
    case 4: return crowded ? nullptr : section_threads<4, false>(threads, pu);
    default: return nullptr;
  }
}

}  // namespace it
