// Plain one-step stencil kernel (gfx950).
//
// Step kernel: one explicit time step of both ion species (eq. theEquation
// with the Appendix's difference scheme, written as per-node coefficients),
// plus the per-step tallies.  Each block (8 or 16 waves) owns a 64 x 8,
// 64 x 16 or 32 x 16 column tile (plain_tile_step), or a 128 x 8 or
// 128 x 16 tile of column pairs (pair_tile_step), and a chunk of planes and
// marches up it; with one step per launch an extra block records the
// previous step from its partials.  Every thread
// keeps n_{k-1}, n_k, n_{k+1} of its column in registers, the block stages
// plane k of the tile in LDS for the lateral neighbours, and neighbours
// outside the tile (its one-node rim, or a periodic wrap) are read from
// global memory, where they are L2 hits of the neighbouring tiles.  Results
// go out with non-temporal stores: the new densities are not read again in
// this launch, and keeping them out of L2 leaves it to the reused inputs.
// No MFMA: the update is a 7-point stencil, not a contraction, and the
// kernel is bound by HBM bandwidth (32 bytes per node and step).
#include <algorithm>

#include "stencil_plain.h"

namespace it {

// With p.prev_partials set, the launch has one block more than tiles: that
// block sums the previous step's partials in a fixed order and records the
// step (finalize_steps), while the others compute this step.  The kernel
// boundary before this launch makes the previous partials visible; the
// state it writes is read by the next launch.  Once it finds the run stopped,
// this launch has computed a step past the stop, whose output goes to the field
// pair not holding the stop step; the launches after it skip (see stop_flag.h).
// Tiles of column pairs aim at 8 waves per CU, so they may use more
// registers (at least 2 waves per SIMD instead of 4).
template <int SY, bool SC, bool AB, int TX>
__global__ __launch_bounds__(kTX * SY) __attribute__((amdgpu_waves_per_eu(TX == 2 * kTX ? 2 : 4, 8))) void step_plain_kernel(StepParams p) {
  if (p.prev_partials && blockIdx.x == gridDim.x - 1) {
    __shared__ RunState now;
    __shared__ double totals[kAcc * kMaxT];
    snapshot_state(p.state, &now);
    reduce_partials<kTX * SY>(p.prev_partials, p.prev_nblocks, kAcc * p.prev_T, kAcc * p.prev_T, totals);
    if (threadIdx.x == 0 && threadIdx.y == 0) {
      if (now.done)
        p.state->done = kStopAll;
      else
        finalize_steps(p.state, &now, p.trace, totals, p.prev_T, p.prev_step, p.cp, p.cn, p.dV, p.stop_tol,
                       p.min_stop_step);
    }
    return;
  }
  // set by an earlier launch: every block skips (read here, looked at once the
  // first planes are on their way)
  const bool done = launch_skips(p.state->done, p.parity);
  const TileCoord t = decode_tile(p.tiles_x, p.tiles_y, p.ntiles, p.per_xcd);
  if constexpr (TX == 2 * kTX)
    pair_tile_step<SY, SC, AB>(p, t, done, p.partials + (size_t)blockIdx.x * kAcc);
  else
    plain_tile_step<SY, SC, AB, TX>(p, t, done, p.partials + (size_t)blockIdx.x * kAcc);
}

// One block: sums the per-block partial tallies of a stepping launch in a
// fixed order and turns them into T trace records (see finalize_steps).
// Running as its own launch, it sees every partial without device-wide
// fences in the stepping kernel.
__global__ __launch_bounds__(1024) void reduce_steps_kernel(StepParams p, int nblocks, int T) {
  __shared__ RunState now;
  __shared__ double totals[kAcc * kMaxT];
  snapshot_state(p.state, &now);
  reduce_partials<1024>(p.partials, nblocks, kAcc * T, kAcc * T, totals);
  if (threadIdx.x == 0) {
    if (now.done)
      p.state->done = kStopAll;
    else
      finalize_steps<true>(p.state, &now, p.trace, totals, T, p.step0, p.cp, p.cn, p.dV, p.stop_tol, p.min_stop_step);
  }
}

hipError_t launch_reduce_steps(const StepParams& p, int nblocks, int T, hipStream_t s) {
  hipLaunchKernelGGL(reduce_steps_kernel, dim3(1), dim3(1024), 0, s, p, nblocks, T);
  return hipGetLastError();
}

namespace {

__global__ __launch_bounds__(256) void zero_electrodes_kernel(double* a, double* b, double* c, double* d, size_t plane,
                                                              size_t top) {
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < plane; i += (size_t)gridDim.x * 256) {
    a[i] = b[i] = c[i] = d[i] = 0.0;
    a[top + i] = b[top + i] = c[top + i] = d[top + i] = 0.0;
  }
}

}  // namespace

hipError_t launch_zero_electrodes(double* const (&pair0)[2], double* const (&pair1)[2], size_t plane, int nz,
                                  hipStream_t s) {
  const unsigned grid = (unsigned)std::min<size_t>((plane + 255) / 256, 2048);
  hipLaunchKernelGGL(zero_electrodes_kernel, dim3(grid), dim3(256), 0, s, pair0[0], pair0[1], pair1[0], pair1[1], plane,
                     plane * nz);
  return hipGetLastError();
}

int plain_tile_rows(int tile_y, int tile_x) { return tile_x == 32 || tile_y == 16 ? 16 : 8; }

namespace {

template <int SY, bool SC, bool AB, int TX>
void launch_plain_instance(const StepParams& p, dim3 g, hipStream_t s) {
  hipLaunchKernelGGL((step_plain_kernel<SY, SC, AB, TX>), g, dim3(kTX, SY), 0, s, p);
}

template <int SY, int TX>
void launch_plain_terms(const StepParams& p, dim3 g, hipStream_t s) {
  const bool sc = p.gsp != 0.0 || p.gsn != 0.0;
  const bool ab = p.absorbing != 0;
  switch ((sc ? 2 : 0) + (ab ? 1 : 0)) {
    case 0: launch_plain_instance<SY, false, false, TX>(p, g, s); break;
    case 1: launch_plain_instance<SY, false, true, TX>(p, g, s); break;
    case 2: launch_plain_instance<SY, true, false, TX>(p, g, s); break;
    default: launch_plain_instance<SY, true, true, TX>(p, g, s); break;
  }
}

// the kernel instance for the tile shape, the space-charge term and the
// lateral boundary option of the run
void launch_plain_variant(const StepParams& p, int tile_y, int tile_x, dim3 g, hipStream_t s) {
  if (plain_tile_cols(tile_x) == 128) {
    if (plain_tile_rows(tile_y, tile_x) == 16) launch_plain_terms<16, 128>(p, g, s);
    else launch_plain_terms<8, 128>(p, g, s);
  } else if (plain_tile_cols(tile_x) == 32) launch_plain_terms<8, 32>(p, g, s);
  else if (plain_tile_rows(tile_y, tile_x) == 16) launch_plain_terms<16, 64>(p, g, s);
  else launch_plain_terms<8, 64>(p, g, s);
}

}  // namespace

hipError_t launch_step_plain(const StepParams& p, int tile_y, int tile_x, hipStream_t s, hipEvent_t ev_begin,
                             hipEvent_t ev_end, bool fused) {
  const int grid = 8 * p.per_xcd;
  if (ev_begin && hipEventRecord(ev_begin, s) != hipSuccess) return hipErrorInvalidValue;
  const dim3 g(grid + (p.prev_partials ? 1 : 0));
  launch_plain_variant(p, tile_y, tile_x, g, s);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (ev_end && hipEventRecord(ev_end, s) != hipSuccess) return hipErrorInvalidValue;
  if (fused) return hipSuccess;  // the next launch (or a closing reduction) records this step
  return launch_reduce_steps(p, grid, 1, s);
}

}  // namespace it
