// Deterministic block reductions and the end-of-launch tally finalisation
// shared by the stepping kernels.  Every sum is taken in a fixed order
// (wave butterfly, then waves in index order, then blocks in index order),
// so a run is bitwise reproducible.
#pragma once

#include "internal.h"

namespace it {

constexpr int kWave = 64;

// Workgroup barrier that orders LDS only.  __syncthreads() also waits for
// every outstanding global load and store of the wave, which would drain
// the prefetches the stepping loops keep in flight across their barriers.
__device__ inline void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The value that DPP control CTRL moves to this lane; 0 where it moves none
// (no source lane, or a row outside ROWS).
template <int CTRL, int ROWS>
__device__ inline double dpp_or_zero(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWS, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWS, 0xf, true);
  return __hiloint2double(hi, lo);
}

// Sum over the wave, the same value in every lane: sums within each row of
// 16 lanes (shifts by 1, 2, 4, 8), then across rows (broadcasts of lanes 15
// and 31 of each half to the rows after them).  All in the vector ALU: a
// butterfly through LDS permutes costs 12 of them, 6 clocks of the CU's one
// LDS pipe each, and the closing sums of a block's tallies then took 10 us
// of a blocked pass (8 waves x 39 sums) and 2.5 us of a one-step pass.
__device__ inline double wave_sum(double v) {
  v += dpp_or_zero<0x111, 0xf>(v);  // row_shr:1
  v += dpp_or_zero<0x112, 0xf>(v);
  v += dpp_or_zero<0x114, 0xf>(v);
  v += dpp_or_zero<0x118, 0xf>(v);
  v += dpp_or_zero<0x142, 0xa>(v);  // row_bcast:15
  v += dpp_or_zero<0x143, 0xc>(v);  // row_bcast:31
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), kWave - 1);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), kWave - 1);
  return __hiloint2double(hi, lo);
}

__device__ inline double wave_max(double v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v = fmax(v, __shfl_xor(v, off, kWave));
  return v;
}

// Sums N values per thread over a block of NT threads; thread 0 writes the N
// block totals to out[0..N).  lds must hold (NT/64) * N doubles.  Slots set
// in ZERO (bit q for slot q) are known to be zero in every thread, slots set
// in LANE0 hold their wave's whole sum in lane 0: both without the wave
// reduction.
template <int N, int NT, uint64_t ZERO = 0u, uint64_t LANE0 = 0u>
__device__ inline void block_sum_store(double (&acc)[N], double* out, double* lds) {
  constexpr int W = NT / kWave;
  const int tid = threadIdx.x + threadIdx.y * blockDim.x;
  const int wave = tid / kWave, lane = tid % kWave;
#pragma unroll
  for (int q = 0; q < N; ++q) {
    const double v = (ZERO >> q) & 1u ? 0.0 : (LANE0 >> q) & 1u ? acc[q] : wave_sum(acc[q]);
    if (lane == 0) lds[wave * N + q] = v;
  }
  lds_barrier();  // not __syncthreads(), which would wait for the stores of the block's fields
  if (tid < N) {
    double s = lds[tid];
#pragma unroll
    for (int w = 1; w < W; ++w) s += lds[w * N + tid];
    out[tid] = s;
  }
}

// Called by all threads of every block after the block wrote its partials.
// Returns true in exactly one block: the last to arrive.  That block then
// sees every other block's partials.  (Used only by the rare deposit launch:
// the device-scope fence of every block costs an L2 write-back, so the
// stepping kernels leave their partials to the next launch, whose kernel
// boundary makes them visible.)
// nblocks: blocks that take part.
template <int NT>
__device__ inline bool arrive_last(unsigned* counter, unsigned nblocks) {
  __shared__ int last;
  __syncthreads();
  const int tid = threadIdx.x + threadIdx.y * blockDim.x;
  if (tid == 0) {
    __threadfence();
    const unsigned ticket = atomicAdd(counter, 1u);
    last = ticket == nblocks - 1;
  }
  __syncthreads();
  if (last) __threadfence();
  return last != 0;
}

// totals[q] = sum over blocks b of partials[b * stride + q] for q < n.
// Component q is reduced by wave q % W, two components at a time; its lanes
// take the blocks in a fixed stride (8 independent loads in flight each) and the
// wave sums them in a fixed order, so all components finish in a few round
// trips.  NT: threads of the block (0: as launched).  Ends with a barrier.
template <int NT = 0>
__device__ inline void reduce_partials(const double* partials, int nblocks, int stride, int n,
                                       double* totals) {
  const int W = (NT > 0 ? NT : (int)(blockDim.x * blockDim.y)) / kWave;
  constexpr int kBatch = 8;
  const int tid = threadIdx.x + threadIdx.y * blockDim.x;
  const int wave = tid / kWave, lane = tid % kWave;
  for (int q = wave; q < n; q += 2 * W) {
    const int q2 = q + W < n ? q + W : q;
    double s = 0.0, s2 = 0.0;
    for (int b0 = lane; b0 < nblocks; b0 += kWave * kBatch) {
      double v[kBatch], v2[kBatch];
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        const int b = b0 + u * kWave;
        v[u] = b < nblocks ? partials[(size_t)b * stride + q] : 0.0;
        v2[u] = b < nblocks ? partials[(size_t)b * stride + q2] : 0.0;
      }
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        s += v[u];
        s2 += v2[u];
      }
    }
    s = wave_sum(s);
    s2 = wave_sum(s2);
    if (lane == 0) {
      totals[q] = s;
      totals[q2] = s2;
    }
  }
  __syncthreads();
}

// Copies the run state into LDS, where the recording thread reads it after
// the next barrier: its loads then overlap those of the partial sums.
__device__ inline void snapshot_state(const RunState* st, RunState* snap) {
  static_assert(sizeof(RunState) % 4 == 0, "copied in words");
  const int tid = threadIdx.x + threadIdx.y * blockDim.x, nt = blockDim.x * blockDim.y;
  for (int i = tid; i < (int)(sizeof(RunState) / 4); i += nt) ((uint32_t*)snap)[i] = ((const uint32_t*)st)[i];
}

// Thread 0 of the last block: turns the reduced sums of T consecutive steps
// (tot[s * kAcc + q]) into trace records and updates the run state and the
// stop decision (trace may be NULL: no per-step records kept).  Works on
// register copies of the fields it updates (a whole-struct copy would pass
// the untouched fields through private memory); now: the state as it stands
// (gst itself, or a copy in LDS).  inject_at >= 0: a pulse of
// a batched pulse train released inj_pos and inj_neg ions before the step
// step0 + inject_at, which are booked with that step.  Returns the stop flag left
// (ALONE: by a launch without tile blocks): the launch's parity is that of the
// launches recorded so far plus one, as it records the launch before it.
template <bool ALONE = false>
__device__ inline int finalize_steps(RunState* gst, const RunState* now, double* trace, const double* tot, int T,
                                      int64_t step0, const Coef& cp, const Coef& cn, double dV,
                                      double stop_tol, int64_t min_stop_step, int inject_at = -1,
                                      double inj_pos = 0.0, double inj_neg = 0.0) {
  double released = now->released, released_neg = now->released_neg;
  double pending = now->released_pending, pending_neg = now->released_pending_neg;
  double sums[5], last[4], screened[2], escaped[2];
#pragma unroll
  for (int q = 0; q < 5; ++q) sums[q] = now->sums[q];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    screened[q] = now->screened[q];
    escaped[q] = now->escaped[q];
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) last[q] = now->last[q];
  int64_t steps = now->steps;
  const int stop = ALONE ? kStopAll : stop_after((now->passes + 1) & 1);
  int done = 0, flags = now->flags;
  const int64_t period_step = now->period_step;
  bool injected = false;
  for (int s = 0; s < T && !done; ++s) {
    const int64_t l = step0 + s;
    const double* a = tot + s * kAcc;
    if (s == inject_at) {
      released += inj_pos;
      released_neg += inj_neg;
      pending += inj_pos;
      pending_neg += inj_neg;
      injected = true;
    }
    double rec[IT_TRACE_COLS];
    rec[0] = a[0] * dV;
    rec[1] = cp.azp * a[1] * dV;
    rec[2] = cp.azm * a[2] * dV;
    rec[3] = cn.azp * a[3] * dV;
    rec[4] = cn.azm * a[4] * dV;
    rec[5] = a[5] * dV;
    rec[6] = a[6] * dV;
    rec[7] = a[7] * dV;
    rec[8] = a[8] * dV;
    rec[9] = pending;
    rec[10] = a[9] * dV;
    rec[11] = a[10] * dV;
    rec[12] = pending_neg;
    rec[13] = a[11] * dV;
    rec[14] = a[12] * dV;
    pending = 0.0;
    pending_neg = 0.0;
    if (l == period_step) {  // the last period of a pulse train begins with this step
#pragma unroll
      for (int q = 0; q < 5; ++q) gst->period_sums[q] = sums[q];
      gst->period_rel[0] = rec[9];
      gst->period_rel[1] = rec[12];
      gst->period_started = 1;
    }
    bool finite = true;
#pragma unroll
    for (int q = 0; q < IT_TRACE_COLS; ++q) {
      if (trace) trace[l * IT_TRACE_COLS + q] = rec[q];
      finite = finite && isfinite(rec[q]);
    }
#pragma unroll
    for (int q = 0; q < 5; ++q) sums[q] += rec[q];
#pragma unroll
    for (int q = 0; q < 4; ++q) last[q] = rec[5 + q];
    screened[0] += rec[10];
    screened[1] += rec[11];
    escaped[0] += rec[13];
    escaped[1] += rec[14];
    steps = l + 1;
    if (!finite) {
      flags |= IT_FLAG_NONFINITE;
      done = stop;
    } else if (l >= min_stop_step && rec[7] <= stop_tol * released && rec[8] <= stop_tol * released_neg) {
      done = stop;
    }
  }
  gst->released_pending = pending;
  gst->released_pending_neg = pending_neg;
  if (injected) {
    gst->released = released;
    gst->released_neg = released_neg;
    gst->released_q = now->released_q + inj_neg;  // negative charge: the ions (no free electrons in a train)
  }
#pragma unroll
  for (int q = 0; q < 5; ++q) gst->sums[q] = sums[q];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    gst->screened[q] = screened[q];
    gst->escaped[q] = escaped[q];
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) gst->last[q] = last[q];
  gst->steps = steps;
  gst->done = done;
  gst->flags = flags;
  gst->passes = now->passes + 1;
  return done;
}

// Tile coordinates: column tile (tx, ty) and z chunk.
struct TileCoord {
  int tx, ty, zc;
  bool valid;
};

// Tile l of a tiling with tiles_x x tiles_y columns and zchunks chunks, in
// the order (chunk, row, column): consecutive tiles are lateral neighbours
// at the same depth, so a run of them on one XCD shares the rim rows and
// columns through that XCD's L2 while they march up z together.
__device__ inline TileCoord tile_of(int l, int tiles_x, int tiles_y) {
  TileCoord t;
  t.tx = l % tiles_x;
  const int rest = l / tiles_x;
  t.ty = rest % tiles_y;
  t.zc = rest / tiles_y;
  return t;
}

// Block -> tile, XCD-aware: the dispatcher deals blocks to the 8 XCDs in
// turn, so block b runs on XCD b % 8; XCD x gets the contiguous tile run
// [x * per_xcd, (x + 1) * per_xcd).
__device__ inline TileCoord decode_tile(int tiles_x, int tiles_y, int ntiles, int per_xcd) {
  const int b = blockIdx.x;
  const int L = (b & 7) * per_xcd + (b >> 3);
  const bool valid = L < ntiles;
  TileCoord t = tile_of(valid ? L : 0, tiles_x, tiles_y);
  t.valid = valid;
  return t;
}

}  // namespace it
