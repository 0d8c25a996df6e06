// One pass (T explicit time steps) of one block over the whole cross-section
// of a narrow periodic chamber and a chunk of planes: the batched kernel's
// tile where every chamber of the batch is narrow (kernels_section.hip).
//
// On a 24 x 24 chamber an extended tile of the blocked pass computes 2048
// nodes per plane and level for 576 owned ones.  Here the block holds exactly
// the cross-section: thread `tid` has R consecutive rows of one column
// (column tid % nx, rows (tid / nx) R ...), so there is no lateral rim, and
// the lateral neighbours are the periodic ones: rows of the thread from its
// registers, all others from LDS, where every level keeps its current plane
// (both species of a node together, 16-byte accesses; row r of thread tid at
// [r][tid], so a thread's own slots and its four neighbours' are five
// addresses with constant offsets).
//
// The block marches up the chunk as the blocked pass does: at iteration K
// level 0 is on plane K and level t computes plane K - t from level t-1 on
// planes K-t-1, K-t and K-t+1.  An iteration has two halves.  The first adds
// the lateral part and the sink of every level to a_{z-} times the plane
// below (all levels independent of each other, from the planes that stand in
// LDS); the second adds a_{z+} times the plane above, which is the one serial
// chain over the levels, tallies, and puts the new planes into LDS.  A barrier
// stands between the halves and one between iterations, so one copy of each
// plane suffices: LDS holds T planes, and several blocks share a CU and cover
// each other's barriers and LDS reads.
//
// What bounds it: issue and LDS together, each at half of its peak (per node,
// level and both species 25 FP64 instructions, 2.7 16-byte LDS reads and one
// write at three rows per thread), then the time of one iteration where few
// chambers run.  On MI355X, 192 chambers of 24 x 24 nodes and 26 800 planes in
// all take 45 us per step (mean of steps 90 to 282, no chamber stopping), 107 in
// blocked passes.
//
// Threads beyond the cross-section carry zeros (their loads and stores fall
// outside the plane's buffer and do nothing).
#pragma once

#include "stencil_blocked.h"

namespace it {

// PU: as in blocked_tile_pass (the pulse due after the step of level add_j).
// kAhead: 1 or 2, see above batch_section_kernel.
template <int T, int R, int NTP, bool PU, int kAhead>
__device__ __forceinline__ void section_pass(const StepParams& p, int chunk, double* partial_out, int add_j,
                                             const double* add_p, const double* add_n) {
  __shared__ double2_t lev[T][R][NTP];
  __shared__ double edge_sum[T][NTP / kWave][4];  // per-wave sums of n on the planes next to the electrodes
  __shared__ double wave_part[(NTP / kWave) * T * 5];

  const int tid = threadIdx.x;
  const int lane = tid % kWave;
  const int w = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int nwaves = blockDim.x / kWave;
  const int nx = p.nx, nz = p.nz;
  const int groups = p.ny / R;  // whole (checked on the host)
  const bool active = tid < groups * nx;
  const int g = tid / nx, x = tid - g * nx;
  const size_t plane = (size_t)nx * p.ny;
  const unsigned plane_bytes = (unsigned)plane * 8u;
  // slots of the four neighbours' threads (an idle thread: its own)
  const int left = !active ? tid : x > 0 ? tid - 1 : tid + nx - 1;
  const int right = !active ? tid : x < nx - 1 ? tid + 1 : tid - (nx - 1);
  const int above = !active ? tid : g > 0 ? tid - nx : tid + (groups - 1) * nx;
  const int below = !active ? tid : g < groups - 1 ? tid + nx : x;
  unsigned off[R];  // in-plane byte offsets; outside the plane for an idle thread
#pragma unroll
  for (int r = 0; r < R; ++r) off[r] = active ? (unsigned)((g * R + r) * nx + x) * 8u : kOutside;

  const int za = 1 + chunk * p.zc, zb = min(za + p.zc, nz);
  const Coef cp = p.cp, cn = p.cn;
  const double beta = p.beta;
  double add_max = 0.0;
  if (lane < 4)
#pragma unroll
    for (int t = 0; t < T; ++t) edge_sum[t][w][lane] = 0.0;

  // level t at the start of iteration K: its plane K-t-1 and, for the next
  // step's update on that plane, a_{z-} times its plane K-t-2
  double cpv[T][R], cnv[T][R], sp[T][R], sn[T][R];
  double acc[T][5];
#pragma unroll
  for (int t = 0; t < T; ++t) {
#pragma unroll
    for (int r = 0; r < R; ++r) cpv[t][r] = cnv[t][r] = sp[t][r] = sn[t][r] = 0.0;
#pragma unroll
    for (int q = 0; q < 5; ++q) acc[t][q] = 0.0;
  }
  // level 0's planes are loaded kAhead iterations ahead (two: into two buffers
  // that alternate)
  double pa[R], na[R], pb[R], nb[R];
  auto load0 = [&](int K, double (&lp)[R], double (&ln)[R]) {
    const int Kc = min(max(K, 0), nz);
    const rsrc_t bp = plane_rsrc(p.pin + (size_t)Kc * plane, plane_bytes);
    const rsrc_t bn = plane_rsrc(p.nin + (size_t)Kc * plane, plane_bytes);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      lp[r] = load_b64(bp, off[r]);
      ln[r] = load_b64(bn, off[r]);
    }
  };
  // the planes before the first, and finite values where no plane counts
#pragma unroll
  for (int t = 0; t < T; ++t)
#pragma unroll
    for (int r = 0; r < R; ++r) lev[t][r][tid] = double2_t{0.0, 0.0};
  // One iteration, straight-line but for what is rare: levels on planes that
  // no output depends on are computed all the same (their values are finite
  // and not used), those on an electrode or beyond are set to zero, and
  // planes that are not the chunk's enter the tallies times zero.
  auto iterate = [&](int K, double (&lp)[R], double (&ln)[R]) {
    lds_barrier();  // the planes written in the last iteration
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const double2_t up = lev[t][R - 1][above], dn = lev[t][0][below];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const double2_t l = lev[t][r][left], h = lev[t][r][right];
        const double pc = cpv[t][r], nc = cnv[t][r];
        const double bp = beta * pc;
        sp[t][r] += cp.a0 * pc;
        sn[t][r] += cn.a0 * nc;
        sp[t][r] += cp.ax * (l.x + h.x);
        sn[t][r] += cn.ax * (l.y + h.y);
        sp[t][r] += cp.ay * ((r > 0 ? cpv[t][r - 1] : up.x) + (r < R - 1 ? cpv[t][r + 1] : dn.x));
        sn[t][r] += cn.ay * ((r > 0 ? cnv[t][r - 1] : up.y) + (r < R - 1 ? cnv[t][r + 1] : dn.y));
        sp[t][r] -= bp * nc;
        sn[t][r] -= bp * nc;
      }
      // formed here, and not where it is used (the neighbours of every level
      // would stay in registers until then)
#pragma unroll
      for (int r = 0; r < R; ++r) asm volatile("" : "+v"(sp[t][r]), "+v"(sn[t][r]));
    }
    // the old values of a step next to an electrode (some level's plane of
    // this iteration is the chunk's first or last one and lies there)
    if ((za == 1 && K <= T + 1) || (zb == nz && K >= nz)) {
#pragma unroll
      for (int t = 0; t < T; ++t) {
        const int q = K - t - 1;
        if (!(q >= za && q < zb && (q == 1 || q == nz - 1))) continue;  // block-uniform
        double a = 0.0, b = 0.0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
          a += cpv[t][r];
          b += cnv[t][r];
        }
        a = wave_sum(a);
        b = wave_sum(b);
        if (lane == 0) {
          if (q == 1) {
            edge_sum[t][w][0] += a;
            edge_sum[t][w][2] += b;
          }
          if (q == nz - 1) {
            edge_sum[t][w][1] += a;
            edge_sum[t][w][3] += b;
          }
        }
      }
    }
    lds_barrier();  // every plane in LDS has been read
    double vp[R], vn[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      vp[r] = lp[r];
      vn[r] = ln[r];
    }
    load0(K + kAhead, lp, ln);  // past the chunk's last plane: a plane that is not used
#pragma unroll
    for (int t = 1; t <= T; ++t) {
      const int q = K - t;
      const bool interior = q >= 1 && q <= nz - 1, counted = q >= za && q < zb;  // block-uniform
      const double one = counted ? 1.0 : 0.0, beta_c = counted ? beta : 0.0;
      double np[R], nn[R];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        np[r] = sp[t - 1][r] + cp.azp * vp[r];
        nn[r] = sn[t - 1][r] + cn.azp * vn[r];
        np[r] = interior ? np[r] : 0.0;
        nn[r] = interior ? nn[r] : 0.0;
        acc[t - 1][0] += beta_c * cpv[t - 1][r] * cnv[t - 1][r];
        acc[t - 1][1] += one * np[r];
        acc[t - 1][2] += one * nn[r];
        acc[t - 1][3] += one * fabs(np[r]);
        acc[t - 1][4] += one * fabs(nn[r]);
      }
      if (PU && t == add_j && interior) {  // block-uniform: the pulse due after this level's step
        const rsrc_t pp = plane_rsrc(add_p + (size_t)q * plane, plane_bytes);
        const rsrc_t pn = plane_rsrc(add_n + (size_t)q * plane, plane_bytes);
#pragma unroll
        for (int r = 0; r < R; ++r) {
          np[r] += load_b64(pp, off[r]);
          nn[r] += load_b64(pn, off[r]);
          if (counted) add_max = fmax(add_max, fmax(np[r], nn[r]));
        }
      }
#pragma unroll
      for (int r = 0; r < R; ++r) {
        sp[t - 1][r] = cp.azm * cpv[t - 1][r];
        sn[t - 1][r] = cn.azm * cnv[t - 1][r];
        cpv[t - 1][r] = vp[r];
        cnv[t - 1][r] = vn[r];
        lev[t - 1][r][tid] = double2_t{vp[r], vn[r]};
        vp[r] = np[r];
        vn[r] = nn[r];
      }
#pragma unroll
      for (int k = 0; k < 5; ++k) asm volatile("" : "+v"(acc[t - 1][k]));  // summed here, not later
      __builtin_amdgcn_sched_barrier(0);
    }
    // Level T on plane K - T: the pass's output.  The stores are not branched
    // around (before the chunk's first plane they go to an empty buffer), so
    // that the number of accesses in flight is known and the wait for a plane
    // of level 0 is not one for the stores after it too.
    const unsigned bytes = K - T >= za ? plane_bytes : 0u;  // K - T < zb: the loop ends at zb + T - 1
    const size_t o = (size_t)max(K - T, 0) * plane;
    const rsrc_t op = plane_rsrc(p.pout + o, bytes), on = plane_rsrc(p.nout + o, bytes);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      store_b64(op, off[r], vp[r]);
      store_b64(on, off[r], vn[r]);
    }
  };
  const int Klo = za - T, Khi = zb + T - 1;
  load0(Klo, pa, na);
  if constexpr (kAhead == 2) {
    load0(Klo + 1, pb, nb);
    int K = Klo;
    for (; K + 1 <= Khi; K += 2) {
      iterate(K, pa, na);
      iterate(K + 1, pb, nb);
    }
    if (K <= Khi) iterate(K, pa, na);
  } else {
    for (int K = Klo; K <= Khi; ++K) iterate(K, pa, na);
  }

  // the block's T records: wave sums, then waves in index order
#pragma unroll
  for (int t = 0; t < T; ++t)
#pragma unroll
    for (int q = 0; q < 5; ++q) {
      const double s = wave_sum(acc[t][q]);
      if (lane == 0) wave_part[(w * T + t) * 5 + q] = s;
    }
  lds_barrier();  // and the edge sums of the last planes
  for (int i = tid; i < T * kAcc; i += blockDim.x) {
    const int t = i / kAcc, q = i - t * kAcc;
    double s = 0.0;
    if (q >= 1 && q <= 4) {
      for (int k = 0; k < nwaves; ++k) s += edge_sum[t][k][q - 1];
    } else if (q == 0 || q <= 8) {
      const int slot = q == 0 ? 0 : q - 4;
      for (int k = 0; k < nwaves; ++k) s += wave_part[(k * T + t) * 5 + slot];
    }
    partial_out[i] = s;
  }
  if (PU && add_j > 0) {  // block-uniform
    const double v = beta * wave_max(add_max);
    if (lane == 0)  // non-negative doubles order like their bit patterns
      atomicMax((unsigned long long*)&p.state->max_beta_n,
                (unsigned long long)__double_as_longlong(v > 0.0 ? v : 0.0));
  }
}

}  // namespace it
