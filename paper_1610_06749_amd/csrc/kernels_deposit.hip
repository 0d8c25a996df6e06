// Deposition (eq. Gaussian around each track axis, eq. linear_density for N0).
//
// A block owns 256 consecutive nodes of a plane (rows run on, so no lane idles
// on narrow cells) and a chunk of planes.  Tracks parallel to the field give
// the same density on every plane, so their sum is formed once per node
// column; tilted tracks are evaluated per node, four planes at a time.  The
// perpendicular distance is |w x u| with w the node's offset from the axis
// point (x0, y0, d/2), its transverse part wrapped to the nearest periodic
// image (taken as it is with absorbing lateral boundaries); the profile is cut
// at r^2 > (8 b)^2.
//
// Each wave first sorts out the tracks whose cut lies beyond all of its nodes:
// its lanes test 64 tracks at once against the wave's rectangle of nodes, and
// only those that pass are evaluated, in the order given (a track left out
// would have added zero).  With 400 tracks on 256 x 256 nodes a wave evaluates
// a tenth of them.
//
// What bounds it is HBM.  The first deposit of a run writes the densities (and
// the zeros of the electrode planes) without reading what was there, so no
// field is cleared beforehand; a later one reads everything, for the largest
// density, and writes only where a wave adds something.  Before, every deposit
// read and wrote everything and evaluated every track at every node.  On
// MI355X: 400 tracks on 256 x 256 x 200 nodes 182 us (571 and 75 for clearing
// the fields before), a later tilted track on 512 x 512 x 256 nodes 416 us
// (826), all deposits of 192 chambers of 24 x 24 nodes 0.48 ms in one launch
// (4.7 ms in 1152 launches), of 16 chambers of 64 to 256 nodes square 1.1 ms
// (6.1 ms).
#include "reduce.h"

namespace it {

namespace {

constexpr int kDNT = 256;   // threads of a block, nodes of its tile
constexpr int kPlanes = 4;  // planes taken at a time

__device__ inline double wrap_near(double d, double L) { return d - L * floor(d / L + 0.5); }

__device__ inline double lateral_offset(const DepositParams& p, double d, double L) {
  return p.absorbing ? d : wrap_near(d, L);
}

__device__ inline double axis_r2(const DepTrack& tr, double wx, double wy, double wz) {
  const double cx = wy * tr.uz - wz * tr.uy;
  const double cy = wz * tr.ux - wx * tr.uz;
  const double cz = wx * tr.uy - wy * tr.ux;
  return cx * cx + cy * cy + cz * cz;
}

// Densities of the positive and (with its own radius) negative ions.
__device__ inline void track_values(const DepTrack& tr, double wx, double wy, double wz, bool same,
                                    double& dp, double& dn) {
  const double r2 = axis_r2(tr, wx, wy, wz);
  dp = r2 > tr.cut2 ? 0.0 : tr.peak * exp(-r2 * tr.inv_b2);
  dn = same ? dp : (r2 > tr.cut2_n ? 0.0 : tr.peak_n * exp(-r2 * tr.inv_b2_n));
}

// A rectangle of nodes (centre and half extents) and a range of heights over
// mid-gap.
struct Box {
  double xc, yc, hx, hy, z_lo, z_hi;
};

// Smallest distance along one axis between the rectangle's offsets from the
// track (centre c, half extent h) and the axis's shift at the heights of the
// box (between s0 and s1); 0 where the rectangle may wrap.
__device__ inline double gap_1d(const DepositParams& p, double centre, double axis, double h, double L, double s0,
                                double s1) {
  const double w = lateral_offset(p, centre - axis, L);
  if (!p.absorbing && fabs(w) + h > 0.499 * L) return 0.0;  // some nodes may take another image
  const double lo = w - h - fmax(s0, s1), hi = w + h - fmin(s0, s1);
  const double rounding = 1e-14 * (fabs(axis) + L + fabs(s0) + fabs(s1));  // of these and of a node's own offset
  return fmax(0.0, fmax(lo, -hi) - rounding);
}

// False only if the track's density is zero on every node of the box: at one
// height, the perpendicular distance is at least u_z times the transverse
// distance from the axis.
__device__ inline bool track_near(const DepositParams& p, const DepTrack& tr, const Box& b) {
  const double uz = fabs(tr.uz);
  if (!(uz > 1e-3)) return true;
  const double tx = tr.ux / tr.uz, ty = tr.uy / tr.uz;
  const double gx = gap_1d(p, b.xc, tr.x0, b.hx, p.Lx, b.z_lo * tx, b.z_hi * tx);
  const double gy = gap_1d(p, b.yc, tr.y0, b.hy, p.Ly, b.z_lo * ty, b.z_hi * ty);
  const double cut2 = fmax(tr.cut2, tr.cut2_n);
  return !(uz * uz * (gx * gx + gy * gy) > 1.000001 * cut2);
}

// Calls f(track) for the tracks of tr[0..n) near the box, in order (the same
// for the whole wave).
template <class F>
__device__ inline void for_near(const DepositParams& p, const DepTrack* tr, int n, const Box& b, F f) {
  const int lane = threadIdx.x % kWave;
  for (int base = 0; base < n; base += kWave) {
    unsigned long long m = __ballot(base + lane < n && track_near(p, tr[base + lane], b));
    while (m) {
      const int q = base + __builtin_ctzll(m);
      m &= m - 1;
      f(tr[q]);
    }
  }
}

// Tile l of the deposit: its densities, and its partial sums and largest
// density into p.partials; the last tile of the deposit to arrive books them.
__device__ inline void deposit_tile(const DepositParams& p, int l) {
  constexpr int NP = 5;  // partials: released n+, n- ions, electrons, negative charge; max density
  __shared__ double lds[(kDNT / kWave) * NP];
  double acc[NP] = {0.0, 0.0, 0.0, 0.0, 0.0};
  const bool same = p.same_radii != 0;
  const int lane = threadIdx.x % kWave;
  const int nx = p.nx, nz = p.nz;
  const unsigned plane = (unsigned)nx * p.ny;  // at most 2^28 (checked on the host)
  const int tile = l % p.tiles, zc = l / p.tiles;
  const unsigned node0 = (unsigned)tile * kDNT + (threadIdx.x - lane);  // the wave's first node
  const unsigned node = node0 + lane;
  const bool active = node < plane;
  const int k0 = 1 + zc * p.zc;
  const int k1 = min(k0 + p.zc, nz);
  if (node0 < plane) {  // wave-uniform
    const unsigned at = active ? node : plane - 1;
    const int j = (int)(at / (unsigned)nx), i = (int)(at - (unsigned)j * nx);
    const double x = i * p.dx, y = j * p.dy;
    Box box;
    {
      const unsigned last = min(node0 + kWave - 1, plane - 1);
      const int ja = (int)(node0 / (unsigned)nx), jb = (int)(last / (unsigned)nx);
      const int ia = ja == jb ? (int)(node0 - (unsigned)ja * nx) : 0;
      const int ib = ja == jb ? (int)(last - (unsigned)jb * nx) : nx - 1;
      box.xc = 0.5 * (ia + ib) * p.dx;
      box.hx = 0.5 * (ib - ia) * p.dx;
      box.yc = 0.5 * (ja + jb) * p.dy;
      box.hy = 0.5 * (jb - ja) * p.dy;
      box.z_lo = box.z_hi = 0.0;
    }
    double g0p = p.uniform, g0n = p.uniform;
    for_near(p, p.par, p.npar, box, [&](const DepTrack& tr) {
      double dp, dn;
      track_values(tr, lateral_offset(p, x - tr.x0, p.Lx), lateral_offset(p, y - tr.y0, p.Ly), 0.0, same, dp, dn);
      g0p += dp;
      g0n += dn;
    });
    for (int k = k0; k < k1; k += kPlanes) {
      double d_p[kPlanes], d_n[kPlanes];
#pragma unroll
      for (int u = 0; u < kPlanes; ++u) {
        d_p[u] = g0p;
        d_n[u] = g0n;
      }
      if (p.ntilt) {
        box.z_lo = k * p.dz - p.half_gap;
        box.z_hi = (k + kPlanes - 1) * p.dz - p.half_gap;
        for_near(p, p.tilt, p.ntilt, box, [&](const DepTrack& tr) {
          const double wx = lateral_offset(p, x - tr.x0, p.Lx), wy = lateral_offset(p, y - tr.y0, p.Ly);
#pragma unroll
          for (int u = 0; u < kPlanes; ++u) {
            double dp, dn;
            track_values(tr, wx, wy, (k + u) * p.dz - p.half_gap, same, dp, dn);
            d_p[u] += dp;
            d_n[u] += dn;
          }
        });
      }
      double old_p[kPlanes], old_n[kPlanes];
      size_t c = (size_t)k * plane + at;
      bool adds = false;
#pragma unroll
      for (int u = 0; u < kPlanes; ++u) {
        const bool there = k + u < k1;  // block-uniform
        old_p[u] = !p.fresh && there ? p.pos[c + (size_t)u * plane] : 0.0;
        old_n[u] = !p.fresh && there ? p.neg[c + (size_t)u * plane] : 0.0;
        adds = adds || d_p[u] != 0.0 || d_n[u] != 0.0;
      }
      const bool store = p.fresh || __any(adds);
#pragma unroll
      for (int u = 0; u < kPlanes; ++u, c += plane) {
        if (k + u >= k1 || !active) continue;
        const double a = old_p[u] + d_p[u];
        acc[0] += d_p[u];
        acc[3] += d_n[u];
        double b;
        if (p.free_e) {  // eq. ion_elec_distribution: ions (1 - e^{-a z}), electrons p (one deposit, fresh)
          const double di = d_n[u] * -expm1(-p.attach * ((k + u) * p.dz)), de = d_n[u] * p.pfree;
          b = old_n[u] + di;
          p.ele[c] = de;
          acc[1] += di;
          acc[2] += de;
          acc[4] = fmax(acc[4], fmax(a, b + de));
        } else {
          b = old_n[u] + d_n[u];
          acc[1] += d_n[u];
          acc[4] = fmax(acc[4], fmax(a, b));
        }
        if (store) {
          p.pos[c] = a;
          p.neg[c] = b;
        }
        if (p.pulse_pos) {
          p.pulse_pos[c] = a;
          p.pulse_neg[c] = b;
        }
      }
    }
    if (p.fresh && active) {  // the electrode planes of both field pairs
      if (k0 == 1) {
        p.pos[at] = p.neg[at] = p.pos2[at] = p.neg2[at] = 0.0;
        if (p.free_e) p.ele[at] = p.ele2[at] = 0.0;
      }
      if (k1 == nz) {
        const size_t c = (size_t)nz * plane + at;
        p.pos[c] = p.neg[c] = p.pos2[c] = p.neg2[c] = 0.0;
        if (p.free_e) p.ele[c] = p.ele2[c] = 0.0;
      }
    }
  }
  const int tid = threadIdx.x;
  auto block_sums = [&](double (&v)[NP], double (&r)[NP]) {  // r: of thread 0
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = wave_sum(v[q]);
    v[4] = wave_max(v[4]);
    __syncthreads();
    if (lane == 0)
      for (int q = 0; q < NP; ++q) lds[(tid / kWave) * NP + q] = v[q];
    __syncthreads();
    if (tid == 0) {
      for (int q = 0; q < NP; ++q) r[q] = lds[q];
      for (int w = 1; w < kDNT / kWave; ++w) {
        for (int q = 0; q < 4; ++q) r[q] += lds[w * NP + q];
        r[4] = fmax(r[4], lds[w * NP + 4]);
      }
    }
  };
  double r[NP];
  block_sums(acc, r);
  if (tid == 0)
    for (int q = 0; q < NP; ++q) p.partials[(size_t)l * NP + q] = r[q];
  if (!arrive_last<kDNT>(&p.state->dep_arrived, (unsigned)p.ntiles)) return;
  double v[NP] = {0.0, 0.0, 0.0, 0.0, 0.0};
  for (int b = tid; b < p.ntiles; b += kDNT) {
    for (int q = 0; q < 4; ++q) v[q] += p.partials[(size_t)b * NP + q];
    v[4] = fmax(v[4], p.partials[(size_t)b * NP + 4]);
  }
  block_sums(v, r);
  if (tid == 0) {
    RunState* st = p.state;
    st->released += r[0] * p.dV;
    st->released_pending += r[0] * p.dV;
    st->released_neg += r[1] * p.dV;
    st->released_pending_neg += r[1] * p.dV;
    st->released_e += r[2] * p.dV;
    st->released_q += r[3] * p.dV;
    st->max_beta_n = fmax(st->max_beta_n, p.beta * r[4]);
    st->dep_arrived = 0u;
  }
}

__global__ __launch_bounds__(kDNT) void deposit_kernel(DepositParams p) { deposit_tile(p, blockIdx.x); }

// The first deposits of all chambers of a batch in one launch: a block finds
// its chamber by binary search over the chambers' first tiles.
__global__ __launch_bounds__(kDNT) void deposit_batch_kernel(const DepositParams* __restrict__ table, int n) {
  const int l = blockIdx.x;
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (table[mid].tile_begin <= l) lo = mid; else hi = mid - 1;
  }
  deposit_tile(table[lo], l - table[lo].tile_begin);
}

}  // namespace

hipError_t launch_deposit(const DepositParams& p, hipStream_t s) {
  hipLaunchKernelGGL(deposit_kernel, dim3(p.ntiles), dim3(kDNT), 0, s, p);
  return hipGetLastError();
}

hipError_t launch_deposit_batch(const DepositParams* table, int n, int tiles, hipStream_t s) {
  hipLaunchKernelGGL(deposit_batch_kernel, dim3(tiles), dim3(kDNT), 0, s, table, n);
  return hipGetLastError();
}

}  // namespace it
