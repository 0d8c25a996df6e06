// One temporally blocked pass (T explicit time steps) of one block over one
// extended tile: the device code shared by the single-chamber blocked
// kernel and the batched one.
//
// A block of 8 waves owns an extended tile of 64 columns by 8 R rows: lane l
// holds column l, and wave w the R consecutive rows w R .. w R + R - 1, in
// registers.  Every lane loads its periodically wrapped column, so lane and
// row neighbours are always the periodic x and y neighbours.  Each of the T
// steps (levels) is exact on one node less on every side, so after T steps
// the centre (64 - 2T) x (8 R - 2T) columns are exact: the block's owned
// columns.  The block marches up a chunk of planes with a software pipeline
// over the levels: at iteration K it has level 0 on plane K (loaded one or
// two iterations ahead) and computes level t on plane K - t for t = 1..T
// from level t-1 on planes K-t-1, K-t and K-t+1, which the thread keeps in
// registers (per level the current plane and a_{z-} times the one below it,
// plus the plane just computed).
//
// Lateral neighbours of level t-1 on plane K-t: x from the adjacent lanes
// (whole-wave DPP shifts), y from the thread's own rows; only the first and
// the last row of a wave's strip need the row of the wave above or below,
// which the waves exchange through LDS: at the end of an iteration every
// wave writes the edge rows of each level's newest plane into one of two
// buffers, and a single barrier at the top of the next iteration makes them
// visible (the other buffer is being read meanwhile).  Only level T goes
// back to HBM (non-temporal stores), so a pass reads and writes each owned
// node once for T steps; the price is the redundant work on the tile's rim
// and on the T planes of z halo at each end of a chunk.
//
// A level's rows are computed in straight-line code, stage by stage, and its
// tallies follow in a branch of their own; planes that no output of the chunk
// depends on are skipped (T (T + 1) of a chunk's T (zc + 2 T) level-planes).
// Against per-row branches, global addresses in vector registers and edge rows
// of one species per access: 184.8 us instead of 189 per step on the
// 512 x 512 x 256 grid, 39.7 instead of 40.2 on 256 x 256 x 200 (T = 3, R = 4).
// What bounds the pass is latency at two waves per SIMD: counters give VALU
// issue in 0.54 of the slots (23 FP64 instructions and 8 lane shifts per node,
// level and both species, 1.44 nodes computed per owned one on 512 x 512 x 256)
// and 0.58 of the HBM peak in traffic.  Without its loads and stores of planes it
// still took 156 of 185 us per step, so most of the rest is the chain of the
// levels, their LDS exchange and the barrier per plane, not HBM.
//
// The per-step tallies (the same quantities as the one-step kernel, one
// record per level) are taken on owned columns and on the block's own chunk
// of planes only, so every node and electrode face is counted once.
#pragma once

#include "stencil_plain.h"

namespace it {

constexpr int kBW = 8;                // waves per block
constexpr int kBX = 64;               // columns of the extended tile
constexpr int kBNT = kBW * kWave;     // threads per block

// A plane as a buffer resource: its base and size in scalar registers, so a
// node costs one 32-bit offset register, and an access beyond the plane reads
// zero or stores nothing.
typedef __amdgpu_buffer_rsrc_t rsrc_t;
typedef unsigned uint2_t __attribute__((ext_vector_type(2)));

__device__ inline rsrc_t plane_rsrc(const void* plane, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)(__attribute__((address_space(1))) void*)uniform_ptr(plane), 0, bytes,
                                           0x00027000);
}

__device__ inline double load_b64(rsrc_t r, unsigned off) {
  return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
}

constexpr unsigned kOutside = 0xfffffff0u;  // an offset beyond every plane

__device__ inline void store_b64(rsrc_t r, unsigned off, double v) {
  __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(uint2_t, v), r, off, 0, 0);
}

__device__ inline void store_b64_nt(rsrc_t r, unsigned off, double v) {
  constexpr int kNonTemporal = 2;
  __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(uint2_t, v), r, off, 0, kNonTemporal);
}

// Block b of a blocked launch of 8 per_xcd blocks -> its entry in the tile
// list.  A blocked block fills a CU, so a launch runs in rounds of 256
// blocks, 32 per XCD (the dispatcher deals blocks to the 8 XCDs in turn).
// Round r takes the 256 consecutive tiles from 256 r, XCD x the x-th run of
// them: each XCD works on a compact patch of lateral neighbours (their rims
// meet in its L2), and the patches of a round are neighbours too, so the
// rims between them are read by two XCDs at about the same time.  (Giving
// each XCD one contiguous run of the whole list instead put the XCDs on
// unrelated patches and took 2.7 % longer on the 512 x 512 x 256 grid.)
__device__ inline int blocked_tile_index(int b, int per_xcd) {
  constexpr int kXcds = 8, kCusPerXcd = 32;
  const int x = b % kXcds, j = b / kXcds;
  const int r = j / kCusPerXcd, within = j % kCusPerXcd;
  const int run = min(kCusPerXcd, per_xcd - kCusPerXcd * r);  // tiles per XCD in this round
  return kXcds * kCusPerXcd * r + run * x + within;
}

// Values of the neighbouring lanes (whole-wave DPP shifts by one lane); the
// lane at the wave's edge, which has no such neighbour, gets 0.
__device__ inline double lane_from_left(double v) {  // value of lane - 1
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), 0x138, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), 0x138, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}

__device__ inline double lane_from_right(double v) {  // value of lane + 1
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), 0x130, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), 0x130, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}

// One pass of the block over tile tc (tc.valid false: an idle block, which
// still stores zero partials); the block's T records of kAcc partial
// tallies go to partial_out.  The caller has checked the run's stop flag.
// PU: with add_j in 1..T (block-uniform), a pulse of a pulse train falls due
// after the step of level add_j: the densities add_p and add_n join that
// level's outputs once its tallies are taken (on every node the tile
// computes but those beyond an absorbing boundary, so the later levels step
// from them), and beta times the largest owned output enters the run's
// max_beta_n, as a deposit does.
// AB: honours p.absorbing (absorbing lateral boundaries; a batch mixes both
// kinds): the tile's nodes beyond the cell hold zero at every level
// instead of the periodic image, and each owned node next to the boundary
// adds a_x (a_y) times its old density per missing neighbour to the escaped
// tally of its species, as in the one-step kernel.
template <int T, int R, bool SC, bool PU = false, bool AB = false>
__device__ __forceinline__ void blocked_tile_pass(const StepParams& p, const TileCoord tc, double* partial_out,
                                                  int add_j = 0, const double* add_p = nullptr,
                                                  const double* add_n = nullptr) {
  constexpr int EY = kBW * R;             // rows of the extended tile
  constexpr int OX = kBX - 2 * T, OY = EY - 2 * T;
  constexpr int NE = SC ? 7 : 5;          // index of the escaped tallies (AB)
  constexpr int NA = NE + (AB ? 2 : 0);   // tallies kept per level
  // edge rows of each level's newest plane, both species of a node together
  // (16-byte accesses): [buffer][level][wave][first/last][lane]
  __shared__ double2_t edge_rows[2][T][kBW][2][kWave];
  __shared__ double edge_sum[T][kBW][4];  // per-wave sums of n on the planes next to the electrodes
  __shared__ double lds[(kBNT / kWave) * kAcc * T];

  const int lane = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.y);  // the wave (uniform)
  const int x0 = tc.tx * OX, y0 = tc.ty * OY;
  const int nx = p.nx, ny = p.ny, nz = p.nz;
  // wrapped position of this lane's column and of the thread's rows
  int xs = (x0 - T + lane) % nx;
  if (xs < 0) xs += nx;
  const bool own_x = lane >= T && lane < kBX - T && x0 + (lane - T) < nx;
  unsigned off[R];  // in-plane byte offsets of the thread's nodes
  bool own_y[R];    // the row is owned (wave-uniform)
  bool all_own = true;
  // absorbing: the node lies in the cell (else it holds zero), and the
  // missing neighbours of the lane's column and of each row
  const bool absorbing = AB && p.absorbing;
  const int gx = x0 - T + lane;
  const bool in_x = !absorbing || (gx >= 0 && gx < nx);
  const double miss_x = absorbing ? (double)((gx == 0) + (gx == nx - 1)) : 0.0;
  bool in_y[R];
  double miss_y[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int g = w * R + r;  // row in the extended tile
    int ys = (y0 - T + g) % ny;
    if (ys < 0) ys += ny;
    off[r] = (unsigned)(ys * nx + xs) * 8u;
    own_y[r] = tc.valid && g >= T && g < EY - T && y0 + (g - T) < ny;
    all_own = all_own && own_y[r];
    const int gy = y0 - T + g;
    in_y[r] = !absorbing || (gy >= 0 && gy < ny);
    miss_y[r] = absorbing ? (double)((gy == 0) + (gy == ny - 1)) : 0.0;
    // beyond an absorbing boundary: an offset outside the plane, which reads
    // zero (a select on the loaded value waited for each load at once)
    if (AB && !(in_x && in_y[r])) off[r] = kOutside;
  }
  const int za = 1 + tc.zc * p.zc;
  const int zb = tc.valid ? min(za + p.zc, nz) : za;
  const size_t plane = (size_t)nx * ny;
  const unsigned plane_bytes = (unsigned)plane * 8u;  // at most 2^31 (checked on the host)
  const Coef cp = p.cp, cn = p.cn;
  const double beta = p.beta, gsp = p.gsp, gsn = p.gsn;
  double add_max = 0.0;  // largest owned output density after a pulse is added

  if (lane < 4)
#pragma unroll
    for (int t = 0; t < T; ++t) edge_sum[t][w][lane] = 0.0;

  // level t (0..T-1) at the start of iteration K: cpv/cnv its plane K-t-1,
  // mp/mn the lower z-neighbour term of the next step's update on that plane,
  // a_{z-} times its plane K-t-2 (kept instead of the plane itself, so the
  // march shifts one register pair less per node, level and species)
  double mp[T][R], mn[T][R], cpv[T][R], cnv[T][R];
  double acc[T][NA];  // tallies of the owned rows, all columns (masked at the end)
#pragma unroll
  for (int t = 0; t < T; ++t) {
#pragma unroll
    for (int r = 0; r < R; ++r) mp[t][r] = mn[t][r] = cpv[t][r] = cnv[t][r] = 0.0;
#pragma unroll
    for (int q = 0; q < NA; ++q) acc[t][q] = 0.0;
  }

  const int Klo = za - T, Khi = zb + T - 1;
  // Level 0 of plane K into (lp, ln).  Planes before the anode and beyond the
  // cathode read the electrode plane itself, which always holds zero: the
  // loads need no branch or select, so they stay in flight across the
  // iteration (a branch around them made the compiler wait for them at once).
  // Where the registers allow (T R <= 12 and R <= 4: the default rows at
  // T = 3 and 4, and T = 2 passes cut short in such runs), two buffers
  // alternate and each plane is loaded two iterations ahead, the march taking
  // two iterations per loop trip (1 % faster on the 512 x 512 x 256 grid, 2 %
  // on the 96-chamber sweep); otherwise one buffer, one plane ahead.  The
  // absorbing terms and, at T = 4, the space-charge tallies take the registers
  // of the second one (T = 4 and three rows with space charge on 256 x 256 x 200
  // nodes: 69.5 us per step with two and 35 registers spilled, 52.3 with one).
  constexpr bool kTwoBuffers = T * R <= 12 && R <= 4 && !(AB && T * R > 9) && !(SC && T == 4);
  constexpr int kAhead = kTwoBuffers ? 2 : 1;
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
  // the zero planes' edge rows held at the start
#pragma unroll
  for (int t = 0; t < T; ++t) {
    edge_rows[Klo & 1][t][w][0][lane] = double2_t{0.0, 0.0};
    edge_rows[Klo & 1][t][w][1][lane] = double2_t{0.0, 0.0};
  }
  const int wu = w > 0 ? w - 1 : 0, wd = w < kBW - 1 ? w + 1 : kBW - 1;

  // One iteration: planes K - t of levels t = 1..T, then the edge rows of
  // every level's newest plane for the next iteration; level 0 of plane K
  // comes from (lp, ln), which then take the plane kAhead further (with two
  // buffers, past the chunk's last plane a clamped plane, unused).
  // The update of a level's rows is straight-line code, so that the compiler
  // interleaves their chains; the tallies follow in a branch of their own.
  auto iterate = [&](int K, double (&lp)[R], double (&ln)[R]) {
    const int buf = K & 1;
    lds_barrier();  // the edge rows written at the end of the previous iteration
    double vp[R], vn[R];  // the newest level's values, plane K - t
#pragma unroll
    for (int r = 0; r < R; ++r) {
      vp[r] = lp[r];
      vn[r] = ln[r];
    }
    // neighbours above the strip's first row and below its last, level t-1 on
    // plane K - t (the other waves' edge rows): requested one level ahead
    double2_t up = edge_rows[buf][0][wu][1][lane], dn = edge_rows[buf][0][wd][0][lane];
    if (kTwoBuffers || K + 1 <= Khi) load0(K + kAhead, lp, ln);
#pragma unroll
    for (int t = 1; t <= T; ++t) {
      const double2_t up_t = up, dn_t = dn;
      if (t < T) {
        up = edge_rows[buf][t][wu][1][lane];
        dn = edge_rows[buf][t][wd][0][lane];
      }
      __builtin_amdgcn_sched_barrier(0);
      const int q = K - t;  // plane of level t in this iteration (block-uniform)
      // planes this level has to have: those the chunk's last level depends
      // on, electrode planes and beyond hold zero (block-uniform)
      const bool wanted = q >= max(1, za - T + t) && q <= nz - 1;
      const bool counted = q >= za && q < zb;
      if (counted && (q == 1 || q == nz - 1)) {  // the old values of step t next to an electrode
        double sp_ = 0.0, sn_ = 0.0;
#pragma unroll
        for (int r = 0; r < R; ++r)
          if (own_y[r]) {
            sp_ += cpv[t - 1][r];
            sn_ += cnv[t - 1][r];
          }
        sp_ = wave_sum(own_x ? sp_ : 0.0);
        sn_ = wave_sum(own_x ? sn_ : 0.0);
        if (lane == 0) {
          if (q == 1) {
            edge_sum[t - 1][w][0] += sp_;
            edge_sum[t - 1][w][2] += sn_;
          }
          if (q == nz - 1) {
            edge_sum[t - 1][w][1] += sp_;
            edge_sum[t - 1][w][3] += sn_;
          }
        }
      }
      double np[R], nn[R];
      if (wanted) {
        double bp[R], scp[SC ? R : 1], scn[SC ? R : 1];
        // Two rows of both species at a time, stage by stage: four independent
        // chains whose links stand far enough apart (an FP64 result is ready
        // 8.5 cycles after its issue, which takes 4.5) for one wave to keep
        // issuing while the other of its SIMD waits.  The strip's first row
        // comes last: its upper neighbour comes from LDS.
#pragma unroll
        for (int i0 = 0; i0 < R; i0 += 2) {
          double xp[2], xn[2], yp[2], yn[2], ap[2], an[2];
          constexpr int kPair = 2;
          auto each = [&](auto f) {
#pragma unroll
            for (int u = 0; u < kPair; ++u)
              if (i0 + u < R) f(u, (i0 + u + 1) % R);
            __builtin_amdgcn_sched_barrier(0);
          };
          each([&](int u, int r) {
            xp[u] = lane_from_left(cpv[t - 1][r]) + lane_from_right(cpv[t - 1][r]);
            xn[u] = lane_from_left(cnv[t - 1][r]) + lane_from_right(cnv[t - 1][r]);
          });
          each([&](int u, int r) {
            bp[r] = beta * cpv[t - 1][r];
            ap[u] = mp[t - 1][r] + cp.a0 * cpv[t - 1][r];
            an[u] = mn[t - 1][r] + cn.a0 * cnv[t - 1][r];
          });
          each([&](int u, int r) {
            yp[u] = (r > 0 ? cpv[t - 1][r - 1] : up_t.x) + (r < R - 1 ? cpv[t - 1][r + 1] : dn_t.x);
            yn[u] = (r > 0 ? cnv[t - 1][r - 1] : up_t.y) + (r < R - 1 ? cnv[t - 1][r + 1] : dn_t.y);
          });
          each([&](int u, int) {
            ap[u] += cp.ax * xp[u];
            an[u] += cn.ax * xn[u];
          });
          each([&](int u, int) {
            ap[u] += cp.ay * yp[u];
            an[u] += cn.ay * yn[u];
          });
          each([&](int u, int r) {
            ap[u] += cp.azp * vp[r];
            an[u] += cn.azp * vn[r];
          });
          each([&](int u, int r) {
            ap[u] -= bp[r] * cnv[t - 1][r];
            an[u] -= bp[r] * cnv[t - 1][r];
            if constexpr (SC) {  // (not "+ 0.0" without it: x + 0 is not folded away, as -0 + 0 = +0)
              const double net = cpv[t - 1][r] - cnv[t - 1][r];
              scp[r] = gsp * cpv[t - 1][r] * net;
              scn[r] = gsn * cnv[t - 1][r] * net;
              ap[u] += scp[r];
              an[u] += scn[r];
            }
            if (AB && !(in_x && in_y[r])) ap[u] = an[u] = 0.0;  // beyond an absorbing boundary
            np[r] = ap[u];
            nn[r] = an[u];
          });
        }
        if (counted) {  // the columns are masked at the end
          auto tally = [&](int r) {
            acc[t - 1][0] += bp[r] * cnv[t - 1][r];
            acc[t - 1][1] += np[r];
            acc[t - 1][2] += nn[r];
            acc[t - 1][3] += fabs(np[r]);
            acc[t - 1][4] += fabs(nn[r]);
            if constexpr (SC) {
              acc[t - 1][5] += scp[r];
              acc[t - 1][6] += scn[r];
            }
            if constexpr (AB) {
              acc[t - 1][NE] += (cp.ax * miss_x + cp.ay * miss_y[r]) * cpv[t - 1][r];
              acc[t - 1][NE + 1] += (cn.ax * miss_x + cn.ay * miss_y[r]) * cnv[t - 1][r];
            }
          };
          if (all_own) {  // wave-uniform
#pragma unroll
            for (int r = 0; r < R; ++r) tally(r);
          } else {
#pragma unroll
            for (int r = 0; r < R; ++r)
              if (own_y[r]) tally(r);
          }
        }
      } else {
#pragma unroll
        for (int r = 0; r < R; ++r) np[r] = nn[r] = 0.0;
      }
      if (PU && t == add_j && wanted) {  // block-uniform: the pulse due after this level's step
        const rsrc_t pp = plane_rsrc(add_p + (size_t)q * plane, plane_bytes);
        const rsrc_t pn = plane_rsrc(add_n + (size_t)q * plane, plane_bytes);
#pragma unroll
        for (int r = 0; r < R; ++r) {
          np[r] += load_b64(pp, off[r]);
          nn[r] += load_b64(pn, off[r]);
          if (counted && own_y[r] && own_x) add_max = fmax(add_max, fmax(np[r], nn[r]));
        }
      }
      // level t-1 moves on: plane K-t gives the lower-neighbour term, K-t+1
      // becomes its current plane
#pragma unroll
      for (int r = 0; r < R; ++r) {
        mp[t - 1][r] = cp.azm * cpv[t - 1][r];
        mn[t - 1][r] = cn.azm * cnv[t - 1][r];
        cpv[t - 1][r] = vp[r];
        cnv[t - 1][r] = vn[r];
        vp[r] = np[r];
        vn[r] = nn[r];
      }
      // its edge rows, for the next iteration
      edge_rows[buf ^ 1][t - 1][w][0][lane] = double2_t{cpv[t - 1][0], cnv[t - 1][0]};
      edge_rows[buf ^ 1][t - 1][w][1][lane] = double2_t{cpv[t - 1][R - 1], cnv[t - 1][R - 1]};
    }
    // level T on plane K - T: the pass's output
    const int q = K - T;
    // The stores are not branched around (what is not owned, or not the
    // chunk's, goes to an offset outside the plane), so that the number of
    // accesses in flight is known and the wait for a plane of level 0 is not
    // one for the stores after it too.
    const bool out = q >= za && q < zb;
    const size_t o = (size_t)max(q, 0) * plane;
    const rsrc_t op = plane_rsrc(p.pout + o, plane_bytes), on = plane_rsrc(p.nout + o, plane_bytes);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const unsigned at = own_x && own_y[r] && out ? off[r] : kOutside;
      store_b64_nt(op, at, vp[r]);
      store_b64_nt(on, at, vn[r]);
    }
  };

  if (tc.valid) {
    load0(Klo, pa, na);
    if constexpr (kTwoBuffers) {
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
  }

  lds_barrier();  // edge sums of the last planes
  // block reduction of T records of kAcc slots (layout [level][slot]); the
  // tallies of columns outside the owned ones are selected away here
  double a[kAcc * T];
#pragma unroll
  for (int t = 0; t < T; ++t) {
    a[t * kAcc + 0] = own_x ? acc[t][0] : 0.0;
    a[t * kAcc + 1] = lane == 0 ? edge_sum[t][w][0] : 0.0;
    a[t * kAcc + 2] = lane == 0 ? edge_sum[t][w][1] : 0.0;
    a[t * kAcc + 3] = lane == 0 ? edge_sum[t][w][2] : 0.0;
    a[t * kAcc + 4] = lane == 0 ? edge_sum[t][w][3] : 0.0;
    a[t * kAcc + 5] = own_x ? acc[t][1] : 0.0;
    a[t * kAcc + 6] = own_x ? acc[t][2] : 0.0;
    a[t * kAcc + 7] = own_x ? acc[t][3] : 0.0;
    a[t * kAcc + 8] = own_x ? acc[t][4] : 0.0;
    if constexpr (SC) {
      a[t * kAcc + 9] = own_x ? acc[t][5] : 0.0;
      a[t * kAcc + 10] = own_x ? acc[t][6] : 0.0;
    } else {
      a[t * kAcc + 9] = 0.0;
      a[t * kAcc + 10] = 0.0;
    }
    if constexpr (AB) {  // escaped (absorbing boundaries)
      a[t * kAcc + 11] = own_x ? acc[t][NE] : 0.0;
      a[t * kAcc + 12] = own_x ? acc[t][NE + 1] : 0.0;
    } else {
      a[t * kAcc + 11] = 0.0;
      a[t * kAcc + 12] = 0.0;
    }
  }
  constexpr uint64_t kZero1 = (SC ? 0u : 3u << 9) | (AB ? 0u : 3u << 11), kLane1 = 0x1eu;
  uint64_t constexpr kLevels = T == 2 ? 1ull | 1ull << kAcc : T == 3 ? 1ull | 1ull << kAcc | 1ull << 2 * kAcc
                                                             : 1ull | 1ull << kAcc | 1ull << 2 * kAcc | 1ull << 3 * kAcc;
  static_assert(T >= 2 && T <= 4 && 4 * kAcc <= 64, "slot masks");
  block_sum_store<kAcc * T, kBNT, kZero1 * kLevels, kLane1 * kLevels>(a, partial_out, lds);
  if (PU && add_j > 0) {  // block-uniform
    __shared__ double wave_maxima[kBW];
    const double m = wave_max(add_max);
    if (lane == 0) wave_maxima[w] = m;
    __syncthreads();
    if (lane == 0 && w == 0) {
      double b = wave_maxima[0];
      for (int i = 1; i < kBW; ++i) b = fmax(b, wave_maxima[i]);
      const double v = beta * b;
      // non-negative doubles order like their bit patterns
      atomicMax((unsigned long long*)&p.state->max_beta_n,
                (unsigned long long)__double_as_longlong(v > 0.0 ? v : 0.0));
    }
  }
}


}  // namespace it
