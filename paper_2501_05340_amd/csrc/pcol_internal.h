// Internal declarations of the pcol HIP library: device helpers shared by the
// kernels and the launch wrappers the C-ABI layer calls.  gfx950 only.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#pragma clang fp contract(off)

namespace pcol {

// Cell-sorted start-of-step record of one sphere (64 B, one HBM burst).  It
// carries the sphere's caller index o (the tie-break key of the partner rule and
// the output position) and its box in the batched form, so binning writes one
// record per sphere and nothing else in sorted order; the mass, needed only
// for a collision, is read from the caller's array at o.
struct alignas(16) Rec {
  double x, y, z, r;
  double vx, vy, vz;
  int o;    // caller index
  int box;  // box of the batched form (0 otherwise)
};

// Sphere status during a step: ACTIVE has a valid partner key (or none yet),
// DIRTY is active but its partner collided with another sphere, so its key
// must be recomputed; FREE has no contact left in the step; COLLIDED is done.
enum : uint8_t { ST_ACTIVE = 0, ST_FREE = 1, ST_COLLIDED = 2, ST_DIRTY = 3 };

// End-of-step state of one collided sphere in cell-sorted order (64 B), copied
// to the caller's order by a final gather.
struct alignas(16) OutRec {
  double x, y, z, vx, vy, vz, t;
  int partner;          // caller index
  unsigned int pad;
};

// Uniform grid over the periodic box.  Cells are numbered (cz * nc1 + cy) * nc0 + cx,
// so the cells of one x-row are consecutive and so are their spheres after sorting.
//
// With the extent split (see k_cell_hist) the spheres of large extent sit in a
// second layer of the same cells, numbered layer2 + c; layer2 = 0 means one
// layer.  rho_max > 0 is the largest extent, which sets the radius of exact
// searches in a split grid; rho_max = 0 means cell side >= reach, so the 27
// surrounding cells hold every possible partner.
struct Grid {
  int nc[3];
  int ncell;        // cells of one layer
  double inv_h[3];  // nc / L, for cell assignment only
  double L[3];
  double halfL[3];  // 0.5 * L, the minimum-image threshold
  double h[3];      // L / nc, cell side
  int layer2;       // first cell of the second layer (0: none)
  int walls;        // bit k: reflective walls at 0 and L on axis k (else periodic)
  double rho_max;
  double inv_row;    // 1 / nc0 and 1 / (nc0 nc1): cell coordinates without division
  double inv_layer;
  double sL[3];      // periodic image shift: L on a periodic axis, 0 on a wall axis
};

// Coordinates of cell number c of one layer (c < 2^26, nc0 nc1 <= 2^20)
// without integer division: (c + 0.5) inv is within 2^-26 of the exact
// quotient, whose fractional part is at least 0.5 / divisor >= 2^-21 from an
// integer, so truncating it gives the exact floor.
__device__ __forceinline__ void cell_xyz(const Grid &G, int c, int &cx, int &cy, int &cz) {
  cz = (int)(((double)c + 0.5) * G.inv_layer);
  const int rem = c - cz * (G.nc[0] * G.nc[1]);
  cy = (int)(((double)rem + 0.5) * G.inv_row);
  cx = rem - cy * G.nc[0];
}

// Extent of a sphere over a step, r + |v| dt: two spheres can touch within the
// step only if their separation is at most the sum of their extents.  Written
// once so every kernel classifies a sphere identically.
__device__ __forceinline__ double extent(double r, double vx, double vy, double vz, double dt) {
  return r + __builtin_sqrt((vx * vx + vy * vy) + vz * vz) * dt;
}

// Range-free histogram of positive doubles: the top 16 bits of the binary64
// pattern (11 exponent bits, 4 fraction bits) over exponents 2^-64 .. 2^63,
// 16 bins per octave (bin width at most 1/16 of its lower edge).
constexpr int RHO_BINS = 2048;
__device__ __forceinline__ int rho_bin(double v) {
  const long long b = __double_as_longlong(v) >> 48;  // v > 0: exponent and 4 fraction bits
  const long long k = b - (long long)((1023 - 64) << 4);
  return k < 0 ? 0 : (k >= RHO_BINS ? RHO_BINS - 1 : (int)k);
}

// FP32 copy of a home sphere's record for the pair filter, staged in LDS by
// the detect kernel: position relative to the centre of the home cell, radius,
// velocity (32 B).
struct alignas(16) Rec32 {
  float x, y, z, r;
  float vx, vy, vz, pad;
};

// One workgroup's share of the reach pass: the bits of its maxima (of
// non-negative doubles, so they order as the values), of its smallest radius
// (+inf if none) and its validity bits.
constexpr int REACH_BLOCKS = 1024;
struct ReachPart {
  unsigned long long v2max, rmax, rmin, rhomax;
  unsigned int bad, pad;
};
__host__ __device__ inline ReachPart reach_merge(const ReachPart &a, const ReachPart &b) {
  return ReachPart{a.v2max > b.v2max ? a.v2max : b.v2max, a.rmax > b.rmax ? a.rmax : b.rmax,
                   a.rmin < b.rmin ? a.rmin : b.rmin, a.rhomax > b.rhomax ? a.rhomax : b.rhomax,
                   a.bad | b.bad, 0u};
}

// The grid of the literal order's space-filling curve: nc cells of side h =
// L / nc per axis (nc <= 2048), independent of the pair-test grid.
struct CurveGrid {
  int nc[3];
  double h[3];
};

// Scratch of the reach pass: REACH_BLOCKS partial results and the extent histogram
// (RHO_BINS bins, zero between passes).
struct ReachScratch {
  ReachPart *parts;
  unsigned int *hist;
};

// Exclusive scan: SCAN_T threads of SCAN_E cells per tile; the words (zero before
// a scan) hold each tile's sum or running total.
constexpr int SCAN_T = 1024;
constexpr int SCAN_E = 4;
constexpr int SCAN_B = SCAN_T * SCAN_E;
// Tiles of a scan of n cells (n up to 2^31 - 1: rounding up must not leave int).
__host__ __device__ constexpr int scan_tiles(int64_t n) {
  return (int)((n + (SCAN_B - 1)) / SCAN_B);
}
struct ScanState {
  int ticket, pad;
  unsigned long long word[1];  // one per tile, and one more
};

// What a step's plan is made of besides its data.
enum : unsigned int {
  PLAN_INVALID = 1u,   // non-finite value, r <= 0 or m <= 0
  PLAN_POSITION = 2u,  // position outside [0, L)
  PLAN_BOX = 4u,       // a box side <= 2 * reach
  PLAN_AGAIN = 8u      // not what the queued kernels were sized for: the host starts over
};
struct PlanArgs {
  int64_t n, cell_cap;
  double L[3], dt, cell_mult, band_rel, quantile;
  int home_cells, fp32, walls, curve;
  int allow_split, allow_small;  // kernels for them are queued behind the plan
  // the grid that the reach pass has counted the spheres on (tried)
  int tried, tried_nc[3], tried_layer2;
  double tried_rho_c;
};
struct StepPlan {
  unsigned int err;   // PLAN_* bits; nonzero: the step does nothing
  int hit;            // the spheres have been counted on this grid
  int small;          // some axis has fewer than 3 cells
  int split;
  int cells;          // of both layers
  int cpw;            // home cells per workgroup of the pair tests
  double reach, rho_c, rho_max;  // rho_c: +inf without a split
  double band, tol64, tol_wide;
  float kband, dt2f;
  Grid G;
  CurveGrid C;
};

// Contact-distance factor of the FP32 filter.  Bounds (unit roundoff u = 2^-24)
// on the FP32 errors of the filter quantities for any pair the binary64 rule
// can keep (|d| <= reach, |u| <= 2 vmax, coordinates within 1.5 h of the home
// cell centre):
//   separation   Dd = (2 h + reach) u       relative velocity  Du = 4 vmax u
//   c' = |d|^2 - (s k)^2:  2 sqrt3 reach Dd + 3 u reach^2 + 6 u (2 rmax k)^2
//   b' dt2f = d.u dt2f:    (sqrt3 (reach Du + 2 vmax Dd) + 6 u reach vmax) 2 dt (1 + 2^-11)
// The inflation (k^2 - 1) s_min^2 >= 2 (k - 1) s_min^2 must cover their sum; k
// is chosen so that it covers twice the sum, and never below 1 + band_rel.
// Returns the band.
__host__ __device__ inline double fp32_band(double h, double R, double V, double rmax, double rmin,
                                            double band_rel, double dt) {
  const double u = 0x1.0p-24, smin = 2.0 * rmin;
  const double k0 = 1.0 + band_rel + 1e-3;  // generous k for the radius term
  const double Dd = (2.0 * h + R) * u, Du = 4.0 * V * u;
  const double ec = 2.0 * sqrt(3.0) * R * Dd + 3.0 * u * R * R +
                    6.0 * u * (2.0 * rmax * k0) * (2.0 * rmax * k0);
  const double eb = (sqrt(3.0) * (R * Du + 2.0 * V * Dd) + 6.0 * u * R * V) * 2.0 * dt *
                    (1.0 + 0x1.0p-11);
  const double need = 2.0 * (ec + eb) / (2.0 * smin * smin);
  return band_rel > need ? band_rel : need;
}

// Tolerance of the binary64 Gram filter (filter 0).  The filter evaluates
// g = beta_i + <P_i, Q_j> (seven FMAs from beta_i) and passes the pair when
// g <= fl(tol - beta_j); in real numbers that is F = g + beta_j <= tol.  For a
// pair the rule keeps, the real F is at most
// E0 = 3 eps ((reach^2 + (2 r_max)^2) + reach 2 v_max dt2) (the binary64 argument:
// the kept root c / (-b + sqrt D) <= dt gives c <= 2 |b| dt (1 + 6 eps) < |b| dt2).
// The evaluation differs from the real F by
//  * the image shift of the candidate: one rounding per axis of a value below
//    L + h, so the separation d is off by at most delta = 2 eps (Lmax + h), which
//    moves F by at most delta (2 reach + 2 v_max dt2) + delta^2;
//  * beta_i, beta_j, Q, (a few roundings each, <= 6 eps relative) and the seven
//    FMAs of the sum (<= 7 eps of the sum of magnitudes): at most
//    16 eps (2 B + S) with B, S the bounds of |beta| and sum_k |P_k Q_k| for
//    |x| <= X, the norm of the box sides each lengthened by a cell;
//  * the threshold's one rounding, at most eps (tol + |beta_j|): the eps tol part
//    is covered by the factor two below, the eps B part by a 17th eps.
// The tolerance is twice the sum.
__host__ __device__ inline double gram64_tolerance(double X, double h, double R, double V,
                                                   double r, double Lmax, double dt2) {
  const double eps = 0x1.0p-53;
  X *= 1.0 + 1e-6;
  const double B = X * X + dt2 * X * V + r * r;
  const double S = X * (2.0 * X + dt2 * V) + V * dt2 * X + 2.0 * r * r;
  const double E0 = 3.0 * eps * ((R * R + 4.0 * r * r) + R * 2.0 * V * dt2);
  const double delta = 2.0 * eps * (Lmax + h);
  const double Epos = delta * (2.0 * R + 2.0 * V * dt2) + delta * delta;
  const double E = 17.0 * eps * (2.0 * B + S);
  return 2.0 * (E0 + Epos + E);
}

// Norm of the box sides, each lengthened by a cell: bounds every position and
// periodic image that the pair tests meet.
__host__ __device__ inline double grid_norm(const Grid &G) {
  double q = 0.0;
  for (int a = 0; a < 3; ++a) q += (G.L[a] + G.h[a]) * (G.L[a] + G.h[a]);
  return sqrt(q);
}

// The plan of a step from its reach pass: the verdict on the data, the split extent
// (kbin: the histogram bin where the split quantile of the extents falls, -1 for
// none), the grid and what the pair tests derive from it.
__host__ __device__ inline void make_plan(const PlanArgs &A, const ReachPart &r, int kbin,
                                          StepPlan &P) {
  union Bits {
    unsigned long long u;
    double d;
  };
  const double inf = __builtin_inf();
  P = StepPlan{};
  P.rho_c = inf;
  P.err = (r.bad & 1u ? PLAN_INVALID : 0u) | (r.bad & 2u ? PLAN_POSITION : 0u);
  if (P.err) return;
  const double rmax = Bits{r.rmax}.d, rmin = Bits{r.rmin}.d;
  const double vmax = __builtin_sqrt(Bits{r.v2max}.d);
  const double reach = 2.0 * rmax + 2.0 * vmax * A.dt;
  P.reach = reach;
  for (int a = 0; a < 3; ++a)
    if (!(A.L[a] > 2.0 * reach)) P.err = PLAN_BOX;
  if (P.err) return;
  // Extent split: the first layer holds the spheres whose extent is at most
  // rho_c, the upper edge of the bin; pairs of them are at most 2 rho_c apart
  // when they can touch.  Used only when it shrinks the cells enough to pay for
  // the separate search of the others, and the grid keeps 3 cells per axis.
  double rho_c = inf;
  if (A.quantile > 0.0 && A.quantile < 1.0 && A.n >= 4096 && kbin >= 0) {
    rho_c = Bits{(unsigned long long)((1023 - 64) * 16 + kbin + 1) << 48}.d;
    if (!(2.0 * rho_c < 0.85 * reach)) rho_c = inf;
    for (int a = 0; a < 3; ++a)
      if (A.L[a] / (2.0 * rho_c * A.cell_mult * (1.0 + 1e-9)) < 3.0) rho_c = inf;
  }
  const bool split = rho_c < inf;
  const double reach_pass = split ? 2.0 * rho_c : reach;
  // grid: cell side >= (split ? 2 rho_c : reach) * cell_mult, at most 2^26 cells per layer
  Grid &G = P.G;
  double cell = reach_pass * A.cell_mult;
  if (!(cell > 0.0)) cell = A.L[0];  // no motion and no size: one cell
  for (;;) {
    long long ncell = 1;
    for (int a = 0; a < 3; ++a) {
      double q = floor(A.L[a] / (cell * (1.0 + 1e-9)));
      if (!(q >= 1.0)) q = 1.0;
      if (q > 1024.0) q = 1024.0;
      G.nc[a] = (int)q;
      ncell *= G.nc[a];
    }
    if (ncell <= (1 << 26)) {
      G.ncell = (int)ncell;
      break;
    }
    cell *= 1.25;
  }
  G.walls = A.walls;
  double h = 0.0, Lmax = 0.0;
  for (int a = 0; a < 3; ++a) {
    const bool wall = (A.walls >> a) & 1;
    G.L[a] = A.L[a];
    // between walls there is no minimum image and no periodic image shift
    G.halfL[a] = wall ? inf : 0.5 * A.L[a];
    G.sL[a] = wall ? 0.0 : A.L[a];
    G.inv_h[a] = (double)G.nc[a] / A.L[a];
    G.h[a] = A.L[a] / G.nc[a];
    h = G.h[a] > h ? G.h[a] : h;
    Lmax = A.L[a] > Lmax ? A.L[a] : Lmax;
    if (G.nc[a] < 3) P.small = 1;
  }
  G.layer2 = split ? G.ncell : 0;
  P.rho_max = Bits{r.rhomax}.d;
  G.rho_max = split ? P.rho_max : 0.0;
  G.inv_row = 1.0 / G.nc[0];
  G.inv_layer = 1.0 / ((double)G.nc[0] * G.nc[1]);
  P.split = split;
  P.rho_c = rho_c;
  P.cells = split ? 2 * G.ncell : G.ncell;
  if ((long long)P.cells + 2 > A.cell_cap || (P.small && !A.allow_small) ||
      (split && !A.allow_split)) {
    P.err = PLAN_AGAIN;
    return;
  }
  P.hit = A.tried && A.tried_nc[0] == G.nc[0] && A.tried_nc[1] == G.nc[1] &&
          A.tried_nc[2] == G.nc[2] && A.tried_layer2 == G.layer2 &&
          (!split || A.tried_rho_c == rho_c);
  // sparse cells (the split grid holds about 13 spheres per cell at 16M): four
  // cells per workgroup, so their survivors are decided together; home_cells
  // overrides the choice
  P.cpw = P.small ? 0
                  : (A.home_cells > 0 ? A.home_cells : (A.n < 24 * (long long)G.ncell ? 4 : 1));
  // first-layer bounds: extent <= rho_c gives |v| <= (rho_c - r_min) / dt, r <= rho_c
  const double vb = (rho_c - rmin) / A.dt;
  const double V = split && vb < vmax ? vb : vmax, rp = split && rho_c < rmax ? rho_c : rmax;
  const double dt2 = 2.0 * A.dt * (1.0 + 0x1.0p-20);
  P.tol64 = gram64_tolerance(grid_norm(G), h, reach_pass, V, rp, Lmax, dt2);
  // pairs with a sphere above the split extent: |d| up to the full reach
  const double sw = 2.0 * rmax;
  P.tol_wide = 16.0 * 0x1.0p-53 * (reach * reach + sw * sw + reach * 2.0 * vmax * dt2);
  if (A.fp32 && !P.small) {
    P.band = fp32_band(h, reach_pass, V, rp, rmin, A.band_rel, A.dt);
    // round the factor up so the float never shrinks the inflation
    const double kb = 1.0 + P.band;
    P.kband = (float)kb;
    if ((double)P.kband < kb) P.kband = P.kband * (1.0f + 0x1.0p-23f);
  }
  P.dt2f = (float)(2.0 * A.dt * (1.0 + 0x1.0p-12));
  // the literal order's curve grid: cell side >= the reach (whatever grid the pair
  // tests use), at most 2048 cells per axis
  for (int a = 0; a < 3 && A.curve; ++a) {
    double q = floor(A.L[a] / (reach * (1.0 + 1e-9)));
    if (!(q >= 1.0)) q = 1.0;
    if (q > 2048.0) q = 2048.0;
    P.C.nc[a] = (int)q;
    P.C.h[a] = A.L[a] / P.C.nc[a];
  }
}

// Counters of a step, zero at its start.  Sums are spread over NSHARD counters on
// separate 128-B lines (one atomic per workgroup on shard blockIdx % NSHARD), so
// no single address takes an atomic per wave; the pairs of a sweep over four.
constexpr int NSHARD = 64;
constexpr int PAIR_SHARDS = 4;
constexpr int ACTIVE_SHARDS = 8;  // of a masked detect's active spheres
constexpr int MAX_QUEUE = 256;  // sweeps queued without the host looking at them
struct alignas(128) CounterShard {
  unsigned long long contacts;  // contacts found (each counted from both spheres)
  unsigned long long recheck;   // FP32 filter survivors rechecked in FP64 (counted per wave)
  unsigned long long tests;     // pair tests
  unsigned long long pairs;     // pairs resolved by the first sweep
  unsigned long long active;    // masked detect: its active spheres (zero between calls)
  unsigned long long pad[11];
};
struct alignas(128) ListShard {
  int n[3];  // spheres in this shard of the list of the later sweeps, three sweeps in turn
  int pad[29];
};
struct SweepCounters {
  CounterShard shard[NSHARD];
  ListShard list[NSHARD];
  unsigned int n_overflow;  // spheres with more contacts than slots (list length)
  unsigned int ovf_later;   // the same among those that took a new partner later
  unsigned int maxcell;     // largest cell occupancy
  unsigned int pad[29];
  unsigned long long pairs[MAX_QUEUE][PAIR_SHARDS];  // pairs resolved by each later sweep
};

// What the host reads of a step (page-locked host memory, written by k_finish).
struct StepReport {
  unsigned long long contacts, recheck, tests;
  unsigned int n_overflow, maxcell;
  int wide_first;  // sorted position of the first sphere above the split extent
  int small_sweeps, small_done, pad;  // k_sweeps_small: sweeps run, and whether the last found none
  unsigned long long small_pairs;     // and the pairs of them all
  unsigned long long pairs[MAX_QUEUE];
};

// ---------------------------------------------------------------- the rule

// Contact time of a pair from its minimum-image separation d = x_j - x_i and
// relative velocity u = v_j - v_i (rule 1 of pcol.h; eq. detect1/detect2).
__device__ __forceinline__ bool contact_time(double d0, double d1, double d2, double u0, double u1,
                                             double u2, double s, double dt, double &t) {
  const double a = (u0 * u0 + u1 * u1) + u2 * u2;
  const double b = (d0 * u0 + d1 * u1) + d2 * u2;
  const double c = ((d0 * d0 + d1 * d1) + d2 * d2) - s * s;
  if (!(a > 0.0) || !(b < 0.0) || !(c > 0.0)) return false;
  const double D = b * b - a * c;
  if (!(D >= 0.0)) return false;
  t = c / (-b + __builtin_sqrt(D));
  return t <= dt;
}

// Minimum-image separation along one axis (rule 1).
__device__ __forceinline__ double wrap_sep(double d, double L, double halfL) {
  if (d > halfL) {
    d = d - L;
  } else if (d < -halfL) {
    d = d + L;
  }
  return d;
}

// Final coordinate back into [0, L) (rule 5).
__device__ __forceinline__ double wrap_pos(double p, double L) {
  if (p >= L) {
    p = p - L;
  } else if (p < 0.0) {
    p = p + L;
  }
  if (p >= L) p = 0.0;
  return p;
}

// Time of flight of a centre at x with velocity v until it reaches a wall
// plane (x_k = 0 or L_k on a wall axis), +inf if it moves along no wall axis
// (Sec. "Particle Collisions": a collision counts only before an intersection
// with a domain boundary).
__device__ __forceinline__ double time_to_wall(double x0, double x1, double x2, double v0,
                                               double v1, double v2, const Grid &G) {
  const double x[3] = {x0, x1, x2}, v[3] = {v0, v1, v2};
  double tw = __longlong_as_double(0x7ff0000000000000LL);
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    if (!((G.walls >> k) & 1)) continue;
    double t;
    if (v[k] > 0.0)
      t = (G.L[k] - x[k]) / v[k];
    else if (v[k] < 0.0)
      t = -x[k] / v[k];
    else
      continue;
    tw = t < tw ? t : tw;
  }
  return tw;
}

// Contact at time t of spheres (xa, va) and (xb, vb) allowed by the walls:
// no later than either centre's time of flight to a wall.
__device__ __forceinline__ bool before_walls(double xa0, double xa1, double xa2, double va0,
                                             double va1, double va2, double xb0, double xb1,
                                             double xb2, double vb0, double vb1, double vb2,
                                             const Grid &G, double t) {
  return G.walls == 0 || (t <= time_to_wall(xa0, xa1, xa2, va0, va1, va2, G) &&
                          t <= time_to_wall(xb0, xb1, xb2, vb0, vb1, vb2, G));
}

// Exact contact time of two records with the canonical minimum image (none
// across a wall: halfL is +inf there).  The detect kernels record every such
// contact; the wall condition is applied where partners are chosen
// (k_slot_min, and pair_time_walls in the exact search).
__device__ __forceinline__ bool pair_time(const Rec &a, const Rec &b, const Grid &G, double dt,
                                          double &t) {
  const double d0 = wrap_sep(b.x - a.x, G.L[0], G.halfL[0]);
  const double d1 = wrap_sep(b.y - a.y, G.L[1], G.halfL[1]);
  const double d2 = wrap_sep(b.z - a.z, G.L[2], G.halfL[2]);
  return contact_time(d0, d1, d2, b.vx - a.vx, b.vy - a.vy, b.vz - a.vz, a.r + b.r, dt, t);
}

// pair_time, valid only before either sphere reaches a wall
__device__ __forceinline__ bool pair_time_walls(const Rec &a, const Rec &b, const Grid &G,
                                                double dt, double &t) {
  return pair_time(a, b, G, dt, t) &&
         before_walls(a.x, a.y, a.z, a.vx, a.vy, a.vz, b.x, b.y, b.z, b.vx, b.vy, b.vz, G, t);
}

// End of a flight along axis k, p the unconstrained coordinate: wrapped on a
// periodic axis; on a wall axis reflected at the plane crossed (a perfectly
// reflective wall, Sec. "Intersection of Particles with Solid Walls": the
// velocity component v changes sign), at most one plane per step; a coordinate
// that lands on L itself becomes the largest double below L.
__device__ __forceinline__ double fly_axis(double p, double L, bool wall, double &v) {
  if (!wall) return wrap_pos(p, L);
  if (p >= L) {
    p = L - (p - L);
    v = -v;
  } else if (p < 0.0) {
    p = -p;
    v = -v;
  }
  if (p >= L) p = nextafter(L, 0.0);
  return p;
}

// Post-collision state of sphere `a` colliding with `b` at time t (rule 4,
// Sec. "Inter-Particle Collisions" with friction 0, eq. update_vel/update_rho).
// Bitwise independent of which of the two is `a`.
__device__ __forceinline__ void resolve_one(const Rec &a, const Rec &b, double ma, double mb,
                                            const Grid &G, double t, double dt, double e,
                                            double out_x[3], double out_v[3]) {
  const double d0 = wrap_sep(b.x - a.x, G.L[0], G.halfL[0]);
  const double d1 = wrap_sep(b.y - a.y, G.L[1], G.halfL[1]);
  const double d2 = wrap_sep(b.z - a.z, G.L[2], G.halfL[2]);
  const double u0 = b.vx - a.vx, u1 = b.vy - a.vy, u2 = b.vz - a.vz;
  const double s = a.r + b.r;
  const double n0 = (d0 + t * u0) / s;
  const double n1 = (d1 + t * u1) / s;
  const double n2 = (d2 + t * u2) / s;
  const double g = (u0 * n0 + u1 * n1) + u2 * n2;
  const double mr = (ma * mb) / (ma + mb);
  const double J = (mr * (1.0 + e)) * g;
  const double ai = J / ma;
  out_v[0] = a.vx + ai * n0;
  out_v[1] = a.vy + ai * n1;
  out_v[2] = a.vz + ai * n2;
  const double rest = dt - t;
  out_x[0] = fly_axis((a.x + t * a.vx) + rest * out_v[0], G.L[0], G.walls & 1, out_v[0]);
  out_x[1] = fly_axis((a.y + t * a.vy) + rest * out_v[1], G.L[1], G.walls & 2, out_v[1]);
  out_x[2] = fly_axis((a.z + t * a.vz) + rest * out_v[2], G.L[2], G.walls & 4, out_v[2]);
}

// Angular velocities (caller order, updated in place for collided spheres) and
// the Coulomb friction coefficient of a step with spin; wx == nullptr: none.
struct Spin {
  double *wx, *wy, *wz;
  double mu;
};

// Post-collision state of sphere `a` colliding with `b` at time t with Coulomb
// friction mu and spins wa, wb (Sec. "Inter-Particle Collisions": impulse
// J = J_n n + J_t t_p, J_t = max(mu J_n, -(2/7)(1+e) m_r |v_rt|), jump
// relations of momentum and angular momentum; solid-sphere inertia m d^2 / 10,
// Sec. "Dispersed Phase").  The contact-point velocity is evaluated as
// v_r + (r_a w_a + r_b w_b) x n, so b's evaluation is the exact negation of a's
// and the two sides agree bitwise; with J_t = 0 the tangential terms are left
// out (then the velocity equals resolve_one's and the spin is unchanged).
__device__ __forceinline__ void resolve_one_spin(const Rec &a, const Rec &b, double ma, double mb,
                                                 const double wa[3], const double wb[3],
                                                 const Grid &G, double t, double dt, double e,
                                                 double mu, double out_x[3], double out_v[3],
                                                 double out_w[3]) {
  const double d0 = wrap_sep(b.x - a.x, G.L[0], G.halfL[0]);
  const double d1 = wrap_sep(b.y - a.y, G.L[1], G.halfL[1]);
  const double d2 = wrap_sep(b.z - a.z, G.L[2], G.halfL[2]);
  const double u[3] = {b.vx - a.vx, b.vy - a.vy, b.vz - a.vz};
  const double s = a.r + b.r;
  const double n[3] = {(d0 + t * u[0]) / s, (d1 + t * u[1]) / s, (d2 + t * u[2]) / s};
  const double g = (u[0] * n[0] + u[1] * n[1]) + u[2] * n[2];
  const double mr = (ma * mb) / (ma + mb);
  const double Jn = (mr * (1.0 + e)) * g;
  double S[3];
  for (int k = 0; k < 3; ++k) S[k] = a.r * wa[k] + b.r * wb[k];
  const double Sxn[3] = {S[1] * n[2] - S[2] * n[1], S[2] * n[0] - S[0] * n[2],
                         S[0] * n[1] - S[1] * n[0]};
  double vc[3];
  for (int k = 0; k < 3; ++k) vc[k] = -u[k] + Sxn[k];
  const double vcn = (vc[0] * n[0] + vc[1] * n[1]) + vc[2] * n[2];
  double vrt[3];
  for (int k = 0; k < 3; ++k) vrt[k] = vc[k] - vcn * n[k];
  const double vt = __builtin_sqrt((vrt[0] * vrt[0] + vrt[1] * vrt[1]) + vrt[2] * vrt[2]);
  double Jt = 0.0, tp[3] = {0.0, 0.0, 0.0};
  if (vt > 0.0) {
    for (int k = 0; k < 3; ++k) tp[k] = vrt[k] / vt;
    const double slide = mu * Jn;
    const double stick = -((((2.0 / 7.0) * (1.0 + e)) * mr) * vt);
    Jt = slide > stick ? slide : stick;
  }
  const double an = Jn / ma, at = Jt / ma;
  const double va[3] = {a.vx, a.vy, a.vz}, xa[3] = {a.x, a.y, a.z};
  const double rest = dt - t;
  for (int k = 0; k < 3; ++k) {
    double v = va[k] + an * n[k];
    if (Jt != 0.0) v = v + at * tp[k];
    double vk = v;  // reflected on a wall axis (the spin is unchanged by an elastic wall)
    out_x[k] = fly_axis((xa[k] + t * va[k]) + rest * v, G.L[k], (G.walls >> k) & 1, vk);
    out_v[k] = vk;
    out_w[k] = wa[k];
  }
  if (Jt != 0.0) {
    const double da = 2.0 * a.r;
    const double I = (ma * (da * da)) / 10.0;
    const double K = (a.r * Jt) / I;
    const double nxt[3] = {n[1] * tp[2] - n[2] * tp[1], n[2] * tp[0] - n[0] * tp[2],
                           n[0] * tp[1] - n[1] * tp[0]};
    for (int k = 0; k < 3; ++k) out_w[k] = wa[k] + K * nxt[k];
  }
}

__device__ __forceinline__ int cell_coord(double x, double inv_h, int nc) {
  int c = (int)(x * inv_h);
  c = c < 0 ? 0 : c;
  return c > nc - 1 ? nc - 1 : c;
}

// ---------------------------------------------------------------- launches

struct Particles {
  int64_t n;
  double *x, *y, *z, *vx, *vy, *vz;
  const double *r, *m;
  const double *wx = nullptr, *wy = nullptr, *wz = nullptr;  // spins, validated when given
};

// Boxes that one workgroup bins (k_bin_small): fewer spheres than a plan needs to
// split, and cells whose counts fit LDS.  And boxes that one workgroup sweeps
// (k_sweeps_small): up to two spheres a thread.  A step of 500, 1,000, 2,000, 3,000
// and 4,000 spheres (phi 0.05) takes 54, 60, 75, 91 and 106 us with it, and 74, 76,
// 82, 88 and 89 with the queued kernels, which the launches bound.
constexpr int SMALL_N = 4096;
constexpr int SMALL_CELLS = 8192;
constexpr int SMALL_TAIL = 2048;

// How a masked detect goes on: by the pair tests of all spheres and a choice among
// the slots of the active ones if more than one in 24 are active, else by the exact
// search of each active sphere.  Either leaves the same keys.  A call for 50,000,
// 300,000 and 2M spheres takes 30, 107 and 602 us with the pair tests whatever the
// mask, with the search 28, 69 and 309 us for one active in 64, 41, 145 and 728 us
// for one in 17 and 188, 1224 and 7970 us for all.
__device__ __forceinline__ bool masked_dense(const SweepCounters *ctr, int n) {
  unsigned long long active = 0ull;
#pragma unroll
  for (int k = 0; k < ACTIVE_SHARDS; ++k) active += ctr->shard[k].active;
  return active * 24ull > (unsigned long long)n;
}

// gradient with respect to a step's positions and velocities (SoA)
struct StateGrad {
  double *x, *y, *z, *vx, *vy, *vz;
};

// Device tables of the batched form: one grid per box, boxes' cells numbered
// consecutively (cell_base), the box of every sphere, and status flags that
// let every kernel of a captured step skip its work.
enum { FLAG_ERR = 0 };
enum : unsigned int { ERR_INVALID = 1u, ERR_REPLAN = 2u, ERR_BOX = 4u };
// A box's maxima during the batched reach pass (bits of non-negative doubles)
// and its validity bits; zero between passes.
struct BoxMax {
  unsigned long long v2, rm;
  unsigned int bad, pad;
};
// Spheres per workgroup of the batched reach pass (a box spans one or more).
constexpr int BREACH_CHUNK = 4096;

struct BatchDev {
  const Grid *gtab;       // [nbox]
  const int *cell_base;   // [nbox + 1]
  const int *box_of;      // caller order: box of each sphere
  const int64_t *box_off; // [nbox + 1] sphere ranges (caller order)
  double *breach;         // [nbox] reach found by the last step
  unsigned int *flags;    // FLAG_* words
  int nbox;
  int nchunk;             // chunks of the reach pass: box chunk_box[k], spheres from chunk_lo[k]
  const int *chunk_box;
  const int64_t *chunk_lo;
  BoxMax *bmax;           // [nbox]
};

// Everything the sweeps need.
struct SweepArgs {
  int n, K;
  int small;         // no contact slots: every search is exact
  int exact;         // the later sweeps can search (else a step with overflowing slots stops)
  int shards, shard_blocks;  // shards of the list, each with room for so many workgroups
  const Rec *rec;
  const int *start;
  const Grid *G;     // device: the single box's grid (null in the batched form)
  BatchDev B;        // tables of the batched form (gtab null: one box)
  double dt, e;
  const double *mass;
  const int *cnt, *slot_j;
  const double *slot_t;
  double *key_t;
  uint8_t *status;
  OutRec *out;
  int *list[2];      // n entries each and one workgroup more for each shard
  SweepCounters *ctr;
  const unsigned long long *crank;
  const unsigned int *err;  // nonzero: the step does nothing
  Spin spin;         // wx null: none
  int turn = 0, rekeyed = 0;  // host: sweeps over the list queued so far, and sweep 1's DIRTY done
};

// Everything the sweep-1 detect needs.
struct DetectArgs {
  const Rec *rec;
  const int *start;   // ncell + 1
  int *cnt;           // per sorted sphere: contacts found
  double *slot_t;     // [n * K]
  int *slot_j;        // [n * K]
  SweepCounters *ctr;
  int n;              // spheres (slot arrays are k-major: slot[k * n + i])
  int K;
  const StepPlan *plan;  // one box: grid and tolerances (null in the batched form)
  const unsigned int *err;  // one box: nonzero: do nothing
  int masked;         // only if a masked detect takes the pair tests (masked_dense)
  double dt;
  double dt2;         // 2 dt (1 + 2^-20): step bound of the FP64 filter
  double tol64;       // binary64 Gram filter tolerance (see gram64_tolerance)
  float kband;        // FP32 filter: contact distance inflated to s * kband
  float dt2f;         // FP32 filter: 2 dt (1 + 2^-12)
};

hipError_t launch_fill_u32(hipStream_t s, unsigned int *p, unsigned int v, int64_t n);
hipError_t launch_fill_i32(hipStream_t s, int *p, int v, int64_t n);
// The reach pass and the plan.  hist_shift: the extent histogram covers the
// spheres whose index is a multiple of 2^hist_shift.  G given: the pass also bins
// the spheres on G with split extent rho_c into cid, slot and count (zero on
// entry), as launch_cell_hist does.
hipError_t launch_reach(hipStream_t s, const Particles &P, double dt, int hist_shift,
                        const PlanArgs &A, const ReachScratch &R, SweepCounters *ctr,
                        ScanState *scan, StepPlan *plan, StepPlan *plan_host,
                        const Grid *G = nullptr, double rho_c = 0.0, int *cid = nullptr,
                        int *slot = nullptr, int *count = nullptr);
// tried_cells: cells of the grid that the reach pass counted on (0: none)
hipError_t launch_cell_hist(hipStream_t s, const Particles &P, const StepPlan *plan, double dt,
                            int tried_cells, int *cid, int *slot, int *count);
// the spheres of the second layer, if there is one
hipError_t launch_detect_wide(hipStream_t s, const DetectArgs &A);
// one-pass scan of plan->cells counts (ncell: as many as the host expects) or, with
// no plan, of ncell; clears the counts on request; *st zero on entry
hipError_t launch_scan(hipStream_t s, int *count, int ncell, const StepPlan *plan, int *start,
                        ScanState *st, unsigned int *maxcell, bool clear);
hipError_t launch_scatter(hipStream_t s, const Particles &P, const int *cid, const int *slot,
                          const int *start, Rec *rec, int *rank, int *cnt, const BatchDev *B,
                          const unsigned int *err);
hipError_t launch_detect_half(hipStream_t s, const DetectArgs &A, bool fp32, int groups);
hipError_t launch_slot_min(hipStream_t s, int n, const int *cnt, const double *slot_t,
                           const int *slot_j, int K, const Rec *rec, int *key_j, double *key_t,
                           int *ovf_list, SweepCounters *ctr, const unsigned int *err,
                           const Grid *G = nullptr,  // device: walls of the box (none: periodic)
                           const unsigned long long *crank = nullptr);  // literal order's ranks
hipError_t launch_gather_exact(hipStream_t s, const int *list, int nlist, const unsigned int *nlist_dev,
                               const Rec *rec, const int *start, const Grid *G, double dt, int *key_j,
                               double *key_t, const BatchDev *B, const unsigned int *err,
                               const unsigned long long *crank = nullptr);
hipError_t launch_masked_keys(hipStream_t s, const SweepCounters *ctr, int n, bool pairs, int K,
                              const int *cnt, const double *slot_t, const int *slot_j,
                              const Rec *rec, const int *start, const Grid *G, double dt,
                              const uint8_t *status, int *key_j, double *key_t);
hipError_t launch_curve_rank(hipStream_t s, const Rec *rec, int n, const StepPlan *plan,
                             unsigned long long *crank);
// The sweeps of a step (sweep_shards sets the list's shards).  first: every sphere;
// rekey: new partners for those it left DIRTY; sweep k >= 1: the list, keys in
// `in`, the next sweep's into `out`, the turn-th such sweep of the step.
void sweep_shards(SweepArgs &A);
hipError_t launch_sweep_first(hipStream_t s, const SweepArgs &A, const int *key);
hipError_t launch_rekey(hipStream_t s, const SweepArgs &A, int *key);
hipError_t launch_sweep(hipStream_t s, const SweepArgs &A, const int *in, int *out, int k,
                        bool first, int turn);
// the last nsweep sweeps have been queued: report, and the end-of-step state if the
// last of them resolved nothing
hipError_t launch_finish(hipStream_t s, const Particles &P, const int *rank, const OutRec *out,
                         const uint8_t *status, int *partner, double *tcoll, double dt,
                         const StepPlan *plan, const int *start, const BatchDev *B,
                         const SweepCounters *ctr, int nsweep, bool exact, const unsigned int *err,
                         StepReport *rep);
// P.n <= SMALL_N: the binning (reach, plan, sort, ranks), and everything after the
// pair tests, by one workgroup each
hipError_t launch_bin_small(hipStream_t s, const Particles &P, const PlanArgs &A,
                            SweepCounters *ctr, StepPlan *plan, StepPlan *plan_host, int *start,
                            Rec *rec, int *rank, int *cnt, unsigned long long *crank);
hipError_t launch_sweeps_small(hipStream_t s, const SweepArgs &A, const Particles &P, int *partner,
                               double *tcoll, int cap, StepReport *rep);
hipError_t launch_fill_box_of(hipStream_t s, int nbox, const int64_t *box_off, int *box_of);
// count given (zero on entry): the pass also takes every sphere's global cell
// (box's first cell + local cell on its planned grid) and its slot in that cell
// into cid, slot and count
hipError_t launch_breach(hipStream_t s, const Particles &P, const BatchDev &B, double dt,
                         int check_plan, int *cid = nullptr, int *slot = nullptr,
                         int *count = nullptr);
// cpw consecutive global cells per workgroup (one wave) over total_cells
hipError_t launch_detect_batched(hipStream_t s, const DetectArgs &A, const BatchDev &B,
                                 int total_cells, int cpw);
hipError_t launch_advance(hipStream_t s, const Particles &P, const int *partner, double dt,
                          const double L[3]);
// counts the active spheres into ctr's shards (zero on entry)
hipError_t launch_status_from_active(hipStream_t s, const uint8_t *active, const Rec *rec, int n,
                                     uint8_t *status, int *cnt, SweepCounters *ctr);
// status given: a masked detect ends (the counts of its active spheres are cleared)
hipError_t launch_export_keys(hipStream_t s, int n, const Rec *rec, const int *key_j,
                              const double *key_t, const uint8_t *status, SweepCounters *ctr,
                              uint64_t *key_out, double *tmin_out);
hipError_t launch_step_backward(hipStream_t s, const Particles &P, const Grid &G, double dt,
                                double e, const int *partner, const double *tcoll,
                                const StateGrad &gout, const StateGrad &gin, double *epart,
                                double *ge);  // epart: (n + 255) / 256 sums
// Deposition of per-sphere sources onto the corner nodes of a periodic
// Cartesian grid: positions x, y, z (n), sources a[q * n + i] (comp <= 8),
// nc cells of side h = L / nc per axis, out[node * comp + q] (nnode nodes,
// one per element).  Scratch: eid, slot (n each), cnt (nnode), start (nnode + 1), rec (n records of deposit_record_bytes(comp)).
struct DepositArgs {
  const double *x, *y, *z, *a;
  int64_t n;
  int comp;
  int nc[3];
  double L[3], h[3];
  int64_t nnode;
  double *out;
  int *eid, *slot, *cnt, *start;
  void *rec;
  ScanState *scan;
  unsigned int *flag;       // a position is bad: nothing of the caller's is written
  unsigned int *flag_host;  // nullable: host memory that receives the flag (n > 0)
};
int64_t deposit_record_bytes(int comp);
// element and slot of every sphere (clears cnt, scan and flag first); positions
// outside [0, L) or not finite set bit 0 of *flag and are skipped
hipError_t launch_deposit_count(hipStream_t s, const DepositArgs &D);
// after the scan of cnt into start: scatter, then element corner sums and node
// sums over tiles of nodes; known (nullable) is recorded behind the scatter, which
// writes *flag_host
hipError_t launch_deposit(hipStream_t s, const DepositArgs &D, hipEvent_t known);
hipError_t launch_resolve_public(hipStream_t s, int n, const Rec *rec, const int *rank,
                                 const Grid &G, double dt, double e, const uint64_t *key,
                                 const Particles &P, uint8_t *active, int *partner, double *tcoll,
                                 long long *npairs);

}  // namespace pcol
