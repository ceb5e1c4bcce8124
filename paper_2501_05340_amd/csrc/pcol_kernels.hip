// HIP kernels of the pcol collision step (gfx950, wave64).  Each kernel states
// the step of the method it implements; the rule numbers refer to the header
// comment of include/pcol.h.
#include "pcol_internal.h"

#include <math.h>

#include <algorithm>

namespace pcol {

namespace {

constexpr int WAVE = 64;

// Any object read or written by words: these may alias every type.
typedef unsigned long long __attribute__((may_alias)) Word64;

__device__ __forceinline__ unsigned long long dbits(double v) {
  return (unsigned long long)__double_as_longlong(v);
}

// Exclusive position of this lane among the lanes of the wave for which `pred`
// holds, and one atomic per wave on `counter` for all of them.  Returns the
// slot of this lane (valid only where pred).
__device__ __forceinline__ unsigned int wave_append(bool pred, unsigned int *counter) {
  const unsigned long long mask = __ballot(pred);
  if (mask == 0ull) return 0u;
  const unsigned int lane = __lane_id();
  const unsigned int below = __popcll(mask & ((1ull << lane) - 1ull));
  const int leader = __ffsll((long long)mask) - 1;
  unsigned int base = 0u;
  if ((int)lane == leader) base = atomicAdd(counter, (unsigned int)__popcll(mask));
  base = __shfl(base, leader);
  return base + below;
}

// Slot of this lane's key among all items of that key (key < 0: none, returns
// 0): consecutive lanes with one key (inputs stored in key order) share one
// atomic on count[key] per run and take consecutive slots.  Every lane of the
// wave must call it.
__device__ __forceinline__ int run_slot(int key, int *count) {
  const int lane = (int)__lane_id();
  const int prev = __shfl_up(key, 1);
  const unsigned long long starts = __ballot(lane == 0 || prev != key);
  const unsigned long long upto = starts & ((2ull << lane) - 1ull);  // bit 0 always set
  const int h = 63 - __clzll(upto);                                   // this lane's run start
  const unsigned long long after = starts & ~((2ull << lane) - 1ull);
  int base = 0;
  if (key >= 0 && lane == h) {
    const int len = (after ? __ffsll((long long)after) - 1 : WAVE) - h;
    base = atomicAdd(&count[key], len);
  }
  return __shfl(base, h) + (lane - h);
}

template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
  for (int o = WAVE / 2; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// blockIdx -> logical block so that each of the 8 XCDs (which receive
// workgroups round-robin) walks one contiguous range of logical blocks: spatial
// neighbours then share that XCD's L2.
__device__ __forceinline__ int xcd_remap(int bid, int nblocks) {
  const int q = nblocks / 8, r = nblocks % 8;
  const int x = bid % 8;
  return x * q + (x < r ? x : r) + bid / 8;
}

// Sum of v over the workgroup added to *target by one atomic (blockDim a
// multiple of the wave size, at most 1024 threads).
__device__ __forceinline__ void block_add(unsigned long long v, unsigned long long *target) {
  __shared__ unsigned long long part[1024 / WAVE];
  v = wave_sum(v);
  const int w = threadIdx.x / WAVE, nw = blockDim.x / WAVE;
  if (__lane_id() == 0) part[w] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long tot = 0ull;
    for (int k = 0; k < nw; ++k) tot += part[k];
    if (tot) atomicAdd(target, tot);
  }
  __syncthreads();
}

// Records of PARTS x 16 B that a wave writes at one position per lane go through
// the wave's own LDS, so that consecutive lanes store the parts of one record and
// an instruction writes whole records: a lane that stores its own 64 B does it in
// four instructions of 64 quarters, and the memory takes as many transactions (the
// sorted records of 16M spheres: 916 us, whole 600 us; runs of eight records in a
// row, but by quarters, took longer still).  Reads gain nothing from it: the caches
// merge the quarters (the copy back, 657 us either way).
struct alignas(16) Part16 {
  unsigned int w[4];
};

template <int PARTS>
struct Stage {
  Part16 part[WAVE * (PARTS | 1)];  // an odd number of parts a record: no bank conflicts
  int pos[WAVE];
};

// Each lane's record r to dst[pos] (pos < 0: none).  Every lane of the wave calls it.
template <typename R, int PARTS = sizeof(R) / 16>
__device__ __forceinline__ void store_records(const R &r, int pos, R *dst, Stage<PARTS> &S) {
  constexpr int STRIDE = PARTS | 1;
  const int lane = __lane_id();
  Part16 mine[PARTS];  // copied as bytes: the records are objects of other types
  static_assert(sizeof(R) == sizeof(mine), "whole parts");
  __builtin_memcpy(mine, &r, sizeof(R));
#pragma unroll
  for (int p = 0; p < PARTS; ++p) S.part[lane * STRIDE + p] = mine[p];
  S.pos[lane] = pos;
  __builtin_amdgcn_wave_barrier();  // (a wave's LDS operations stay in order)
#pragma unroll
  for (int q = 0; q < PARTS; ++q) {
    const int at = q * WAVE + lane, who = at / PARTS, p = at % PARTS;
    const int to = S.pos[who];
    if (to >= 0) {
      char *part = reinterpret_cast<char *>(dst + to) + p * sizeof(Part16);
      __builtin_memcpy(__builtin_assume_aligned(part, 16), &S.part[who * STRIDE + p],
                       sizeof(Part16));
    }
  }
  __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ CounterShard &my_shard(SweepCounters *ctr) {
  return ctr->shard[blockIdx.x % NSHARD];
}

}  // namespace

// ---------------------------------------------------------------- fills

__global__ void k_fill_u32(unsigned int *p, unsigned int v, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

static int fill_grid(int64_t n) {
  int64_t g = (n + 255) / 256;
  if (g > 4096) g = 4096;
  return g < 1 ? 1 : (int)g;
}

hipError_t launch_fill_u32(hipStream_t s, unsigned int *p, unsigned int v, int64_t n) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_u32, dim3(fill_grid(n)), dim3(256), 0, s, p, v, n);
  return hipGetLastError();
}
hipError_t launch_fill_i32(hipStream_t s, int *p, int v, int64_t n) {
  return launch_fill_u32(s, (unsigned int *)p, (unsigned int)v, n);
}

// ---------------------------------------------------------------- a1: reach + validation

// Largest |v|^2, radius and extent r + |v| dt, smallest radius, data validity,
// and the histogram of extents (Sec. "Collision Operator": the halo must hold
// every partner a sphere can reach within the step).  The maxima and the
// validity cover every sphere; the histogram, which only picks the split
// extent (a performance choice), covers the spheres whose index is a multiple
// of 2^hist_shift.  Grid-stride over at most REACH_BLOCKS workgroups; each
// histograms in LDS, adds the bins it has (some 50) to the result, and stores its
// maxima in parts, which k_plan reduces.  (Partial histograms and a kernel to add
// them up, 9 us at 1M spheres and 12 at 16M, cost more than up to 1024 adds to an
// address, 3 us at 1M and none at 16M, that end while others still read.)
// BIN: the same pass also takes each sphere's cell and slot on the grid G with
// split extent rho_c, exactly as k_cell_hist does (the binning of a step whose
// grid is planned before its reach is known; the plan is checked against the
// reach afterwards).  A sphere that fails the checks still gets a cell inside
// the grid, and the caller discards the pass.
template <bool BIN>
__global__ __launch_bounds__(256) void k_reach(Particles P, double L0, double L1, double L2,
                                               double dt, int hist_shift, ReachPart *parts,
                                               unsigned int *sum, Grid G, double rho_c, int *cid,
                                               int *slot, int *count) {
  __shared__ unsigned int hist[RHO_BINS];
  for (int k = threadIdx.x; k < RHO_BINS; k += 256) hist[k] = 0u;
  __syncthreads();
  double v2 = 0.0, rm = 0.0, rn = INFINITY, em = 0.0;
  unsigned int bad = 0u;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t hmask = ((int64_t)1 << hist_shift) - 1;
  // four elements per thread per step: their loads are issued together.  The
  // loop runs while the wave's first element is in range, so that every lane
  // of a wave takes each step (the binning's run_slot needs the whole wave);
  // lanes past the end hold no element.
  const int64_t wbase = blockIdx.x * (int64_t)blockDim.x + (threadIdx.x & ~(WAVE - 1));
  for (int64_t w0 = wbase; w0 < P.n; w0 += 4 * stride) {
    const int64_t i0 = w0 + (threadIdx.x & (WAVE - 1));
    double x[4], y[4], z[4], vx[4], vy[4], vz[4], r[4], m[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t i = i0 + u * stride;
      if (i < P.n) {
        x[u] = P.x[i];
        y[u] = P.y[i];
        z[u] = P.z[i];
        vx[u] = P.vx[i];
        vy[u] = P.vy[i];
        vz[u] = P.vz[i];
        r[u] = P.r[i];
        m[u] = P.m[i];
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const bool in = i0 + u * stride < P.n;
      bool has = false;
      int bin = -1;
      if (in) {
        const double w = (vx[u] * vx[u] + vy[u] * vy[u]) + vz[u] * vz[u];
        const bool fin = isfinite(x[u]) && isfinite(y[u]) && isfinite(z[u]) && isfinite(w) &&
                         isfinite(r[u]) && isfinite(m[u]);
        if (!fin || !(r[u] > 0.0) || !(m[u] > 0.0)) bad |= 1u;
        if (P.wx) {
          const int64_t i = i0 + u * stride;
          if (!isfinite(P.wx[i]) || !isfinite(P.wy[i]) || !isfinite(P.wz[i])) bad |= 1u;
        }
        if (!(x[u] >= 0.0 && x[u] < L0) || !(y[u] >= 0.0 && y[u] < L1) ||
            !(z[u] >= 0.0 && z[u] < L2))
          bad |= 2u;
        if (fin) {
          v2 = w > v2 ? w : v2;
          rm = r[u] > rm ? r[u] : rm;
          rn = r[u] < rn ? r[u] : rn;
          if (r[u] > 0.0) {
            const double ex = extent(r[u], vx[u], vy[u], vz[u], dt);
            em = ex > em ? ex : em;
            has = ((i0 + u * stride) & hmask) == 0;
            if (has) bin = rho_bin(ex);  // -1 (no lane's bin) for the others
          }
        }
      }
      if (BIN) {  // the cell and slot (every lane of the wave takes part)
        int c = -1;
        if (in) {
          const int cx = cell_coord(x[u], G.inv_h[0], G.nc[0]);
          const int cy = cell_coord(y[u], G.inv_h[1], G.nc[1]);
          const int cz = cell_coord(z[u], G.inv_h[2], G.nc[2]);
          c = (cz * G.nc[1] + cy) * G.nc[0] + cx;
          if (G.layer2 && !(extent(r[u], vx[u], vy[u], vz[u], dt) <= rho_c)) c += G.layer2;
        }
        const int sl = run_slot(c, count);
        if (c >= 0) {
          cid[i0 + u * stride] = c;
          slot[i0 + u * stride] = sl;
        }
      }
      // histogram: one LDS atomic per distinct bin of the wave (lanes of one
      // bin add together), so the few busy bins see no lane conflicts
      unsigned long long todo = __ballot(has);
      while (todo) {
        const int leader = __ffsll((long long)todo) - 1;
        const int lb = __shfl(bin, leader);
        const unsigned long long same = __ballot(bin == lb);
        if ((int)__lane_id() == leader) atomicAdd(&hist[lb], (unsigned int)__popcll(same));
        todo &= ~same;
      }
    }
  }
  for (int o = WAVE / 2; o > 0; o >>= 1) {
    const double a = __shfl_xor(v2, o), b = __shfl_xor(rm, o), c = __shfl_xor(rn, o),
                 d = __shfl_xor(em, o);
    v2 = a > v2 ? a : v2;
    rm = b > rm ? b : rm;
    rn = c < rn ? c : rn;
    em = d > em ? d : em;
    bad |= __shfl_xor(bad, o);
  }
  __shared__ ReachPart wpart[256 / WAVE];
  if (__lane_id() == 0)
    wpart[threadIdx.x / WAVE] = ReachPart{dbits(v2), dbits(rm), dbits(rn), dbits(em), bad, 0u};
  __syncthreads();
  if (threadIdx.x == 0) {
    ReachPart p = wpart[0];
    for (int w = 1; w < 256 / WAVE; ++w) p = reach_merge(p, wpart[w]);
    parts[blockIdx.x] = p;
  }
  for (int k = threadIdx.x; k < RHO_BINS; k += 256)
    if (hist[k]) atomicAdd(&sum[k], hist[k]);
}

// The step's plan from the reach pass (make_plan: the checks, the split extent,
// the grid and the tolerances that follow from them), by one workgroup, so that
// the kernels behind it can be queued without the host in between: they read the
// plan from device memory and do nothing when it says so (plan.err).  Written to
// the host's memory too.  Leaves the histogram, the step's counters and the
// scan's words zero.
__global__ __launch_bounds__(256) void k_plan(PlanArgs A, int nparts, const ReachPart *parts,
                                              unsigned int *hist, SweepCounters *ctr,
                                              ScanState *scan, StepPlan *plan,
                                              StepPlan *plan_host) {
  const int t = threadIdx.x;
  Word64 *w = (Word64 *)ctr;
  for (int k = t; k < (int)(sizeof(SweepCounters) / 8); k += 256) w[k] = 0ull;
  // the split quantile's bin: the first one whose running count reaches it
  constexpr int PER = RHO_BINS / 256;
  unsigned int h[PER], mine = 0u;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    h[k] = hist[t * PER + k];
    mine += h[k];
    hist[t * PER + k] = 0u;
  }
  ReachPart p{0ull, 0ull, dbits(INFINITY), 0ull, 0u, 0u};
  for (int k = t; k < nparts; k += 256) p = reach_merge(p, parts[k]);
  __shared__ unsigned int cum[256];
  __shared__ ReachPart red[256];
  __shared__ int bin;
  cum[t] = mine;
  red[t] = p;
  if (t == 0) bin = RHO_BINS;
  __syncthreads();
  for (int o = 1; o < 256; o <<= 1) {
    const unsigned int v = t >= o ? cum[t - o] : 0u;
    __syncthreads();
    cum[t] += v;
    __syncthreads();
  }
  for (int o = 128; o > 0; o >>= 1) {
    if (t < o) red[t] = reach_merge(red[t], red[t + o]);
    __syncthreads();
  }
  const double target = ceil(A.quantile * (double)cum[255]);
  unsigned int run = cum[t] - mine;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const bool before = (double)run < target;
    run += h[k];
    if (before && (double)run >= target) atomicMin(&bin, t * PER + k);
  }
  __syncthreads();
  __shared__ StepPlan out;
  if (t == 0) make_plan(A, red[0], bin < RHO_BINS - 1 ? bin : -1, out);
  __syncthreads();
  const Word64 *o = (const Word64 *)&out;
  for (int k = t; k < (int)(sizeof(StepPlan) / 8); k += 256) {
    ((Word64 *)plan)[k] = o[k];
    ((Word64 *)plan_host)[k] = o[k];
  }
  if (out.err != 0u) return;  // (then there may be no room for the cells either)
  for (int k = t; k <= scan_tiles(out.cells); k += 256) scan->word[k] = 0ull;
  if (t == 0) scan->ticket = 0;
}

hipError_t launch_reach(hipStream_t s, const Particles &P, double dt, int hist_shift,
                        const PlanArgs &A, const ReachScratch &R, SweepCounters *ctr,
                        ScanState *scan, StepPlan *plan, StepPlan *plan_host, const Grid *G,
                        double rho_c, int *cid, int *slot, int *count) {
  const int64_t g4 = (P.n + 1023) / 1024, g1 = (P.n + 255) / 256;
  int64_t g = std::max(g4, std::min(g1, (int64_t)128));
  if (g > REACH_BLOCKS) g = REACH_BLOCKS;
  if (g < 1) g = 1;
  if (G)
    hipLaunchKernelGGL(k_reach<true>, dim3((int)g), dim3(256), 0, s, P, A.L[0], A.L[1], A.L[2], dt,
                       hist_shift, R.parts, R.hist, *G, rho_c, cid, slot, count);
  else
    hipLaunchKernelGGL(k_reach<false>, dim3((int)g), dim3(256), 0, s, P, A.L[0], A.L[1], A.L[2],
                       dt, hist_shift, R.parts, R.hist, Grid{}, 0.0, nullptr, nullptr, nullptr);
  hipLaunchKernelGGL(k_plan, dim3(1), dim3(256), 0, s, A, (int)g, R.parts, R.hist, ctr, scan, plan,
                     plan_host);
  return hipGetLastError();
}

// ---------------------------------------------------------------- a2: cell id + histogram

// Cell of each sphere and its rank within the cell (one atomic per sphere, or
// per run of spheres of one cell in consecutive lanes).
// Extent split: a sphere whose extent r + |v| dt exceeds rho_c goes to the
// second layer of cells (number G.layer2 + c), searched separately; the first
// layer then only needs cells of side 2 rho_c.  rho_c = +inf: one layer.
// Not if the reach pass has counted on this very grid (plan.hit).
__global__ __launch_bounds__(256) void k_cell_hist(Particles P, const StepPlan *plan, double dt,
                                                   int *cid, int *slot, int *count) {
  if (plan->err || plan->hit) return;
  const Grid &G = plan->G;
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  int c = -1;
  if (i < P.n) {
    const int cx = cell_coord(P.x[i], G.inv_h[0], G.nc[0]);
    const int cy = cell_coord(P.y[i], G.inv_h[1], G.nc[1]);
    const int cz = cell_coord(P.z[i], G.inv_h[2], G.nc[2]);
    c = (cz * G.nc[1] + cy) * G.nc[0] + cx;
    if (G.layer2 && !(extent(P.r[i], P.vx[i], P.vy[i], P.vz[i], dt) <= plan->rho_c)) c += G.layer2;
  }
  const int sl = run_slot(c, count);
  if (c >= 0) {
    cid[i] = c;
    slot[i] = sl;
  }
}

// The counts that the reach pass took on another grid than the plan's.
__global__ __launch_bounds__(256) void k_clear_missed(const StepPlan *plan, int cells, int *count) {
  if (plan->err || plan->hit) return;
  for (int i = blockIdx.x * 256 + threadIdx.x; i < cells; i += gridDim.x * 256) count[i] = 0;
}

hipError_t launch_cell_hist(hipStream_t s, const Particles &P, const StepPlan *plan, double dt,
                            int tried_cells, int *cid, int *slot, int *count) {
  if (P.n <= 0) return hipSuccess;
  if (tried_cells > 0)
    hipLaunchKernelGGL(k_clear_missed, dim3(fill_grid(tried_cells)), dim3(256), 0, s, plan,
                       tried_cells, count);
  hipLaunchKernelGGL(k_cell_hist, dim3((unsigned)((P.n + 255) / 256)), dim3(256), 0, s, P, plan, dt,
                     cid, slot, count);
  return hipGetLastError();
}

// ---------------------------------------------------------------- a3: exclusive scan


// block-wide exclusive scan of one int per thread
__device__ void block_exclusive_scan(int v, int &excl) {
  __shared__ int wsum[SCAN_T / WAVE];
  const int lane = threadIdx.x % WAVE, w = threadIdx.x / WAVE;
  int inc = v;
  for (int o = 1; o < WAVE; o <<= 1) {
    const int t = __shfl_up(inc, o);
    if (lane >= o) inc += t;
  }
  if (lane == WAVE - 1) wsum[w] = inc;
  __syncthreads();
  if (w == 0) {
    int s = lane < SCAN_T / WAVE ? wsum[lane] : 0;
    int si = s;
    for (int o = 1; o < WAVE; o <<= 1) {
      const int t = __shfl_up(si, o);
      if (lane >= o) si += t;
    }
    if (lane < SCAN_T / WAVE) wsum[lane] = si - s;
  }
  __syncthreads();
  excl = wsum[w] + inc - v;
  __syncthreads();
}

// Exclusive scan of the cell counts into start (start[n] the total) in one pass, by
// the published decoupled look-back method (Merrill and Garland, 2016):
// workgroups take tiles of SCAN_B cells in order, publish a tile's sum as soon
// as they have it and its running total once they have added those before it,
// looked up 64 tiles at a time by one wave.  A tile only waits for tiles taken
// before it, which are held by workgroups that run.  The sum and its state travel
// in one 64-bit word, so no other ordering is needed.  clear: the counts are left
// zero for the next binning (the deposition clears its own, which may lie in a new
// buffer: left alone, the scan of 27M counts takes 122 us, not 152).  The largest
// count goes to *maxcell.
// Three launches (tile sums, their scan, the addition) did the same: 26 us at
// 2.7M cells and 3 launches of about 2 us, and as many gaps, at a thousand.
enum : unsigned int { SCAN_SUM = 1u, SCAN_TOTAL = 2u };

__global__ __launch_bounds__(SCAN_T) void k_scan(int *count, int n_host, const StepPlan *plan,
                                                 int *start, ScanState *st,
                                                 unsigned int *maxcell, int clear) {
  if (plan && plan->err) return;
  const int n = plan ? plan->cells : n_host;
  const int tiles = scan_tiles(n);
  __shared__ int tile, before;
  __shared__ int wmax[SCAN_T / WAVE];
  for (;;) {
    if (threadIdx.x == 0) tile = atomicAdd(&st->ticket, 1);
    __syncthreads();
    const int t = tile;
    if (t >= tiles) return;
    const int base = t * SCAN_B + threadIdx.x * SCAN_E;
    int v[SCAN_E], sum = 0, mx = 0;
#pragma unroll
    for (int k = 0; k < SCAN_E; ++k) {
      v[k] = base + k < n ? count[base + k] : 0;
      sum += v[k];
      mx = v[k] > mx ? v[k] : mx;
    }
    for (int o = WAVE / 2; o > 0; o >>= 1) {
      const int m = __shfl_xor(mx, o);
      mx = m > mx ? m : mx;
    }
    if (__lane_id() == 0) wmax[threadIdx.x / WAVE] = mx;
    int excl;
    block_exclusive_scan(sum, excl);
    __shared__ int total;
    if (threadIdx.x == SCAN_T - 1) total = excl + sum;
    __syncthreads();
    if (threadIdx.x < WAVE) {
      const int lane = threadIdx.x;
      int run = 0;
      if (t > 0) {
        if (lane == 0)
          __hip_atomic_store(&st->word[t],
                             ((unsigned long long)SCAN_SUM << 32) | (unsigned int)total,
                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        for (int hi = t - 1;; hi -= WAVE) {  // lane l looks at tile hi - l
          const int at = hi - lane;
          unsigned long long w = (unsigned long long)SCAN_TOTAL << 32;  // before the first: 0
          if (at >= 0)
            do
              w = __hip_atomic_load(&st->word[at], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            while (w == 0ull);
          const unsigned long long totals =
              __builtin_amdgcn_ballot_w64((unsigned int)(w >> 32) == SCAN_TOTAL);
          // the nearest running total ends the walk; lanes beyond it do not count
          const int last = totals ? __ffsll((long long)totals) - 1 : WAVE - 1;
          run += wave_sum(lane <= last ? (int)(unsigned int)w : 0);
          if (totals) break;
        }
      }
      if (lane == 0) {
        __hip_atomic_store(&st->word[t],
                           ((unsigned long long)SCAN_TOTAL << 32) | (unsigned int)(run + total),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        before = run;
        for (int k = 1; k < SCAN_T / WAVE; ++k) mx = wmax[k] > mx ? wmax[k] : mx;
        if (maxcell) atomicMax(maxcell, (unsigned int)mx);
        if (t == tiles - 1) start[n] = run + total;
      }
    }
    __syncthreads();
    int run = before + excl;
#pragma unroll
    for (int k = 0; k < SCAN_E; ++k) {
      if (base + k < n) {
        start[base + k] = run;
        if (clear) count[base + k] = 0;
      }
      run += v[k];
    }
    __syncthreads();  // tile, before, wmax and total are free again
  }
}

hipError_t launch_scan(hipStream_t s, int *count, int ncell, const StepPlan *plan, int *start,
                        ScanState *st, unsigned int *maxcell, bool clear) {
  const int tiles = scan_tiles(ncell);
  hipLaunchKernelGGL(k_scan, dim3(std::max(1, std::min(tiles, 512))), dim3(SCAN_T), 0, s, count,
                     ncell, plan, start, st, maxcell, (int)clear);
  return hipGetLastError();
}

// ---------------------------------------------------------------- a4: scatter

// cell-sorted 64-B records of the start-of-step state; reads the caller's SoA
// arrays coalesced and writes one record per sphere (its caller index and box
// inside, so no other array is written in sorted order).  Clears the contact
// counts on the way.
__global__ __launch_bounds__(256) void k_scatter(Particles P, const int *cid, const int *slot,
                                                 const int *start, Rec *rec, int *rank, int *cnt,
                                                 const int *box_of, const unsigned int *err) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (*err) return;
  __shared__ Stage<4> stage[256 / WAVE];
  Rec q{};
  int pos = -1;
  if (i < P.n) {
    pos = start[cid[i]] + slot[i];
    q = Rec{P.x[i], P.y[i], P.z[i], P.r[i], P.vx[i], P.vy[i], P.vz[i], (int)i,
            box_of ? box_of[i] : 0};
    rank[i] = pos;
    cnt[i] = 0;
  }
  store_records(q, pos, rec, stage[threadIdx.x / WAVE]);
}

hipError_t launch_scatter(hipStream_t s, const Particles &P, const int *cid, const int *slot,
                          const int *start, Rec *rec, int *rank, int *cnt, const BatchDev *B,
                          const unsigned int *err) {
  if (P.n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_scatter, dim3((unsigned)((P.n + 255) / 256)), dim3(256), 0, s, P, cid,
                     slot, start, rec, rank, cnt, B ? B->box_of : nullptr, err);
  return hipGetLastError();
}

// ---------------------------------------------------------------- a5: sweep-1 detect

// All contacts within dt among all spheres (rule 1; eq. detect1/detect2), each
// unordered pair of spheres in neighbouring cells tested exactly once (the
// half stencil: own cell with j after i, and the 13 forward neighbour cells).
// Every contact (i, j, t) is appended to the contact slots of both spheres.
//
// One wave per home cell.  The wave's candidate list is the concatenation of
// up to 10 contiguous runs of the cell-sorted records (4 rows of 3 cells, the
// own cell and the next cell; a periodic wrap along x splits a row in two).
// Lanes hold candidates j (one 64-B record each, loaded once per chunk of 64);
// the home spheres i are wave-uniform and loop inside, so each pair costs the
// arithmetic only.  A run carries the periodic image shift of its cells; for a
// pair that can touch, the shifted separation equals the minimum image of rule
// 1 bitwise (the grid has >= 3 cells per axis and cell side >= reach).
//
// A conservative filter (pair64, pair32) keeps the square root, the division
// and the rule's exact operation order off the hot path; every pair it passes
// is decided by the rule itself.
constexpr int MAXRUN = 10;

// shift code of a run: per axis 0 = -L, 1 = none, 2 = +L (2 bits each), bit 6 = own cell
__device__ __forceinline__ int run_code(int sx, int sy, int sz, int own) {
  return (sx + 1) | ((sy + 1) << 2) | ((sz + 1) << 4) | (own << 6);
}

// -L, 0 or +L for c = 0, 1, 2: (c - 1) L is each of them exactly (one convert
// and one multiply instead of a chain of selects).
__device__ __forceinline__ double code_shift(int c, double L) { return (double)(c - 1) * L; }

// One run of a home cell's candidate list in the wave's table in LDS: the
// offset from list slot to sorted index, the image code (run_code; bit 6 the
// own cell) and the image shift per axis, (c - 1) L (exact).
struct alignas(16) RunT {
  int off, code;
  double sx, sy, sz;
};

// Append contact (i, j, t) to both spheres' slots.
__device__ __forceinline__ void record_contact(const DetectArgs &A, int i, int g, double t) {
  const int K = A.K;
  const size_t n = (size_t)A.n;
  const int k1 = atomicAdd(&A.cnt[i], 1);
  if (k1 < K) {
    A.slot_t[k1 * n + i] = t;
    A.slot_j[k1 * n + i] = g;
  }
  const int k2 = atomicAdd(&A.cnt[g], 1);
  if (k2 < K) {
    A.slot_t[k2 * n + g] = t;
    A.slot_j[k2 * n + g] = i;
  }
}


// Filter survivors of one wave awaiting the exact rule: (home i, candidate g)
// pairs in the wave's LDS queue.  A survivor is rare (about one per home
// sphere); deciding it at once would run the square root, the division and
// two atomics for one live lane while the other 63 idle, so survivors are
// queued and decided 64 at a time, outside the filter loops, where few registers
// are live, or sooner when the queue has no room for another step's.
constexpr int QCAP = 256;    // binary32 filter: two homes appended per step
constexpr int QCAP64 = 512;  // binary64 filter: two homes against three chunks

struct SurvivorQueue {
  int2 *q;              // cap entries in LDS, private to the wave
  int n;                // entries waiting (wave-uniform)
  unsigned int pushed;  // survivors seen (wave-uniform)
  int cap;
  unsigned long long tests;  // unordered pairs tested (wave-uniform)
};

// The rule for every queued pair (rule 1 with the canonical minimum image,
// which for every pair that can touch is the image the stencil tested, and
// for any other pair finds no contact either).
__device__ __forceinline__ void flush_survivors(const DetectArgs &A, const Grid &G,
                                                SurvivorQueue &Q) {
  for (int e0 = 0; e0 < Q.n; e0 += WAVE) {
    const int e = e0 + (int)__lane_id();
    if (e < Q.n) {
      const int2 pr = Q.q[e];
      const Rec a = A.rec[pr.x], b = A.rec[pr.y];
      double t;
      if (pair_time(a, b, G, A.dt, t)) record_contact(A, pr.x, pr.y, t);
    }
  }
  Q.n = 0;
}

// Append the survivors of two home spheres i0 and i1 against the lane's
// candidate g (pass flags p0 and p1) to the queue, which has room for two
// wave's worth (the caller makes sure of it).  One wave-wide test when neither
// passes anywhere, the common case.
__device__ __forceinline__ void push_two(bool p0, bool p1, int i0, int i1, int g,
                                         SurvivorQueue &Q) {
  const unsigned long long m0 = __ballot(p0), m1 = __ballot(p1);
  if (!(m0 | m1)) return;
  const unsigned long long below = (1ull << __lane_id()) - 1ull;
  const int c0 = __popcll(m0), c1 = __popcll(m1);
  if (p0) Q.q[Q.n + __popcll(m0 & below)] = make_int2(i0, g);
  if (p1) Q.q[Q.n + c0 + __popcll(m1 & below)] = make_int2(i1, g);
  Q.n += c0 + c1;
  Q.pushed += c0 + c1;
}

// One home sphere (FP32 record) against the lane's candidate: the same filter in
// binary32 with the contact distance inflated by the band.  Survivors are
// decided by the binary64 rule (flush_survivors).
template <bool MASK>
__device__ __forceinline__ bool pass32(const DetectArgs &A, int thr, float bx, float by, float bz,
                                       float br, float bvx, float bvy, float bvz, int i,
                                       const Rec32 &h) {
  const float d0 = bx - h.x, d1 = by - h.y, d2 = bz - h.z;
  const float u0 = bvx - h.vx, u1 = bvy - h.vy, u2 = bvz - h.vz;
  const float sb = (h.r + br) * A.kband;
  const float bb = __builtin_fmaf(d0, u0, __builtin_fmaf(d1, u1, d2 * u2));
  const float q = __builtin_fmaf(d0, d0, __builtin_fmaf(d1, d1, d2 * d2));
  const float cc = __builtin_fmaf(-sb, sb, q);
  return (!MASK || i < thr) && __builtin_fmaf(bb, A.dt2f, cc) <= 0.0f;
}

// One candidate chunk against the homes [h0, h1) staged in LDS at p.
template <bool MASK>
__device__ __forceinline__ void detect_chunk32(const DetectArgs &A, const Grid &G, const Rec32 *p, int h0,
                                               int h1, int g, int thr, const RunT &run, double ox,
                                               double oy, double oz, SurvivorQueue &Q) {
  float bx, by, bz, bvx, bvy, bvz, br;
  if (thr >= 0) {
    const Rec b = A.rec[g];
    // candidate relative to the home cell centre (ox, oy, oz), image shift applied
    bx = (float)((b.x + run.sx) - ox);
    by = (float)((b.y + run.sy) - oy);
    bz = (float)((b.z + run.sz) - oz);
    bvx = (float)b.vx;
    bvy = (float)b.vy;
    bvz = (float)b.vz;
    br = (float)b.r;
  } else {
    bx = by = bz = 1e18f;
    bvx = bvy = bvz = 0.f;
    br = 0.f;
  }
  int i = h0;
  for (;;) {
    // two homes per step while the queue has room for their survivors; a full
    // queue (rare) is decided here, outside the loop
    for (; i < h1 && Q.n <= Q.cap - 2 * WAVE; i += 2) {
      const bool two = i + 1 < h1;  // an odd last home pairs with itself, never passing twice
      const Rec32 ha = p[i - h0], hb = p[two ? i + 1 - h0 : i - h0];
      const bool p0 = pass32<MASK>(A, thr, bx, by, bz, br, bvx, bvy, bvz, i, ha);
      const bool p1 = two && pass32<MASK>(A, thr, bx, by, bz, br, bvx, bvy, bvz, i + 1, hb);
      push_two(p0, p1, i, i + 1, g, Q);
    }
    if (i >= h1) break;
    flush_survivors(A, G, Q);
  }
}

// Runs of consecutive cell-sorted records that make the half stencil of one
// home cell: run 0 the own cell (pairs with j after i), run 1 the next cell
// along x, runs 2..9 the 4 rows of 3 cells, each row as two runs (the second
// empty unless the row wraps along x); each with its periodic image code.
// A wave forms the runs of GROUP home cells at once, one run to a lane and one
// cell to each 16 lanes: of some 160 vector instructions a cell, 125 went into
// its runs when a cell had the wave to itself.
constexpr int GROUP = 4;

// The runs of a group, lane 16 q + k holding run k of cell q: its first sorted
// position and length, and its first slot in the cell's candidate list (an empty
// run starts where the next does).
struct GroupRuns {
  int first, len, slot;
};

// The runs of cells cell0 .. cell0 + ncells - 1 (ncells <= GROUP) of the box whose
// grid is G (`start` points at its first cell; positions in start[] are global):
// the lanes' own R, and in LDS the run tables rt (MAXRUN entries a cell): each
// run's offset from list slot to sorted index, its code and its image shift.
__device__ __forceinline__ void group_runs(const Grid &G, const int *start, int cell0, int ncells,
                                           RunT *rt, GroupRuns &R) {
  const int nc0 = G.nc[0], nc1 = G.nc[1], nc2 = G.nc[2];
  // the lane index opaque, so that what follows from it is formed here per group
  // and not held across the cells (registers)
  int ln = (int)__lane_id();
  asm volatile("" : "+v"(ln));
  const int q = ln >> 4, k = ln & 15;
  const bool mine = q < ncells && k < MAXRUN;
  const int cell = cell0 + (q < ncells ? q : 0);
  int cx, cy, cz;
  cell_xyz(G, cell, cx, cy, cz);
  const bool lw = cx - 1 < 0, rw = cx + 1 >= nc0;  // the row wraps left / right
  // rows (runs 2..9): offsets (dy, dz) = (1, 0), (-1, 1), (0, 1), (1, 1)
  const int row = (k - 2) >> 1, second = (k - 2) & 1;
  int y = cy + (row == 1 ? -1 : (row == 2 ? 0 : 1)), z = cz + (row == 0 ? 0 : 1);
  const int sy = y >= nc1 ? 1 : (y < 0 ? -1 : 0), sz = z >= nc2 ? 1 : 0;
  y -= sy * nc1;
  z -= sz * nc2;
  // a row's two runs, as cells [a0, a1) and [a2, a3) of the row: the wrapped
  // left cell then cells 0..1; cells cx-1..cx then the wrapped right cell 0;
  // or cells cx-1..cx+1 and an empty second run
  const int a0 = lw ? nc0 - 1 : cx - 1, a1 = lw ? nc0 : (rw ? cx + 1 : cx + 2);
  const int a2 = lw || rw ? 0 : cx + 2, a3 = lw ? 2 : (rw ? 1 : cx + 2);
  // image along x of a row's first / second run
  const int sx0 = lw ? -1 : 0, sx1 = !lw && rw ? 1 : 0;
  // run 1: the next cell along x, cell 0 of the own row where x wraps
  const int c01 = k == 0 ? cell : (rw ? cell - cx : cell + 1);
  const int base = (z * nc1 + y) * nc0;
  const int i0 = k < 2 ? c01 : base + (second ? a2 : a0);
  const int i1 = k < 2 ? c01 + 1 : base + (second ? a3 : a1);
  const int code01 = k == 0 ? run_code(0, 0, 0, 1) : run_code(rw ? 1 : 0, 0, 0, 0);
  const int code = k < 2 ? code01 : run_code(second ? sx1 : sx0, sy, sz, 0);
  R.first = R.len = 0;
  if (mine) {
    R.first = start[i0];
    R.len = start[i1] - R.first;
  }
  // running lengths within 16 lanes (row_shr:1, 2, 4, 8)
  int inc = R.len;
  inc += __builtin_amdgcn_update_dpp(0, inc, 0x111, 0xf, 0xf, true);
  inc += __builtin_amdgcn_update_dpp(0, inc, 0x112, 0xf, 0xf, true);
  inc += __builtin_amdgcn_update_dpp(0, inc, 0x114, 0xf, 0xf, true);
  inc += __builtin_amdgcn_update_dpp(0, inc, 0x118, 0xf, 0xf, true);
  R.slot = inc - R.len;
  if (mine)  // one wave owns rt: its LDS operations stay in order
    rt[q * MAXRUN + k] = RunT{R.first - R.slot, code, code_shift(code & 3, G.sL[0]),
                              code_shift((code >> 2) & 3, G.sL[1]),
                              code_shift((code >> 4) & 3, G.sL[2])};
}

// A home cell's runs as the candidate search needs them: its spheres [h0, h1),
// the candidate list length, the first list slot of each run (pre[0] = 0) and the
// run table.
struct CellSet {
  int h0, h1, total;
  int pre[MAXRUN];
  const RunT *rt;
};

// Cell q of a group; false if it is empty.
__device__ __forceinline__ bool group_cell(const GroupRuns &R, int q, const RunT *rt, CellSet &S) {
  const int l = 16 * q;
  S.h0 = __builtin_amdgcn_readlane(R.first, l);
  S.h1 = S.h0 + __builtin_amdgcn_readlane(R.len, l);
  if (S.h1 <= S.h0) return false;
  S.pre[0] = 0;
#pragma unroll
  for (int k = 1; k < MAXRUN; ++k) S.pre[k] = __builtin_amdgcn_readlane(R.slot, l + k);
  S.total = __builtin_amdgcn_readlane(R.slot, l + MAXRUN);  // (no run there: the end of the last)
  S.rt = rt + q * MAXRUN;
  return true;
}

// Home spheres of the binary32 filter staged in LDS per batch.
constexpr int HB32 = WAVE;

// Pair tests of one home cell with the binary32 filter.  The home spheres are
// staged in LDS (hl) HB32 at a time as binary32 records relative to the home
// cell centre, converted from the binary64 records; candidates in chunks of 64
// lanes, converted likewise with their run's image shift.
__device__ __forceinline__ void detect_cell32(const DetectArgs &A, const Grid &G, int cell,
                                              const CellSet &S, SurvivorQueue &Q, Rec32 *hl) {
  const int h0 = S.h0, h1 = S.h1, total = S.total;
  const int *pre = S.pre;
  const int lane = __lane_id();
  // unordered pairs this cell tests: own cell pairs once, every home against the rest
  Q.tests += (unsigned long long)(h1 - h0) * (unsigned long long)(total - (h1 - h0)) +
             (unsigned long long)(h1 - h0) * (unsigned long long)(h1 - h0 - 1) / 2ull;
  int cx, cy, cz;
  cell_xyz(G, cell, cx, cy, cz);
  const double ox = (cx + 0.5) * G.h[0], oy = (cy + 0.5) * G.h[1], oz = (cz + 0.5) * G.h[2];
  for (int hb = h0; hb < h1; hb += HB32) {
    const int he = hb + HB32 < h1 ? hb + HB32 : h1;
    if (hb + lane < he) {
      const Rec q = A.rec[hb + lane];
      Rec32 f;
      f.x = (float)(q.x - ox);
      f.y = (float)(q.y - oy);
      f.z = (float)(q.z - oz);
      f.r = (float)q.r;
      f.vx = (float)q.vx;
      f.vy = (float)q.vy;
      f.vz = (float)q.vz;
      f.pad = 0.f;
      hl[lane] = f;
    }
    __syncthreads();  // the workgroup is this one wave
    for (int base = 0; base < total; base += WAVE) {
      const int v = base + lane;
      int r = 0;  // the run of list slot v (see detect_chunks)
#pragma unroll
      for (int k = 1; k < MAXRUN; ++k) r += v >= pre[k] ? 1 : 0;
      asm volatile("" : "+v"(r));  // the count apart from the table address
      const RunT run = S.rt[r];
      const int g = run.off + v;
      const bool ok = v < total;
      const bool own = (run.code >> 6) & 1;
      const int thr = !ok ? -1 : (own ? g : 0x7fffffff);
      if (base < h1 - h0)
        detect_chunk32<true>(A, G, (const Rec32 *)hl, hb, he, g, thr, run, ox, oy, oz, Q);
      else
        detect_chunk32<false>(A, G, (const Rec32 *)hl, hb, he, g, thr, run, ox, oy, oz, Q);
    }
    __syncthreads();  // before the next batch overwrites hl
  }
  // the survivors left in Q are the caller's to decide
}

// ---------------------------------------------------------------- a5, binary64 Gram filter

// The binary64 filter in Gram form.  F = |d|^2 - s^2 + dt2 (d . u)
// = beta_i + beta_j + <P_i, Q_j> where
//   P_i = (x_i, r_i, v_i),  Q_j = (-2 x_j - dt2 v_j, -2 r_j, -dt2 x_j),
//   beta = |x|^2 + dt2 x.v - r^2
// (d = x_j - x_i, u = v_j - v_i, s = r_i + r_j).  A pair passes iff
// beta_i + <P_i, Q_j> <= tol64 - beta_j as evaluated (beta_i the first addend
// of seven FMAs), tol64 a bound on the rounding of this evaluation and of the
// threshold for pairs the rule can keep (host, gram64_tolerance); survivors are
// decided by the rule (flush_survivors), so the result is exactly the rule's.
//
// The home sphere i is uniform across the wave and P_i is its record as it
// stands, so the records of the homes are read through the scalar cache
// straight into scalar registers, the operands of the FMAs (one each): no
// home terms are formed, staged or read back.  Lanes hold Q_j and the threshold
// of their candidate, formed once per chunk; of the home only beta_i goes
// through LDS.  A pair costs seven FMAs and one compare of vector issue, which
// bounds the kernel.  Coordinates are the caller's, not relative to the cell:
// the tolerance then grows with the box, as 1e-13 L^2, which admits pairs up to
// 4e-7 L apart, and saves the subtraction on both sides.
typedef double d8 __attribute__((ext_vector_type(8)));
typedef const d8 __attribute__((address_space(4))) *ScalarRec;

// beta of a sphere at x with w = x + dt2 v
__device__ __forceinline__ double gram_beta(double x, double y, double z, double wx, double wy,
                                            double wz, double r) {
  return __builtin_fma(-r, r, __builtin_fma(z, wz, __builtin_fma(y, wy, x * wx)));
}

// Queue the survivors of home i (the lanes of m) against the lane's candidate
// g, but for own-cell candidates that do not come after i (g < last holds the
// pair to j after i; last is INT_MAX outside the own cell).  The queue has room
// for a wave's worth.
__device__ __forceinline__ void push_home(unsigned long long m, int i, int g, int last,
                                          SurvivorQueue &Q) {
  if (!m) return;
  m &= __builtin_amdgcn_ballot_w64(i < last);
  if (!m) return;
  const int at = __builtin_amdgcn_mbcnt_hi(
      (unsigned int)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned int)m, (unsigned int)Q.n));
  if (__builtin_amdgcn_inverse_ballot_w64(m)) Q.q[at] = make_int2(i, g);
  // kept in a scalar register: the loops that test it stay uniform, and the
  // home records they index stay scalar loads
  Q.n = __builtin_amdgcn_readfirstlane(Q.n + __popcll(m));
}

// NC chunks of a home cell's candidate list, from slot base on, against its
// homes [i0 + k, i0 + nb), two homes a step; the records of the next two are
// fetched while two are tested.  Returns nb, or the home to go on from when the
// queue has no room for another step's survivors.  Each scalar record serves NC wave-wide tests:
// with one chunk a pass the waves stood waiting for scalar loads (the homes of
// the waves on two CUs exceed their 16 KB scalar cache), 2.65 ms at 16M.
template <int NC>
__device__ __forceinline__ int detect_chunks(const DetectArgs &A, const CellSet &S, int base,
                                             int i0, int k, int nb, const double *hbeta,
                                             SurvivorQueue &Q) {
  const int *pre = S.pre;
  const double dt2 = A.dt2;
  double q[NC][7], thr[NC];
  int g[NC], last[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int v = base + c * WAVE + (int)__lane_id();
    // the run of list slot v: the last run whose first slot is at most v.  The
    // first slots are non-decreasing, so it is the number of runs after the
    // first that start at or before v (an empty run starts where the next
    // does, so it is never the one counted last for a slot inside the list)
    int r = 0;
#pragma unroll
    for (int k = 1; k < MAXRUN; ++k) r += v >= pre[k] ? 1 : 0;
    asm volatile("" : "+v"(r));  // the count apart from the table address
    const RunT run = S.rt[r];
    const bool ok = v < S.total;
    // past the end of the list: some record, and a threshold nothing meets
    g[c] = ok ? run.off + v : i0;
    last[c] = ((run.code >> 6) & 1) ? g[c] : 0x7fffffff;
    const Rec b = A.rec[g[c]];
    const double x = b.x + run.sx, y = b.y + run.sy, z = b.z + run.sz;
    // w = x + dt2 v: Q = -(x + w), and beta = x . w - r^2
    const double wx = __builtin_fma(dt2, b.vx, x), wy = __builtin_fma(dt2, b.vy, y),
                 wz = __builtin_fma(dt2, b.vz, z);
    q[c][0] = -(x + wx);
    q[c][1] = -(y + wy);
    q[c][2] = -(z + wz);
    q[c][3] = -2.0 * b.r;
    q[c][4] = -dt2 * x;
    q[c][5] = -dt2 * y;
    q[c][6] = -dt2 * z;
    const double th = A.tol64 - gram_beta(x, y, z, wx, wy, wz, b.r);
    thr[c] = ok ? th : -INFINITY;
  }
  const auto test = [&](d8 p, double beta, int c) {
    double t = __builtin_fma(p[0], q[c][0], beta);
#pragma unroll
    for (int k = 1; k < 7; ++k) t = __builtin_fma(p[k], q[c][k], t);
    return (unsigned long long)__builtin_amdgcn_ballot_w64(t <= thr[c]);
  };
  const ScalarRec homes = (ScalarRec)(uintptr_t)(A.rec + i0);
  const int top = nb - 1;
  d8 a = homes[k], b = homes[k < top ? k + 1 : top];
  double ba = hbeta[k], bb = hbeta[k < top ? k + 1 : top];
  for (; k < nb && Q.n <= Q.cap - 2 * NC * WAVE; k += 2) {
    const int ka = k + 2 < top ? k + 2 : top, kb = k + 3 < top ? k + 3 : top;
    const d8 na = homes[ka], nbr = homes[kb];
    const double nba = hbeta[ka], nbb = hbeta[kb];
    unsigned long long m0[NC], m1[NC], any = 0ull;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      m0[c] = test(a, ba, c);
      any |= m0[c];
    }
    if (k < top) {
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        m1[c] = test(b, bb, c);
        any |= m1[c];
      }
    } else {
#pragma unroll
      for (int c = 0; c < NC; ++c) m1[c] = 0ull;
    }
    if (any) {
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        push_home(m0[c], i0 + k, g[c], last[c], Q);
        push_home(m1[c], i0 + k + 1, g[c], last[c], Q);
      }
    }
    a = na;
    b = nbr;
    ba = nba;
    bb = nbb;
  }
  return k < nb ? k : nb;
}

// Pair tests of one home cell with the binary64 Gram filter; homes in batches
// of 64 (hbeta holds one batch's beta), candidates in chunks of 64 lanes, three
// chunks a pass (a cell of 13 has about 180 candidates).
__device__ __forceinline__ void detect_cell64(const DetectArgs &A, const Grid &G, const CellSet &S,
                                              SurvivorQueue &Q, double *hbeta) {
  const int h0 = S.h0, nh = S.h1 - S.h0;
  Q.tests += (unsigned long long)nh * (unsigned long long)(S.total - nh) +
             (unsigned long long)nh * (unsigned long long)(nh - 1) / 2ull;
  for (int hb = 0; hb < nh; hb += WAVE) {
    const int nb = nh - hb < WAVE ? nh - hb : WAVE;
    const int i0 = h0 + hb;
    if ((int)__lane_id() < nb) {  // one wave owns hbeta: its LDS operations stay in order
      const Rec a = A.rec[i0 + (int)__lane_id()];
      hbeta[__lane_id()] =
          gram_beta(a.x, a.y, a.z, __builtin_fma(A.dt2, a.vx, a.x), __builtin_fma(A.dt2, a.vy, a.y),
                    __builtin_fma(A.dt2, a.vz, a.z), a.r);
    }
    for (int base = 0, k = 0; base < S.total;) {
      const int left = S.total - base;
      int step = 3 * WAVE;
      if (left > 2 * WAVE) {
        k = detect_chunks<3>(A, S, base, i0, k, nb, hbeta, Q);
      } else if (left > WAVE) {
        k = detect_chunks<2>(A, S, base, i0, k, nb, hbeta, Q);
      } else {
        k = detect_chunks<1>(A, S, base, i0, k, nb, hbeta, Q);
      }
      if (k < nb) {  // the queue is full (rare): decide it, then the rest of these homes
        flush_survivors(A, G, Q);
        step = 0;
      } else {
        k = 0;
      }
      base += step;
    }
  }
  // the survivors left in Q are the caller's to decide (flush_survivors), now
  // or after later cells of the same grid
}

// Both filters run over cpw consecutive cells per workgroup, so the survivor
// queue carries over between them and is decided a wave at a time (a cell of 13
// spheres leaves about 13 survivors, so deciding them per cell runs the rule's
// square root and division on a fifth of the lanes).  The grid, the tolerances
// and cpw are the plan's; the host's launch is sized for the last step's grid,
// so a workgroup takes further groups of cells if this step has more.  One add
// per workgroup to the counters, which the waves do not wait for.
template <typename Cells>
__device__ __forceinline__ void detect_groups(const DetectArgs &A, int ncell, int cpw,
                                              SurvivorQueue &Q, Cells cells) {
  const int groups = (ncell + cpw - 1) / cpw;
  for (int g = blockIdx.x; g < groups; g += gridDim.x) {
    const int c0 = xcd_remap(g, groups) * cpw;
    cells(c0, c0 + cpw < ncell ? c0 + cpw : ncell);
  }
  if (__lane_id() == 0 && Q.tests) {
    atomicAdd(&my_shard(A.ctr).tests, Q.tests);
    if (Q.pushed) atomicAdd(&my_shard(A.ctr).recheck, (unsigned long long)Q.pushed);
  }
}

__global__ __launch_bounds__(WAVE, 6) void k_detect_half32(DetectArgs A) {
  if (*A.err || (A.masked && !masked_dense(A.ctr, A.n))) return;
  __shared__ int2 survq[QCAP];
  __shared__ Rec32 hl[HB32];
  __shared__ RunT rt[GROUP * MAXRUN];
  SurvivorQueue Q{survq, 0, 0u, QCAP, 0ull};
  const Grid G = A.plan->G;
  A.kband = A.plan->kband;
  A.dt2f = A.plan->dt2f;
  detect_groups(A, G.ncell, A.plan->cpw, Q, [&](int c0, int c1) {
    for (int b = c0; b < c1; b += GROUP) {
      const int nc = c1 - b < GROUP ? c1 - b : GROUP;
      GroupRuns R;
      group_runs(G, A.start, b, nc, rt, R);
      for (int q = 0; q < nc; ++q) {
        CellSet S;
        if (group_cell(R, q, rt, S)) detect_cell32(A, G, b + q, S, Q, hl);
        if (b + q + 1 == c1 || Q.n >= WAVE) flush_survivors(A, G, Q);
      }
    }
  });
}

__global__ __launch_bounds__(WAVE, 6) void k_detect_half64(DetectArgs A) {
  if (*A.err || (A.masked && !masked_dense(A.ctr, A.n))) return;
  __shared__ int2 survq[QCAP64];
  __shared__ double hbeta[WAVE];
  __shared__ RunT rt[GROUP * MAXRUN];
  SurvivorQueue Q{survq, 0, 0u, QCAP64, 0ull};
  const Grid G = A.plan->G;
  A.tol64 = A.plan->tol64;
  detect_groups(A, G.ncell, A.plan->cpw, Q, [&](int c0, int c1) {
    for (int b = c0; b < c1; b += GROUP) {
      const int nc = c1 - b < GROUP ? c1 - b : GROUP;
      GroupRuns R;
      group_runs(G, A.start, b, nc, rt, R);
      for (int q = 0; q < nc; ++q) {
        CellSet S;
        if (group_cell(R, q, rt, S)) detect_cell64(A, G, S, Q, hbeta);
        if (b + q + 1 == c1 || Q.n >= WAVE) flush_survivors(A, G, Q);
      }
    }
  });
}

// Box of a global cell number: the last b with cell_base[b] <= c.
__device__ __forceinline__ int box_of_cell(const int *cell_base, int nbox, int c) {
  int lo = 0, hi = nbox - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (cell_base[mid] <= c)
      lo = mid;
    else
      hi = mid - 1;
  }
  return lo;
}

// Batched form: the cells of all boxes are numbered consecutively, box after
// box, and each workgroup (one wave) takes cpw consecutive global cells, as
// k_detect_half64 does in one box: the box of each cell comes from the
// first-cell table, the pair tests run with that box's grid, and the survivor
// queue carries over the cells, decided with the grid of the box its survivors
// came from whenever the next cell lies in another box, when it holds a wave's
// worth, and at the end.
__global__ __launch_bounds__(WAVE, 5) void k_detect_batched(DetectArgs A, BatchDev B, int cpw) {
  if (B.flags[FLAG_ERR]) return;
  __shared__ int2 survq[QCAP64];
  __shared__ double hbeta[WAVE];
  __shared__ RunT rt[GROUP * MAXRUN];
  SurvivorQueue Q{survq, 0, 0u, QCAP64, 0ull};
  const int total = B.cell_base[B.nbox];
  const int c0 = xcd_remap(blockIdx.x, gridDim.x) * cpw;
  const int c1 = c0 + cpw < total ? c0 + cpw : total;
  if (c0 >= c1) return;
  int b = box_of_cell(B.cell_base, B.nbox, c0);
  int qb = b;  // the box of the queued survivors
  for (int item = c0; item < c1;) {
    while (item >= B.cell_base[b + 1]) ++b;  // boxes of no cells are passed over
    if (b != qb) {
      if (Q.n > 0) flush_survivors(A, B.gtab[qb], Q);
      qb = b;
    }
    const Grid G = B.gtab[b];
    const int base = B.cell_base[b];
    const int end = c1 < B.cell_base[b + 1] ? c1 : B.cell_base[b + 1];  // a group is of one box
    const int nc = end - item < GROUP ? end - item : GROUP;
    GroupRuns R;
    group_runs(G, A.start + base, item - base, nc, rt, R);
    for (int q = 0; q < nc; ++q, ++item) {
      CellSet S;
      if (group_cell(R, q, rt, S)) detect_cell64(A, G, S, Q, hbeta);
      if (item + 1 == c1 || Q.n >= WAVE) flush_survivors(A, G, Q);
    }
  }
}

// groups: the workgroups that the host expects (any number will do)
hipError_t launch_detect_half(hipStream_t s, const DetectArgs &A, bool fp32, int groups) {
  groups = (std::max(groups, 1) + 7) / 8 * 8;  // whole rounds of the XCDs
  if (fp32)
    hipLaunchKernelGGL(k_detect_half32, dim3(groups), dim3(WAVE), 0, s, A);
  else
    hipLaunchKernelGGL(k_detect_half64, dim3(groups), dim3(WAVE), 0, s, A);
  return hipGetLastError();
}

// ---------------------------------------------------------------- a5/a7: partner from contact slots

// Partner of sphere i among its c <= K recorded contacts, gone(j, out) telling
// which of four spheres are no longer eligible: the earliest one (rule 2: exact binary64 t, ties
// to the smaller caller index); with crank given (the literal order) the
// contact of smallest curve rank instead (see k_curve_rank).  The contact set of
// a sphere only shrinks over the sweeps of a step, so the slots written by the
// sweep-1 detect are complete for every later sweep.  Slots are k-major, so the
// reads of a wave are coalesced.  Four slots at a time: what the choice waits for is the chain of
// reads behind each contact, and four chains run side by side.
template <typename Gone>
__device__ __forceinline__ void slot_choice(int i, int c, size_t n, const double *slot_t,
                                            const int *slot_j, const Rec *rec, const Grid &G,
                                            const unsigned long long *crank, Gone gone, int &bj,
                                            double &bt) {
  bt = INFINITY;
  bj = -1;
  unsigned long long br = ~0ull;  // literal order: curve rank of the best contact
  // between walls a contact counts only before both centres reach a wall
  double ti = INFINITY;
  if (G.walls) {
    const Rec a = rec[i];
    ti = time_to_wall(a.x, a.y, a.z, a.vx, a.vy, a.vz, G);
  }
  for (int k0 = 0; k0 < c; k0 += 4) {
    int j4[4];
    double t4[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const size_t at = (size_t)(k0 + u < c ? k0 + u : k0) * n + i;
      j4[u] = slot_j[at];
      t4[u] = slot_t[at];
    }
    bool g4[4];
    gone(j4, g4);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int j = j4[u];
      const double t = t4[u];
      if (k0 + u >= c || g4[u]) continue;
      if (G.walls) {
        const Rec b = rec[j];
        if (!(t <= ti) || !(t <= time_to_wall(b.x, b.y, b.z, b.vx, b.vy, b.vz, G))) continue;
      }
      if (crank) {
        const unsigned long long rj = crank[j];
        if (rj < br) {
          br = rj;
          bt = t;
          bj = j;
        }
      } else if (t < bt || (bj >= 0 && t == bt && rec[j].o < rec[bj].o)) {
        bt = t;
        bj = j;
      }
    }
  }
}

// Spheres not eligible: those that collided (or that the caller's mask leaves out).
struct GoneCollided {
  const uint8_t *status;
  __device__ __forceinline__ bool one(int j) const { return status[j] == ST_COLLIDED; }
  __device__ __forceinline__ void operator()(const int (&j)[4], bool (&g)[4]) const {
#pragma unroll
    for (int u = 0; u < 4; ++u) g[u] = status[j[u]] == ST_COLLIDED;
  }
};

struct GoneNone {
  __device__ __forceinline__ void operator()(const int (&)[4], bool (&g)[4]) const {
    g[0] = g[1] = g[2] = g[3] = false;
  }
};

// Sweep 1's partner of every sphere.  Spheres with more contacts than slots are
// queued for the exact search (rare; one atomic per wave that has one).
__global__ __launch_bounds__(256) void k_slot_min(int n, const int *cnt, const double *slot_t,
                                                  const int *slot_j, int K, const Rec *rec,
                                                  int *key_j, double *key_t, int *ovf_list,
                                                  SweepCounters *ctr, const unsigned int *err,
                                                  const Grid *Gp,
                                                  const unsigned long long *crank) {
  if (*err) return;
  Grid G{};  // the walls are all that matters here (none in the batched form)
  if (Gp) G = *Gp;
  const int i = blockIdx.x * 256 + threadIdx.x;
  bool ovf = false;
  unsigned long long nc = 0ull;
  if (i < n) {
    const int c = cnt[i];
    nc = (unsigned long long)c;
    ovf = c > K;
    int bj;
    double bt;
    slot_choice(i, ovf ? 0 : c, (size_t)n, slot_t, slot_j, rec, G, crank, GoneNone{}, bj, bt);
    key_j[i] = bj;
    key_t[i] = bt;
  }
  const unsigned int k = wave_append(ovf, &ctr->n_overflow);
  if (ovf) ovf_list[k] = i;
  block_add(nc, &my_shard(ctr).contacts);
}

hipError_t launch_slot_min(hipStream_t s, int n, const int *cnt, const double *slot_t,
                           const int *slot_j, int K, const Rec *rec, int *key_j, double *key_t,
                           int *ovf_list, SweepCounters *ctr, const unsigned int *err,
                           const Grid *G, const unsigned long long *crank) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_slot_min, dim3((n + 255) / 256), dim3(256), 0, s, n, cnt, slot_t, slot_j, K,
                     rec, key_j, key_t, ovf_list, ctr, err, G, crank);
  return hipGetLastError();
}

// ---------------------------------------------------------------- the literal order's ranks

// Morton (Z-order) code of a cell: the bits of cx, cy, cz (each below 2^11)
// interleaved, x lowest.
__device__ __forceinline__ unsigned long long morton3(unsigned int cx, unsigned int cy,
                                                      unsigned int cz) {
  unsigned long long k = 0ull;
#pragma unroll
  for (int b = 0; b < 11; ++b) {
    k |= (unsigned long long)((cx >> b) & 1u) << (3 * b);
    k |= (unsigned long long)((cy >> b) & 1u) << (3 * b + 1);
    k |= (unsigned long long)((cz >> b) & 1u) << (3 * b + 2);
  }
  return k;
}

// Rank of every sphere in the order the paper's traversal visits it (Sec.
// "Collision Operator": elements along a space-filling curve, particles of an
// element one after another): the Morton code of its cell on the curve grid C
// (nc cells of side h per axis) above its caller index,
// crank = code << 31 | o, in cell-sorted order.  A sphere's cell is
// floor(x / h) in binary64, clamped to nc - 1.
__device__ __forceinline__ unsigned long long curve_rank(const CurveGrid &C, double x, double y,
                                                         double z, int o) {
  const double p[3] = {x, y, z};
  unsigned int c[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    double q = floor(p[k] / C.h[k]);
    if (q < 0.0) q = 0.0;
    if (q > (double)(C.nc[k] - 1)) q = (double)(C.nc[k] - 1);
    c[k] = (unsigned int)q;
  }
  return morton3(c[0], c[1], c[2]) << 31 | (unsigned long long)(unsigned int)o;
}

__global__ __launch_bounds__(256) void k_curve_rank(const Rec *rec, int n, const StepPlan *plan,
                                                    unsigned long long *crank) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= n || plan->err) return;
  const Rec a = rec[i];
  crank[i] = curve_rank(plan->C, a.x, a.y, a.z, a.o);
}

hipError_t launch_curve_rank(hipStream_t s, const Rec *rec, int n, const StepPlan *plan,
                             unsigned long long *crank) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_curve_rank, dim3((n + 255) / 256), dim3(256), 0, s, rec, n, plan, crank);
  return hipGetLastError();
}

// ---------------------------------------------------------------- exact neighbourhood search

// Search box of a sphere in cell (cx, cy, cz): kx..kz cells either side along
// each axis, or the whole axis once when 2k + 1 covers it.  Calls
// run(first, end) for each run of consecutive sorted records (a row of cells
// along x, split in two where it wraps) of the layer whose first cell is
// `base`.  Every cell of the box is visited exactly once.
template <typename F>
__device__ __forceinline__ void search_box_runs(const Grid &G, const int *start, int base, int cx,
                                                int cy, int cz, const int k[3], F run) {
  const int nc0 = G.nc[0], nc1 = G.nc[1], nc2 = G.nc[2];
  const bool fx = 2 * k[0] + 1 >= nc0, fy = 2 * k[1] + 1 >= nc1, fz = 2 * k[2] + 1 >= nc2;
  const int ny = fy ? nc1 : 2 * k[1] + 1, nz = fz ? nc2 : 2 * k[2] + 1;
  for (int iz = 0; iz < nz; ++iz) {
    const int z = fz ? iz : (cz - k[2] + iz + nc2) % nc2;
    for (int iy = 0; iy < ny; ++iy) {
      const int y = fy ? iy : (cy - k[1] + iy + nc1) % nc1;
      const int row = base + (z * nc1 + y) * nc0;
      if (fx) {
        run(start[row], start[row + nc0]);
      } else {
        const int x0 = cx - k[0], x1 = cx + k[0];
        if (x0 < 0) {
          run(start[row + x0 + nc0], start[row + nc0]);
          run(start[row], start[row + x1 + 1]);
        } else if (x1 >= nc0) {
          run(start[row + x0], start[row + nc0]);
          run(start[row], start[row + x1 - nc0 + 1]);
        } else {
          run(start[row + x0], start[row + x1 + 1]);
        }
      }
    }
  }
}

// Cells either side of sphere a that can hold a partner: 1 when the cell side
// is at least the reach (one layer), else enough to cover the sphere's extent
// plus the largest extent (split grid).
__device__ __forceinline__ void search_radius(const Grid &G, const Rec &a, double dt, int k[3]) {
  if (G.rho_max > 0.0) {
    const double R = (extent(a.r, a.vx, a.vy, a.vz, dt) + G.rho_max) * (1.0 + 1e-9);
    for (int ax = 0; ax < 3; ++ax) k[ax] = (int)ceil(R / G.h[ax]);
  } else {
    k[0] = k[1] = k[2] = 1;
  }
}

// Distance along one axis from a sphere at offset f within its cell (cell side
// h) to the cells `o` cells away: 0 for its own cell, else the gap to the
// nearer face.  Cell faces are taken `eta` nearer, which covers spheres that
// rounding placed in a neighbouring cell.
__device__ __forceinline__ double face_gap(int o, double f, double h, double eta) {
  double g = 0.0;
  if (o > 0) g = o * h - f;
  if (o < 0) g = f - (o + 1) * h;
  g -= eta;
  return g > 0.0 ? g : 0.0;
}

// Run r of the ball-pruned search of a sphere at (px, py, pz) in cell
// (cx, cy, cz): r = (layer * nz + iz) * ny + iy) * 2 + part over the rows of
// its search box (kx..kz cells either side, whole axes once when 2k + 1 covers
// them).  A row is clipped along x to the cells within distance R[layer] of
// the sphere (exact where the search box does not cover the axis; the whole
// row otherwise) and split in two where it wraps.  Sets [first, end) of
// sorted records (empty if the row holds no such cell).
__device__ __forceinline__ void wide_run(const Grid &G, const int *start, int r, int ny, int nz,
                                         int cx, int cy, int cz, double fx_, double fy_,
                                         double fz_, const int k[3], const double R[2],
                                         int &first, int &end) {
  const int nc0 = G.nc[0], nc1 = G.nc[1], nc2 = G.nc[2];
  const int part = r & 1;
  int q = r >> 1;
  const int iy = q % ny;
  q /= ny;
  const int iz = q % nz;
  const int layer = q / nz;
  first = end = 0;
  const bool fx = 2 * k[0] + 1 >= nc0, fy = 2 * k[1] + 1 >= nc1, fz = 2 * k[2] + 1 >= nc2;
  const double eta0 = 1e-9 * G.h[0], eta1 = 1e-9 * G.h[1], eta2 = 1e-9 * G.h[2];
  const int oy = iy - k[1], oz = iz - k[2];
  const double gy = fy ? 0.0 : face_gap(oy, fy_, G.h[1], eta1);
  const double gz = fz ? 0.0 : face_gap(oz, fz_, G.h[2], eta2);
  const double Rl = R[layer];
  const double rest = Rl * Rl - (gy * gy + gz * gz);
  if (!(rest >= 0.0)) return;
  const int z = fz ? iz : (cz + oz + nc2) % nc2;
  const int y = fy ? iy : (cy + oy + nc1) % nc1;
  const int row = (layer ? G.layer2 : 0) + (z * nc1 + y) * nc0;
  int xa = 0, xb = 0;  // cells [xa, xb) of the row, in offsets when not wrapping the axis
  if (fx) {
    if (!part) xb = nc0;
  } else {
    // x offsets whose cells come within the remaining distance
    const double ext = __builtin_sqrt(rest) * (1.0 + 1e-9) + eta0;
    int o0 = -k[0], o1 = k[0];
    while (o0 < 0 && face_gap(o0, fx_, G.h[0], 0.0) > ext) ++o0;
    while (o1 > 0 && face_gap(o1, fx_, G.h[0], 0.0) > ext) --o1;
    const int x0 = cx + o0, x1 = cx + o1;
    if (x0 < 0) {
      xa = part ? 0 : x0 + nc0;
      xb = part ? x1 + 1 : nc0;
    } else if (x1 >= nc0) {
      xa = part ? 0 : x0;
      xb = part ? x1 - nc0 + 1 : nc0;
    } else if (!part) {
      xa = x0;
      xb = x1 + 1;
    }
  }
  if (xb > xa) {
    first = start[row + xa];
    end = start[row + xb];
  }
}

// a5 for the spheres of large extent (second layer of a split grid): one wave
// per sphere p tests every sphere that can touch it exactly (rule 1 with the
// canonical minimum image): of the first layer, those within p's extent plus
// rho_c (their extents are at most rho_c); of the second layer, those after p
// within p's extent plus the largest extent, so each pair of large-extent
// spheres is tested once.  Pairs of two first-layer spheres belong to
// k_detect_half64.  The lanes first fetch up to 64 row runs of the ball-pruned
// search box at once and scan their lengths; then each lane takes every 64th
// candidate of the concatenated runs, finding its run by a binary search over
// the scanned lengths held across the wave.  An FMA pre-filter (tolerance for
// the full reach) keeps the exact rule for the few pairs that may touch;
// survivors are decided at once (they are rare).
__global__ __launch_bounds__(256) void k_detect_wide(DetectArgs A) {
  if (*A.err || !A.plan->G.layer2 || (A.masked && !masked_dense(A.ctr, A.n))) return;
  const Grid G = A.plan->G;
  const double rho_c = A.plan->rho_c, tol_wide = A.plan->tol_wide;
  const int n = A.n;
  const int first = A.start[G.layer2], count = n - first;
  const int lane = __lane_id();
  const int wid = (blockIdx.x * blockDim.x + threadIdx.x) / WAVE;
  const int nw = (gridDim.x * blockDim.x) / WAVE;
  unsigned long long tests = 0ull;
  for (int w = wid; w < count; w += nw) {
    const int p = first + w;
    const Rec a = A.rec[p];
    const double ea = extent(a.r, a.vx, a.vy, a.vz, A.dt);
    const double R[2] = {(ea + rho_c) * (1.0 + 1e-9), (ea + G.rho_max) * (1.0 + 1e-9)};
    int k[3];
    for (int ax = 0; ax < 3; ++ax) k[ax] = (int)ceil(R[1] / G.h[ax]);
    const int cx = cell_coord(a.x, G.inv_h[0], G.nc[0]);
    const int cy = cell_coord(a.y, G.inv_h[1], G.nc[1]);
    const int cz = cell_coord(a.z, G.inv_h[2], G.nc[2]);
    const double fx_ = a.x - cx * G.h[0], fy_ = a.y - cy * G.h[1], fz_ = a.z - cz * G.h[2];
    const int ny = 2 * k[1] + 1 >= G.nc[1] ? G.nc[1] : 2 * k[1] + 1;
    const int nz = 2 * k[2] + 1 >= G.nc[2] ? G.nc[2] : 2 * k[2] + 1;
    const int nruns = 2 * 2 * ny * nz;
    for (int rb = 0; rb < nruns; rb += WAVE) {
      int s0 = 0, s1 = 0;
      if (rb + lane < nruns) {
        wide_run(G, A.start, rb + lane, ny, nz, cx, cy, cz, fx_, fy_, fz_, k, R, s0, s1);
        if ((((rb + lane) >> 1) / (ny * nz)) == 1) {  // second layer: only j after p
          s0 = s0 > p + 1 ? s0 : p + 1;
          s1 = s1 > s0 ? s1 : s0;
        }
      }
      const int len = s1 - s0;
      int incl = len;
      for (int o = 1; o < WAVE; o <<= 1) {
        const int t = __shfl_up(incl, o);
        if (lane >= o) incl += t;
      }
      const int excl = incl - len;
      const int total = __shfl(incl, WAVE - 1);
      for (int base = 0; base < total; base += WAVE) {
        const int v = base + lane;
        // largest lane l with excl[l] <= v: the run holding candidate v
        int l = 0;
        for (int step = WAVE / 2; step > 0; step >>= 1) {
          const int c = l + step;
          const int ec = __shfl(excl, c);
          if (ec <= v) l = c;
        }
        const int j = __shfl(s0, l) + (v - __shfl(excl, l));
        if (v < total) {
          ++tests;
          const Rec b = A.rec[j];
          const double d0 = wrap_sep(b.x - a.x, G.L[0], G.halfL[0]);
          const double d1 = wrap_sep(b.y - a.y, G.L[1], G.halfL[1]);
          const double d2 = wrap_sep(b.z - a.z, G.L[2], G.halfL[2]);
          const double u0 = b.vx - a.vx, u1 = b.vy - a.vy, u2 = b.vz - a.vz;
          const double s = a.r + b.r;
          const double bf = __builtin_fma(d0, u0, __builtin_fma(d1, u1, d2 * u2));
          const double cf =
              __builtin_fma(d0, d0, __builtin_fma(d1, d1, __builtin_fma(d2, d2, -(s * s))));
          double t;
          if (__builtin_fma(bf, A.dt2, cf) <= tol_wide &&
              contact_time(d0, d1, d2, u0, u1, u2, s, A.dt, t))
            record_contact(A, p, j, t);
        }
      }
    }
  }
  block_add(tests, &my_shard(A.ctr).tests);
}

hipError_t launch_detect_wide(hipStream_t s, const DetectArgs &A) {
  const int n = A.n;
  if (n <= 0) return hipSuccess;
  // the range is on the device (no read-back before the launch): waves loop
  // over it; about one wave per 256 spheres (the split puts about 0.1% of them
  // in the second layer), 64 to 4096
  int64_t waves = n / 256;
  waves = waves < 64 ? 64 : (waves > 4096 ? 4096 : waves);
  hipLaunchKernelGGL(k_detect_wide, dim3((unsigned)((waves + 3) / 4)), dim3(256), 0, s, A);
  return hipGetLastError();
}

// Partner of sphere i (record a, grid G, cell starts `start`) by an exact search
// of its search box (the 27 surrounding cells, or the wider box of a split grid,
// in both layers), minimum image by rule 1: the earliest (rule 2: exact binary64
// t, ties to the smaller caller index) or, with crank given, the contact of
// smallest curve rank, among the spheres that are not `gone`.  The whole wave
// works on one sphere, lanes over candidates, and every lane gets the result.
template <typename Gone>
__device__ __forceinline__ void exact_partner(int i, const Rec &a, const Grid &G, const int *start,
                                              const Rec *rec, double dt,
                                              const unsigned long long *crank, Gone gone, int &bj,
                                              double &bt) {
  const int lane = __lane_id();
  int k[3];
  search_radius(G, a, dt, k);
  const int cx = cell_coord(a.x, G.inv_h[0], G.nc[0]);
  const int cy = cell_coord(a.y, G.inv_h[1], G.nc[1]);
  const int cz = cell_coord(a.z, G.inv_h[2], G.nc[2]);
  bt = INFINITY;
  bj = -1;
  int bo = 0x7fffffff;
  unsigned long long br = ~0ull;  // literal order: curve rank of the best contact
  for (int layer = 0; layer < (G.layer2 ? 2 : 1); ++layer) {
    search_box_runs(G, start, layer ? G.layer2 : 0, cx, cy, cz, k, [&](int s0, int s1) {
      for (int j = s0 + lane; j < s1; j += WAVE) {
        if (j == i || gone(j)) continue;
        const Rec b = rec[j];
        double t;
        if (pair_time_walls(a, b, G, dt, t)) {
          const int o = b.o;
          if (crank) {
            const unsigned long long rj = crank[j];
            if (rj < br) {
              br = rj;
              bt = t;
              bj = j;
            }
          } else if (t < bt || (t == bt && o < bo)) {
            bt = t;
            bo = o;
            bj = j;
          }
        }
      }
    });
  }
  for (int o = WAVE / 2; o > 0; o >>= 1) {
    const double t2 = __shfl_xor(bt, o);
    const int o2 = __shfl_xor(bo, o);
    const int j2 = __shfl_xor(bj, o);
    const unsigned long long r2 = __shfl_xor(br, o);
    if (crank ? r2 < br : (t2 < bt || (t2 == bt && o2 < bo))) {
      bt = t2;
      bo = o2;
      bj = j2;
      br = r2;
    }
  }
}

// Exact partner of sphere i by the whole wave (exact_partner) into its key; on the
// single grid Gp, or on its box's in the batched form.
__device__ __forceinline__ void gather_one(int i, const Rec *rec, const int *start, const Grid *Gp,
                                           double dt, const uint8_t *status, int *key_j,
                                           double *key_t, const BatchDev &B,
                                           const unsigned long long *crank) {
  const Rec a = rec[i];
  const int bx = B.gtab ? a.box : 0;
  const Grid G = B.gtab ? B.gtab[bx] : *Gp;
  const int *st = B.gtab ? start + B.cell_base[bx] : start;
  int bj;
  double bt;
  exact_partner(i, a, G, st, rec, dt, crank,
                [&](int j) { return status && status[j] == ST_COLLIDED; }, bj, bt);
  if (__lane_id() == 0) {
    key_j[i] = bj;
    key_t[i] = bt;
  }
}

// Exact partners of a list of spheres, one wave per sphere: `list` of length nlist,
// or *nlist_dev when given, or, with list NULL, all i < nlist.  For spheres whose
// contacts overflowed the slots and grids with fewer than 3 cells along some axis.
__global__ __launch_bounds__(256) void k_gather_exact(const int *list, int nlist,
                                                      const unsigned int *nlist_dev,
                                                      const Rec *rec, const int *start,
                                                      const Grid *Gp, double dt, int *key_j,
                                                      double *key_t, BatchDev B,
                                                      const unsigned int *err,
                                                      const unsigned long long *crank) {
  if (*err) return;
  const int wid = (blockIdx.x * blockDim.x + threadIdx.x) / WAVE;
  const int nw = (gridDim.x * blockDim.x) / WAVE;
  const int count = nlist_dev ? (int)*nlist_dev : nlist;
  for (int w = wid; w < count; w += nw)
    gather_one(list ? list[w] : w, rec, start, Gp, dt, nullptr, key_j, key_t, B, crank);
}

// Keys of a masked detect's ACTIVE spheres.  Behind the pair tests (pairs: they
// were queued, and taken) from their slots, a lane to a sphere, or where they
// overflowed by the exact search; else all by the search.  There a wave looks at
// every nw-th sphere, so neighbours, which may be active together, go to different
// waves; 64 statuses at a time (one after another, 2M spheres of which none was
// active took 257 us, now 154).
__global__ __launch_bounds__(256) void k_masked_keys(const SweepCounters *ctr, int n, int pairs,
                                                     int K, const int *cnt, const double *slot_t,
                                                     const int *slot_j, const Rec *rec,
                                                     const int *start, const Grid *Gp, double dt,
                                                     const uint8_t *status, int *key_j,
                                                     double *key_t) {
  const BatchDev B{};
  const bool dense = pairs && masked_dense(ctr, n);
  const int nw = (gridDim.x * blockDim.x) / WAVE;
  const int wid = (blockIdx.x * blockDim.x + threadIdx.x) / WAVE;
  // a wave's first sphere and the distance between its lanes' spheres
  const int64_t first = dense ? (int64_t)wid * WAVE : wid;
  const int stride = dense ? 1 : nw;
  for (int64_t w0 = first; w0 < n; w0 += (int64_t)nw * WAVE) {
    const int64_t i = w0 + (int64_t)__lane_id() * stride;
    bool search = i < n && status[i] == ST_ACTIVE;
    if (dense && search) {
      const int c = cnt[i];
      search = c > K;
      if (!search) {
        int bj;
        double bt;
        slot_choice((int)i, c, (size_t)n, slot_t, slot_j, rec, Grid{}, nullptr,
                    GoneCollided{status}, bj, bt);
        key_j[i] = bj;
        key_t[i] = bt;
      }
    }
    unsigned long long todo = __builtin_amdgcn_ballot_w64(search);
    while (todo) {
      const int l = __ffsll((long long)todo) - 1;
      todo &= todo - 1ull;
      gather_one((int)(w0 + (int64_t)l * stride), rec, start, Gp, dt, status, key_j, key_t, B,
                 nullptr);
    }
  }
}

hipError_t launch_gather_exact(hipStream_t s, const int *list, int nlist, const unsigned int *nlist_dev,
                               const Rec *rec, const int *start, const Grid *G, double dt, int *key_j,
                               double *key_t, const BatchDev *B, const unsigned int *err,
                               const unsigned long long *crank) {
  // a list whose length is on the device is mostly short: a wave for 8 of the nlist
  // spheres it could name at most, in 16 to 2048 workgroups (for 64, one contact
  // slot and 100k spheres, a third of them listed, the search took 220 us, not 130)
  int64_t waves = nlist_dev ? std::max((int64_t)64, (int64_t)nlist / 8) : nlist;
  if (nlist <= 0) return hipSuccess;
  if (waves > 8192) waves = 8192;
  const int blocks = (int)((waves + 3) / 4);
  BatchDev none{};
  hipLaunchKernelGGL(k_gather_exact, dim3(blocks), dim3(256), 0, s, list, nlist, nlist_dev, rec,
                     start, G, dt, key_j, key_t, B ? *B : none, err, crank);
  return hipGetLastError();
}

// Workgroups: a lane to a sphere, and for few spheres, where they search, up to
// 8192 waves for them.
hipError_t launch_masked_keys(hipStream_t s, const SweepCounters *ctr, int n, bool pairs, int K,
                              const int *cnt, const double *slot_t, const int *slot_j,
                              const Rec *rec, const int *start, const Grid *G, double dt,
                              const uint8_t *status, int *key_j, double *key_t) {
  if (n <= 0) return hipSuccess;
  const int blocks = (int)std::max(((int64_t)n + 255) / 256, (int64_t)(std::min(n, 8192) + 3) / 4);
  hipLaunchKernelGGL(k_masked_keys, dim3(blocks), dim3(256), 0, s, ctr, n, (int)pairs, K, cnt,
                     slot_t, slot_j, rec, start, G, dt, status, key_j, key_t);
  return hipGetLastError();
}

// ---------------------------------------------------------------- a6: mutual resolve

// Rule 4 for sphere i and its mutual partner p: i's end-of-step state into its
// output record (Sec. "Inter-Particle Collisions"; eq. update_vel, update_rho)
// and its status.  Returns 1 for one of the two spheres of the pair.
// SPIN: the friction-and-spin resolve.  The thread of the smaller sorted index
// resolves both sides and writes both spins in place (the partner's thread
// writes nothing, so no thread reads a spin another one has already changed).
// Without spin the record is the caller's to store (o).
template <bool SPIN>
__device__ __forceinline__ unsigned long long resolve_pair(const SweepArgs &A, int i, int p,
                                                           OutRec &o) {
  if (SPIN) {
    if (i > p) return 0ull;
    const Rec a = A.rec[i], b = A.rec[p];
    const double t = A.key_t[i];
    const double ma = A.mass[a.o], mb = A.mass[b.o];
    const Spin &S = A.spin;
    const double wa[3] = {S.wx[a.o], S.wy[a.o], S.wz[a.o]};
    const double wb[3] = {S.wx[b.o], S.wy[b.o], S.wz[b.o]};
    double xo[3], vo[3], wo[3];
    resolve_one_spin(a, b, ma, mb, wa, wb, *A.G, t, A.dt, A.e, S.mu, xo, vo, wo);
    A.out[i] = OutRec{xo[0], xo[1], xo[2], vo[0], vo[1], vo[2], t, b.o, 0u};
    S.wx[a.o] = wo[0];
    S.wy[a.o] = wo[1];
    S.wz[a.o] = wo[2];
    resolve_one_spin(b, a, mb, ma, wb, wa, *A.G, t, A.dt, A.e, S.mu, xo, vo, wo);
    A.out[p] = OutRec{xo[0], xo[1], xo[2], vo[0], vo[1], vo[2], t, a.o, 0u};
    S.wx[b.o] = wo[0];
    S.wy[b.o] = wo[1];
    S.wz[b.o] = wo[2];
    A.status[i] = ST_COLLIDED;
    A.status[p] = ST_COLLIDED;
    return 1ull;
  }
  const Rec a = A.rec[i], b = A.rec[p];
  const double t = A.key_t[i];
  const double ma = A.mass[a.o], mb = A.mass[b.o];
  double xo[3], vo[3];
  if (A.B.gtab) {
    const Grid G = A.B.gtab[a.box];
    resolve_one(a, b, ma, mb, G, t, A.dt, A.e, xo, vo);
  } else {
    resolve_one(a, b, ma, mb, *A.G, t, A.dt, A.e, xo, vo);
  }
  o = OutRec{xo[0], xo[1], xo[2], vo[0], vo[1], vo[2], t, b.o, 0u};
  A.status[i] = ST_COLLIDED;
  return i < p ? 1ull : 0ull;
}

// Pairs resolved by sweep `s` of the queue.  The first sweep adds its pairs up on
// all shards: 62,500 workgroups adding to four addresses took 0.4 ms at 16M.
__device__ __forceinline__ unsigned long long sweep_pairs(const SweepCounters *ctr, int s) {
  unsigned long long t = 0ull;
  if (s == 0) {
    for (int k = 0; k < NSHARD; ++k) t += ctr->shard[k].pairs;
  }
#pragma unroll
  for (int k = 0; k < PAIR_SHARDS; ++k) t += ctr->pairs[s][k];
  return t;
}

// Append this thread's i (where keep) to shard sh of a list behind one atomic per
// workgroup on its count.
__device__ __forceinline__ void list_append(bool keep, int i, int *count, int *list) {
  __shared__ int part[256 / WAVE];
  __shared__ int at;
  const unsigned long long m = __builtin_amdgcn_ballot_w64(keep);
  const int w = threadIdx.x / WAVE;
  if (__lane_id() == 0) part[w] = __popcll(m);
  __syncthreads();
  if (threadIdx.x == 0) {
    const int c = part[0] + part[1] + part[2] + part[3];
    at = c ? atomicAdd(count, c) : 0;
  }
  __syncthreads();
  int base = at;
  for (int k = 0; k < w; ++k) base += part[k];
  if (keep) list[base + __popcll(m & ((1ull << __lane_id()) - 1ull))] = i;
  __syncthreads();  // part and at are free again
}

// The first sweep (rule 3-4), over every sphere in cell-sorted order.  A sphere
// whose partner has it as partner collides; one whose partner pairs with a
// third sphere becomes DIRTY (k_rekey finds it another); one without a partner
// is FREE for the step.  Each thread writes its own status only and reads keys
// only, so the sweep is a pure function of the keys.  Partners are spatial
// neighbours, so the partner reads stay within a few cells of the sorted order.
// The spheres left for the later sweeps (8.5% at 16M) go to a list: each
// workgroup appends its own behind one atomic, to the part of the list that
// belongs to its shard.  Shards take every 64th workgroup, so the workgroups
// that run at one time spread over all of them (shards of consecutive
// workgroups, and with them one address for most of the chip: 600 us at 16M).
template <bool SPIN>
__global__ __launch_bounds__(256) void k_sweep_first(SweepArgs A, const int *key) {
  if (*A.err || (!A.exact && A.ctr->n_overflow != 0u)) return;
  const int i = blockIdx.x * 256 + threadIdx.x;
  unsigned long long npair = 0ull;
  bool keep = false;
  OutRec o{};
  int to = -1;
  if (i < A.n) {
    const int p = key[i];
    if (p < 0) {
      A.status[i] = ST_FREE;
    } else {
      const int q = key[p];
      if (q == i) {
        npair = resolve_pair<SPIN>(A, i, p, o);
        to = i;
      } else {
        keep = true;
        A.status[i] = q >= 0 && key[q] == p ? ST_DIRTY : ST_ACTIVE;
      }
    }
  }
  if (!SPIN) {
    __shared__ Stage<4> stage[256 / WAVE];
    store_records(o, to, A.out, stage[threadIdx.x / WAVE]);
  }
  const int sh = blockIdx.x % A.shards;
  list_append(keep, i, &A.ctr->list[sh].n[0], A.list[0] + (size_t)sh * A.shard_blocks * 256);
  block_add(npair, &my_shard(A.ctr).pairs);
}

// Spheres no longer eligible after a sweep with the keys `in`: those done before
// it and those that collide in it (in[in[j]] == j), whatever status they have by
// now.
struct GoneInSweep {
  const uint8_t *status;
  const int *in;
  __device__ __forceinline__ bool one(int j) const {
    if (status[j] != ST_ACTIVE) return true;
    const int p = in[j];
    return p >= 0 && in[p] == j;
  }
  __device__ __forceinline__ void operator()(const int (&j)[4], bool (&g)[4]) const {
    bool act[4];
    int p[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      act[u] = status[j[u]] == ST_ACTIVE;
      p[u] = in[j[u]];  // a key only where j is active
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) p[u] = act[u] && p[u] >= 0 ? p[u] : -1;
#pragma unroll
    for (int u = 0; u < 4; ++u) g[u] = !act[u] || (p[u] >= 0 && in[p[u]] == j[u]);
  }
};

// New partner of a listed sphere i (need: it wants one, else the lane only takes
// part) among those not gone: from its slots, or (EXACT) by the exact search,
// the wave on one sphere after another, where its contacts overflowed them or
// the grid is too small for the pair tests.
template <bool EXACT, typename Gone>
__device__ __forceinline__ void new_partner(const SweepArgs &A, bool need, int i, const Gone &gone,
                                            int &bj, double &bt) {
  bj = -1;
  bt = INFINITY;
  bool search = false;
  if (need) {
    const int c = EXACT && A.small ? 0 : A.cnt[i];
    search = EXACT && (A.small || c > A.K);
    Grid G{};  // the walls are all that matters here (none in the batched form)
    if (A.G) G = *A.G;
    if (!search)
      slot_choice(i, c, (size_t)A.n, A.slot_t, A.slot_j, A.rec, G, A.crank, gone, bj, bt);
  }
  if (!EXACT) return;
  unsigned long long todo = __builtin_amdgcn_ballot_w64(search);
  if (!todo) return;
  if (!A.small && (int)__lane_id() == __ffsll((long long)todo) - 1)
    atomicAdd(&A.ctr->ovf_later, (unsigned int)__popcll(todo));
  while (todo) {
    const int l = __ffsll((long long)todo) - 1;
    todo &= todo - 1ull;
    const int w = __builtin_amdgcn_readlane(i, l);
    const Rec a = A.rec[w];
    const auto is_gone = [&](int j) { return gone.one(j); };
    int j;
    double t;
    if (A.B.gtab)
      exact_partner(w, a, A.B.gtab[a.box], A.start + A.B.cell_base[a.box], A.rec, A.dt, A.crank,
                    is_gone, j, t);
    else
      exact_partner(w, a, *A.G, A.start, A.rec, A.dt, A.crank, is_gone, j, t);
    if ((int)__lane_id() == l) {
      bj = j;
      bt = t;
    }
  }
}

// Whether a kernel of the later sweeps has nothing to do: an error, or no exact
// search in a step that needs it (some sphere's contacts overflowed its slots):
// the host sees the overflow and queues the sweeps again with it.  The search
// costs 30 registers, so steps without overflow go without.
template <bool EXACT>
__device__ __forceinline__ bool sweep_off(const SweepArgs &A) {
  return *A.err || (!EXACT && A.ctr->n_overflow != 0u);
}

// Entries of the list that a wave takes at a time: all its lanes one each, but
// where they may have to search, the wave on one sphere after another, one or a
// few (64 searches in a row took 0.4 ms a step in boxes of fewer than 3 cells on an
// axis, where every new partner is a search; with one contact slot, two steps of
// 100k spheres take 1277, 1303 and 1387 us for 2, 4 and 8 entries, of 1M 8346,
// 8098 and 8007).
template <bool EXACT>
__device__ __forceinline__ int wave_share(const SweepArgs &A) {
  return !EXACT ? WAVE : (A.small ? 1 : 4);
}

// This lane's entry, count (none) past the end or its wave's share.
__device__ __forceinline__ int list_entry(int t0, int share, int count) {
  const int l = (int)threadIdx.x % WAVE, t = t0 + (int)threadIdx.x / WAVE * share + l;
  return l < share && t < count ? t : count;
}

// The partners of the spheres that sweep 1 left DIRTY (in place: only DIRTY keys
// change and no key is read).
template <bool EXACT>
__global__ __launch_bounds__(256) void k_rekey(SweepArgs A, int *key) {
  if (sweep_off<EXACT>(A)) return;
  const int sh = blockIdx.y, count = A.ctr->list[sh].n[0];
  const int *list = A.list[0] + (size_t)sh * A.shard_blocks * 256;
  const GoneCollided gone{A.status};
  const int share = wave_share<EXACT>(A), step = share * (256 / WAVE);
  for (int t0 = blockIdx.x * step; t0 < count; t0 += gridDim.x * step) {
    const int t = list_entry(t0, share, count);
    const int i = t < count ? list[t] : 0;
    const bool need = t < count && A.status[i] == ST_DIRTY;
    int bj;
    double bt;
    new_partner<EXACT>(A, need, i, gone, bj, bt);
    if (need) {
      key[i] = bj;
      A.key_t[i] = bt;
      A.status[i] = ST_ACTIVE;
    }
  }
}

// A later sweep over the list, `in` its keys: the mutual pairs collide, and a
// sphere whose partner collides with a third one takes its next partner at
// once, so the keys of the next sweep (out) leave with this kernel and a sweep
// is one launch.  Whether a sphere collides in this sweep follows from the keys
// alone (in[in[j]] == j), so nothing waits for the statuses other threads write
// meanwhile.  Only listed spheres are ever looked up: an eligible contact of an
// active sphere is active itself.  The spheres still active go to the next
// sweep's list: list lin is read, the other one written; of the three counts of
// a shard, this sweep reads count c, adds to the next and clears the one after.
// The sweep runs if the one before it (s - 1) resolved a pair, or if it is the
// first over the list or of its queue.
template <bool SPIN, bool EXACT>
__global__ __launch_bounds__(256) void k_sweep(SweepArgs A, const int *in, int *out, int s,
                                               int first, int lin, int c) {
  if (sweep_off<EXACT>(A)) return;
  if (!first && sweep_pairs(A.ctr, s - 1) == 0ull) return;
  const int sh = blockIdx.y;
  const int c1 = c == 2 ? 0 : c + 1, c2 = c1 == 2 ? 0 : c1 + 1;
  const int count = A.ctr->list[sh].n[c];
  if (blockIdx.x == 0 && threadIdx.x == 0) A.ctr->list[sh].n[c2] = 0;
  const int share = wave_share<EXACT>(A), step = share * (256 / WAVE);
  if ((int)blockIdx.x * step >= count) return;
  const size_t at = (size_t)sh * A.shard_blocks * 256;
  const int *list = A.list[lin] + at;
  int *next = A.list[lin ^ 1] + at;
  const GoneInSweep gone{A.status, in};
  unsigned long long npair = 0ull;
  for (int t0 = blockIdx.x * step; t0 < count; t0 += gridDim.x * step) {
    const int t = list_entry(t0, share, count);
    const int i = t < count ? list[t] : 0;
    bool need = false, keep = false;
    if (t < count && A.status[i] == ST_ACTIVE) {
      const int p = in[i];
      if (p < 0) {
        A.status[i] = ST_FREE;
      } else {
        const int q = in[p];
        if (q == i) {
          OutRec o;
          npair += resolve_pair<SPIN>(A, i, p, o);
          if (!SPIN) A.out[i] = o;
        } else {
          keep = true;
          need = q >= 0 && in[q] == p;
          if (!need) out[i] = p;
        }
      }
    }
    if (__builtin_amdgcn_ballot_w64(need)) {
      int bj;
      double bt;
      new_partner<EXACT>(A, need, i, gone, bj, bt);
      if (need) {
        out[i] = bj;
        A.key_t[i] = bt;
      }
    }
    list_append(keep, i, &A.ctr->list[sh].n[c1], next);
  }
  block_add(npair, &A.ctr->pairs[s][blockIdx.x % PAIR_SHARDS]);
}

// Shards of the list for n spheres (at least 8 workgroups of the first sweep
// each) and their room in it, in workgroups.
void sweep_shards(SweepArgs &A) {
  const int nb = (A.n + 255) / 256;
  A.shards = std::min(NSHARD, std::max(1, nb / 8));
  A.shard_blocks = (nb + A.shards - 1) / A.shards;
}

hipError_t launch_sweep_first(hipStream_t s, const SweepArgs &A, const int *key) {
  if (A.n <= 0) return hipSuccess;
  const dim3 grid((A.n + 255) / 256);
  if (A.spin.wx)
    hipLaunchKernelGGL(k_sweep_first<true>, grid, dim3(256), 0, s, A, key);
  else
    hipLaunchKernelGGL(k_sweep_first<false>, grid, dim3(256), 0, s, A, key);
  return hipGetLastError();
}

// Grid of a kernel over the list: one row of workgroups per shard, enough for
// a quarter of the spheres at once (a tenth is usual; more take another turn).
static dim3 list_grid(const SweepArgs &A) {
  const int per = A.exact ? (A.small ? WAVE : 16) : 1;  // workgroups for 256 entries
  return dim3((unsigned)std::min((int64_t)8192, ((int64_t)A.shard_blocks * per + 3) / 4), A.shards);
}

hipError_t launch_rekey(hipStream_t s, const SweepArgs &A, int *key) {
  if (A.n <= 0) return hipSuccess;
  if (A.exact)
    hipLaunchKernelGGL(k_rekey<true>, list_grid(A), dim3(256), 0, s, A, key);
  else
    hipLaunchKernelGGL(k_rekey<false>, list_grid(A), dim3(256), 0, s, A, key);
  return hipGetLastError();
}

hipError_t launch_sweep(hipStream_t s, const SweepArgs &A, const int *in, int *out, int k,
                        bool first, int turn) {
  if (A.n <= 0) return hipSuccess;
  const auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, list_grid(A), dim3(256), 0, s, A, in, out, k, (int)first, turn & 1,
                       turn % 3);
  };
  if (A.spin.wx)
    A.exact ? go(k_sweep<true, true>) : go(k_sweep<true, false>);
  else
    A.exact ? go(k_sweep<false, true>) : go(k_sweep<false, false>);
  return hipGetLastError();
}

// What the host reads of a step, written to its memory by the last kernel.
__device__ __forceinline__ void write_report(const SweepCounters *ctr, int nsweep,
                                             StepReport *rep) {
  const int t = threadIdx.x;
  for (int k = t; k < nsweep; k += 256) rep->pairs[k] = sweep_pairs(ctr, k);
  if (t < NSHARD) {
    const unsigned long long c = wave_sum(ctr->shard[t].contacts),
                             r = wave_sum(ctr->shard[t].recheck),
                             e = wave_sum(ctr->shard[t].tests);
    if (t == 0) {
      rep->contacts = c;
      rep->recheck = r;
      rep->tests = e;
      rep->n_overflow = ctr->n_overflow + ctr->ovf_later;
      rep->maxcell = ctr->maxcell;
    }
  }
}

// a8 and the copy back: the end-of-step state of every sphere in the caller's
// order (coalesced writes), if the last of the nsweep sweeps queued resolved no
// pair (otherwise the host queues more).  A sphere whose status (sorted order)
// says it collided this step takes the output record its resolve wrote; any
// other flies the whole step from its start state, still in the caller's arrays
// (rule 5).  Only collided spheres read their 64-B output record; the others
// read one status byte (a 1-B-per-sphere array that stays in the device's
// last-level cache).
__global__ __launch_bounds__(256) void k_finish(Particles P, const int *rank,
                                                const OutRec *out, const uint8_t *status,
                                                int *partner, double *tcoll, double dt,
                                                const StepPlan *plan, const int *start, BatchDev B,
                                                const SweepCounters *ctr, int nsweep, int exact,
                                                const unsigned int *err, StepReport *rep) {
  if (blockIdx.x == 0) {
    write_report(ctr, nsweep, rep);
    if (plan && threadIdx.x == 0)
      rep->wide_first = !*err && plan->G.layer2 ? start[plan->G.layer2] : (int)P.n;
  }
  if (*err || (!exact && ctr->n_overflow != 0u) ||
      sweep_pairs(ctr, nsweep - 1) != 0ull)
    return;
  const int64_t o = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (o >= P.n) return;
  double x, y, z, vx, vy, vz, t;
  int pj;
  const int q = rank[o];
  if (status[q] == ST_COLLIDED) {
    const OutRec r = out[q];
    x = r.x;
    y = r.y;
    z = r.z;
    vx = r.vx;
    vy = r.vy;
    vz = r.vz;
    t = r.t;
    pj = r.partner;
  } else {
    const double *L = plan ? plan->G.L : B.gtab[B.box_of[o]].L;
    const int walls = plan ? plan->G.walls : 0;  // the batched form has periodic boxes only
    vx = P.vx[o];
    vy = P.vy[o];
    vz = P.vz[o];
    x = fly_axis(P.x[o] + dt * vx, L[0], walls & 1, vx);
    y = fly_axis(P.y[o] + dt * vy, L[1], walls & 2, vy);
    z = fly_axis(P.z[o] + dt * vz, L[2], walls & 4, vz);
    t = __longlong_as_double(0x7ff8000000000000LL);  // NaN: no collision
    pj = -1;
  }
  P.x[o] = x;
  P.y[o] = y;
  P.z[o] = z;
  P.vx[o] = vx;
  P.vy[o] = vy;
  P.vz[o] = vz;
  partner[o] = pj;
  tcoll[o] = t;
}

hipError_t launch_finish(hipStream_t s, const Particles &P, const int *rank, const OutRec *out,
                         const uint8_t *status, int *partner, double *tcoll, double dt,
                         const StepPlan *plan, const int *start, const BatchDev *B,
                         const SweepCounters *ctr, int nsweep, bool exact, const unsigned int *err,
                         StepReport *rep) {
  // one workgroup also where there are no spheres: the host reads the report
  BatchDev none{};
  const unsigned blocks = P.n > 0 ? (unsigned)((P.n + 255) / 256) : 1u;
  hipLaunchKernelGGL(k_finish, dim3(blocks), dim3(256), 0, s, P, rank, out,
                     status, partner, tcoll, dt, plan, start, B ? *B : none, ctr, nsweep,
                     (int)exact, err, rep);
  return hipGetLastError();
}

// ---------------------------------------------------------------- few spheres

// The kernels of a step of few spheres are a chain of launches of 2 to 7 us each,
// most of it latency: 14 of them took 80 us at 2,000 spheres.  One workgroup does
// what comes before the pair tests and, for fewer still, one what comes after,
// with the cell counts, keys and statuses in LDS and a barrier where the chain had
// a launch; the pair tests between them keep the whole chip.

// Reach, checks, plan, counting sort (and the literal order's ranks) of
// n <= SMALL_N spheres, as k_reach, k_plan, k_cell_hist, k_scan, k_scatter and
// k_curve_rank do them.  No extent split (a plan of fewer than 4096 spheres has
// none).  A grid of more than SMALL_CELLS cells is for the other kernels
// (PLAN_AGAIN).
__global__ __launch_bounds__(1024) void k_bin_small(Particles P, PlanArgs A, SweepCounters *ctr,
                                                    StepPlan *plan, StepPlan *plan_host,
                                                    int *start, Rec *rec, int *rank, int *cnt,
                                                    unsigned long long *crank) {
  const int t = threadIdx.x, n = (int)P.n;
  constexpr int PER = SMALL_N / 1024;
  __shared__ int count[SMALL_CELLS + 1];
  __shared__ StepPlan S;
  Word64 *w = (Word64 *)ctr;
  for (int k = t; k < (int)(sizeof(SweepCounters) / 8); k += 1024) w[k] = 0ull;
  double v2 = 0.0, rm = 0.0, rn = INFINITY, em = 0.0;
  unsigned int bad = 0u;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int i = t + k * 1024;
    if (i >= n) continue;
    const double x = P.x[i], y = P.y[i], z = P.z[i], vx = P.vx[i], vy = P.vy[i], vz = P.vz[i];
    const double r = P.r[i], m = P.m[i];
    const double q = (vx * vx + vy * vy) + vz * vz;
    const bool fin = isfinite(x) && isfinite(y) && isfinite(z) && isfinite(q) && isfinite(r) &&
                     isfinite(m);
    if (!fin || !(r > 0.0) || !(m > 0.0)) bad |= 1u;
    if (P.wx && (!isfinite(P.wx[i]) || !isfinite(P.wy[i]) || !isfinite(P.wz[i]))) bad |= 1u;
    if (!(x >= 0.0 && x < A.L[0]) || !(y >= 0.0 && y < A.L[1]) || !(z >= 0.0 && z < A.L[2]))
      bad |= 2u;
    if (fin) {
      v2 = q > v2 ? q : v2;
      rm = r > rm ? r : rm;
      rn = r < rn ? r : rn;
      if (r > 0.0) {
        const double ex = extent(r, vx, vy, vz, A.dt);
        em = ex > em ? ex : em;
      }
    }
  }
  ReachPart part{dbits(v2), dbits(rm), dbits(rn), dbits(em), bad, 0u};
  __shared__ ReachPart wpart[1024 / WAVE];
  for (int o = WAVE / 2; o > 0; o >>= 1) {
    ReachPart q;
    q.v2max = __shfl_xor(part.v2max, o);
    q.rmax = __shfl_xor(part.rmax, o);
    q.rmin = __shfl_xor(part.rmin, o);
    q.rhomax = __shfl_xor(part.rhomax, o);
    q.bad = __shfl_xor(part.bad, o);
    part = reach_merge(part, q);
  }
  if (__lane_id() == 0) wpart[t / WAVE] = part;
  __syncthreads();
  if (t == 0) {
    for (int k = 1; k < 1024 / WAVE; ++k) part = reach_merge(part, wpart[k]);
    make_plan(A, part, -1, S);
    if (!S.err && S.cells > SMALL_CELLS) S.err = PLAN_AGAIN;
  }
  for (int k = t; k <= SMALL_CELLS; k += 1024) count[k] = 0;
  __syncthreads();
  const Word64 *o = (const Word64 *)&S;
  for (int k = t; k < (int)(sizeof(StepPlan) / 8); k += 1024) {
    ((Word64 *)plan)[k] = o[k];
    ((Word64 *)plan_host)[k] = o[k];
  }
  if (S.err) return;
  const Grid &G = S.G;
  int cell[PER], slot[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int i = t + k * 1024;
    if (i >= n) continue;
    const int cx = cell_coord(P.x[i], G.inv_h[0], G.nc[0]);
    const int cy = cell_coord(P.y[i], G.inv_h[1], G.nc[1]);
    const int cz = cell_coord(P.z[i], G.inv_h[2], G.nc[2]);
    cell[k] = (cz * G.nc[1] + cy) * G.nc[0] + cx;
    slot[k] = atomicAdd(&count[cell[k]], 1);
  }
  __syncthreads();
  constexpr int CPT = SMALL_CELLS / 1024;
  int c[CPT], sum = 0, mx = 0;
#pragma unroll
  for (int k = 0; k < CPT; ++k) {
    c[k] = count[t * CPT + k];
    sum += c[k];
    mx = c[k] > mx ? c[k] : mx;
  }
  int run;
  block_exclusive_scan(sum, run);
#pragma unroll
  for (int k = 0; k < CPT; ++k) {
    count[t * CPT + k] = run;
    run += c[k];
  }
  if (t == 1023) count[SMALL_CELLS] = run;
  for (int q = WAVE / 2; q > 0; q >>= 1) {
    const int m = __shfl_xor(mx, q);
    mx = m > mx ? m : mx;
  }
  if (__lane_id() == 0) atomicMax(&ctr->maxcell, (unsigned int)mx);
  __syncthreads();
  for (int k = t; k <= S.cells; k += 1024) start[k] = count[k];
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int i = t + k * 1024;
    if (i >= n) continue;
    const int pos = count[cell[k]] + slot[k];
    const Rec q{P.x[i], P.y[i], P.z[i], P.r[i], P.vx[i], P.vy[i], P.vz[i], i, 0};
    rec[pos] = q;
    rank[i] = pos;
    cnt[i] = 0;
    if (crank) crank[pos] = curve_rank(S.C, q.x, q.y, q.z, i);
  }
}

hipError_t launch_bin_small(hipStream_t s, const Particles &P, const PlanArgs &A,
                            SweepCounters *ctr, StepPlan *plan, StepPlan *plan_host, int *start,
                            Rec *rec, int *rank, int *cnt, unsigned long long *crank) {
  if (P.n < 1 || P.n > SMALL_N) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_bin_small, dim3(1), dim3(1024), 0, s, P, A, ctr, plan, plan_host, start, rec,
                     rank, cnt, crank);
  return hipGetLastError();
}

// Partners, every sweep, free flight and the report of n <= SMALL_TAIL spheres, as
// k_slot_min, k_sweep_first, k_rekey, k_sweep and k_finish do them (keys in two
// arrays in turn; status and keys in LDS).  cap > 0: the most sweeps; if the last
// still resolved pairs, nothing of the caller's is written.  Contacts
// that overflow their slots are for the other kernels: only the report is written.
__global__ __launch_bounds__(1024) void k_sweeps_small(SweepArgs A, Particles P, int *partner,
                                                       double *tcoll, int cap, StepReport *rep) {
  if (*A.err) return;
  const int t = threadIdx.x, n = A.n;
  __shared__ int key[2][SMALL_TAIL];
  __shared__ uint8_t status[SMALL_TAIL];
  __shared__ unsigned long long total[3];  // contacts; pairs of the sweep, in two words in turn
  __shared__ int overflow;
  if (t < 3) total[t] = 0ull;
  if (t == 3) overflow = 0;
  __syncthreads();
  const Grid G = *A.G;
  unsigned long long nc = 0ull;
  for (int i = t; i < n; i += 1024) {
    const int c = A.cnt[i];
    nc += (unsigned long long)c;
    if (c > A.K) atomicAdd(&overflow, 1);
    int bj;
    double bt;
    slot_choice(i, c > A.K ? 0 : c, (size_t)n, A.slot_t, A.slot_j, A.rec, G, A.crank, GoneNone{},
                bj, bt);
    key[0][i] = bj;
    A.key_t[i] = bt;
    status[i] = bj < 0 ? ST_FREE : ST_ACTIVE;
  }
  nc = wave_sum(nc);
  if (__lane_id() == 0 && nc) atomicAdd(&total[0], nc);
  __syncthreads();
  A.status = status;
  unsigned long long pairs = 0ull;
  int sweeps = 0;
  bool done = false;
  while (!overflow && !done && (cap == 0 || sweeps < cap)) {
    const int *in = key[sweeps & 1];
    int *out = key[~sweeps & 1];
    unsigned long long *now = &total[1 + (sweeps & 1)];
    const GoneInSweep gone{status, in};
    unsigned long long np = 0ull;
    for (int i = t; i < n; i += 1024) {
      if (status[i] != ST_ACTIVE) continue;
      const int p = in[i];
      if (p < 0) {
        status[i] = ST_FREE;
        continue;
      }
      const int q = in[p];
      if (q == i) {
        OutRec o;
        np += resolve_pair<false>(A, i, p, o);
        A.out[i] = o;
        continue;
      }
      int bj = p;
      if (q >= 0 && in[q] == p) {
        double bt;
        slot_choice(i, A.cnt[i], (size_t)n, A.slot_t, A.slot_j, A.rec, G, A.crank, gone, bj, bt);
        A.key_t[i] = bt;
      }
      out[i] = bj;
    }
    np = wave_sum(np);
    if (__lane_id() == 0 && np) atomicAdd(now, np);
    __syncthreads();
    const unsigned long long got = *now;
    if (t == 0) total[1 + (~sweeps & 1)] = 0ull;
    pairs += got;
    done = got == 0ull;
    ++sweeps;
    __syncthreads();
  }
  if (t == 0) {
    rep->contacts = total[0];
    rep->recheck = 0ull;
    rep->tests = 0ull;
    rep->n_overflow = (unsigned int)overflow;
    rep->maxcell = A.ctr->maxcell;
    rep->wide_first = n;
    rep->small_pairs = pairs;
    rep->small_sweeps = sweeps;
    rep->small_done = done;
  }
  if (t < NSHARD) {
    const unsigned long long r = wave_sum(A.ctr->shard[t].recheck),
                             e = wave_sum(A.ctr->shard[t].tests);
    if (t == 0) {
      rep->recheck = r;
      rep->tests = e;
    }
  }
  if (!done) return;
  for (int i = t; i < n; i += 1024) {
    const Rec a = A.rec[i];
    OutRec r;
    if (status[i] == ST_COLLIDED) {
      r = A.out[i];
    } else {
      r.vx = a.vx;
      r.vy = a.vy;
      r.vz = a.vz;
      r.x = fly_axis(a.x + A.dt * a.vx, G.L[0], G.walls & 1, r.vx);
      r.y = fly_axis(a.y + A.dt * a.vy, G.L[1], G.walls & 2, r.vy);
      r.z = fly_axis(a.z + A.dt * a.vz, G.L[2], G.walls & 4, r.vz);
      r.t = __longlong_as_double(0x7ff8000000000000LL);  // NaN: no collision
      r.partner = -1;
    }
    P.x[a.o] = r.x;
    P.y[a.o] = r.y;
    P.z[a.o] = r.z;
    P.vx[a.o] = r.vx;
    P.vy[a.o] = r.vy;
    P.vz[a.o] = r.vz;
    partner[a.o] = r.partner;
    tcoll[a.o] = r.t;
  }
}

hipError_t launch_sweeps_small(hipStream_t s, const SweepArgs &A, const Particles &P, int *partner,
                               double *tcoll, int cap, StepReport *rep) {
  if (A.n < 1 || A.n > SMALL_TAIL || A.spin.wx) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_sweeps_small, dim3(1), dim3(1024), 0, s, A, P, partner, tcoll, cap, rep);
  return hipGetLastError();
}

// ---------------------------------------------------------------- a8: free flight + wrap

// rule 5: spheres that did not collide fly the whole step; coalesced over the
// caller's order.
__global__ __launch_bounds__(256) void k_advance(Particles P, const int *partner, double dt,
                                                 double L0, double L1, double L2) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= P.n || partner[i] >= 0) return;
  P.x[i] = wrap_pos(P.x[i] + dt * P.vx[i], L0);
  P.y[i] = wrap_pos(P.y[i] + dt * P.vy[i], L1);
  P.z[i] = wrap_pos(P.z[i] + dt * P.vz[i], L2);
}

hipError_t launch_advance(hipStream_t s, const Particles &P, const int *partner, double dt,
                          const double L[3]) {
  if (P.n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_advance, dim3((unsigned)((P.n + 255) / 256)), dim3(256), 0, s, P, partner,
                     dt, L[0], L[1], L[2]);
  return hipGetLastError();
}

// ---------------------------------------------------------------- public single-sweep API

// caller active mask -> sorted status (inactive spheres are excluded like
// collided ones); clears the contact counts and counts the active spheres (on one
// address, the 1172 adds for 300,000 spheres took 12 us)
__global__ __launch_bounds__(256) void k_status_from_active(const uint8_t *active,
                                                            const Rec *rec, int n,
                                                            uint8_t *status, int *cnt,
                                                            SweepCounters *ctr) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  bool act = false;
  if (i < n) {
    act = active[rec[i].o] != 0;
    status[i] = act ? ST_ACTIVE : ST_COLLIDED;
    cnt[i] = 0;
  }
  block_add(act ? 1ull : 0ull, &ctr->shard[blockIdx.x % ACTIVE_SHARDS].active);
}

hipError_t launch_status_from_active(hipStream_t s, const uint8_t *active, const Rec *rec, int n,
                                     uint8_t *status, int *cnt, SweepCounters *ctr) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_status_from_active, dim3((n + 255) / 256), dim3(256), 0, s, active, rec,
                     n, status, cnt, ctr);
  return hipGetLastError();
}

// keys in the caller's order: (bits of (float)t) << 32 | caller index of the partner
__global__ __launch_bounds__(256) void k_export_keys(int n, const Rec *rec, const int *key_j,
                                                     const double *key_t, const uint8_t *status,
                                                     SweepCounters *ctr, uint64_t *key_out,
                                                     double *tmin_out) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (status && i < ACTIVE_SHARDS) ctr->shard[i].active = 0ull;
  if (i >= n) return;
  const int o = rec[i].o;
  const int j = key_j[i];
  const bool has = j >= 0 && (!status || status[i] == ST_ACTIVE);
  uint64_t key = ~0ull;
  double t = INFINITY;
  if (has) {
    t = key_t[i];
    const float tf = (float)t;
    key = ((uint64_t)__float_as_uint(tf) << 32) | (uint64_t)(uint32_t)rec[j].o;
  }
  key_out[o] = key;
  if (tmin_out) tmin_out[o] = t;
}

hipError_t launch_export_keys(hipStream_t s, int n, const Rec *rec, const int *key_j,
                              const double *key_t, const uint8_t *status, SweepCounters *ctr,
                              uint64_t *key_out, double *tmin_out) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_export_keys, dim3((n + 255) / 256), dim3(256), 0, s, n, rec, key_j, key_t,
                     status, ctr, key_out, tmin_out);
  return hipGetLastError();
}

// rule 3-4 from caller-order keys; start-of-step data from the binned records
__global__ __launch_bounds__(256) void k_resolve_public(int n, const Rec *rec, const int *rank,
                                                        Grid G, double dt, double e,
                                                        const uint64_t *key, Particles P,
                                                        uint8_t *active, int *partner,
                                                        double *tcoll, long long *npairs) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  unsigned long long np = 0ull;
  if (i < n && active[i] != 0 && key[i] != ~0ull) {
    const int p = (int)(uint32_t)(key[i] & 0xffffffffull);
    if (p >= 0 && p < n && p != i && key[p] != ~0ull &&
        (int)(uint32_t)(key[p] & 0xffffffffull) == i) {
      const Rec a = rec[rank[i]], b = rec[rank[p]];
      double t;
      if (pair_time(a, b, G, dt, t)) {
        double xo[3], vo[3];
        resolve_one(a, b, P.m[i], P.m[p], G, t, dt, e, xo, vo);
        P.x[i] = xo[0];
        P.y[i] = xo[1];
        P.z[i] = xo[2];
        P.vx[i] = vo[0];
        P.vy[i] = vo[1];
        P.vz[i] = vo[2];
        active[i] = 0;
        if (partner) partner[i] = p;
        if (tcoll) tcoll[i] = t;
        if (i < p) np = 1ull;
      }
    }
  }
  np = wave_sum(np);
  if (__lane_id() == 0 && np && npairs) atomicAdd((unsigned long long *)npairs, np);
}

hipError_t launch_resolve_public(hipStream_t s, int n, const Rec *rec, const int *rank,
                                 const Grid &G, double dt, double e, const uint64_t *key,
                                 const Particles &P, uint8_t *active, int *partner, double *tcoll,
                                 long long *npairs) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_resolve_public, dim3((n + 255) / 256), dim3(256), 0, s, n, rec, rank, G,
                     dt, e, key, P, active, partner, tcoll, npairs);
  return hipGetLastError();
}

}  // namespace pcol

namespace pcol {

// ---------------------------------------------------------------- adjoint of one step

// One sphere of k_step_backward: writes its gradients, and its partner's if it has
// the smaller index, and returns the pair's e-gradient.
__device__ __forceinline__ double backward_sphere(int i, const double *x, const double *y,
                                                  const double *z, const double *vx,
                                                  const double *vy, const double *vz,
                                                  const double *r, const double *m, const Grid &G,
                                                  double dt, double e, const int *partner,
                                                  const double *tcoll, const StateGrad &gout,
                                                  const StateGrad &gin) {
  const int j = partner[i];
  const bool both = j >= 0 && partner[j] == i;  // a record of one side only is taken as it is
  if (both && j < i) return 0.0;                 // the partner's thread does both
  const double Gxi[3] = {gout.x[i], gout.y[i], gout.z[i]};
  const double Gvi[3] = {gout.vx[i], gout.vy[i], gout.vz[i]};
  if (j < 0) {
    gin.x[i] = Gxi[0];
    gin.y[i] = Gxi[1];
    gin.z[i] = Gxi[2];
    gin.vx[i] = Gvi[0] + dt * Gxi[0];
    gin.vy[i] = Gvi[1] + dt * Gxi[1];
    gin.vz[i] = Gvi[2] + dt * Gxi[2];
    return 0.0;
  }
  const double Gxj[3] = {gout.x[j], gout.y[j], gout.z[j]};
  const double Gvj[3] = {gout.vx[j], gout.vy[j], gout.vz[j]};
  const double xi[3] = {x[i], y[i], z[i]}, xj[3] = {x[j], y[j], z[j]};
  const double vi[3] = {vx[i], vy[i], vz[i]}, vj[3] = {vx[j], vy[j], vz[j]};
  const double t = tcoll[i];
  double d[3], u[3], nn[3];
  for (int k = 0; k < 3; ++k) {
    d[k] = wrap_sep(xj[k] - xi[k], G.L[k], G.halfL[k]);
    u[k] = vj[k] - vi[k];
  }
  const double s = r[i] + r[j];
  for (int k = 0; k < 3; ++k) nn[k] = (d[k] + t * u[k]) / s;
  const double g = (u[0] * nn[0] + u[1] * nn[1]) + u[2] * nn[2];
  const double mr = (m[i] * m[j]) / (m[i] + m[j]);
  const double c = mr * (1.0 + e);
  const double J = c * g;
  double vin[3], vjn[3];
  for (int k = 0; k < 3; ++k) {
    vin[k] = vi[k] + (J / m[i]) * nn[k];
    vjn[k] = vj[k] - (J / m[j]) * nn[k];
  }
  // adjoints
  double tb = 0.0, Jb = 0.0, bvi[3], bvj[3], bvin[3], bvjn[3], bn[3], bu[3], bd[3];
  for (int k = 0; k < 3; ++k) {
    tb += Gxi[k] * (vi[k] - vin[k]) + Gxj[k] * (vj[k] - vjn[k]);
    bvin[k] = Gvi[k] + (dt - t) * Gxi[k];
    bvjn[k] = Gvj[k] + (dt - t) * Gxj[k];
    bvi[k] = t * Gxi[k] + bvin[k];
    bvj[k] = t * Gxj[k] + bvjn[k];
    Jb += bvin[k] * nn[k] / m[i] - bvjn[k] * nn[k] / m[j];
    bn[k] = (J / m[i]) * bvin[k] - (J / m[j]) * bvjn[k];
  }
  const double gb = c * Jb;
  const double eb = mr * g * Jb;
  for (int k = 0; k < 3; ++k) {
    bu[k] = gb * nn[k];
    bn[k] += gb * u[k];
  }
  double wb[3];
  for (int k = 0; k < 3; ++k) {
    wb[k] = bn[k] / s;
    bd[k] = wb[k];
    tb += wb[k] * u[k];
    bu[k] += t * wb[k];
  }
  for (int k = 0; k < 3; ++k) {
    bd[k] += (-tb / g) * nn[k];
    bu[k] += (-tb * t / g) * nn[k];
  }
  // d = x_j - x_i, u = v_j - v_i
  gin.x[i] = Gxi[0] - bd[0];
  gin.y[i] = Gxi[1] - bd[1];
  gin.z[i] = Gxi[2] - bd[2];
  gin.vx[i] = bvi[0] - bu[0];
  gin.vy[i] = bvi[1] - bu[1];
  gin.vz[i] = bvi[2] - bu[2];
  if (!both) return i < j ? eb : 0.0;
  gin.x[j] = Gxj[0] + bd[0];
  gin.y[j] = Gxj[1] + bd[1];
  gin.z[j] = Gxj[2] + bd[2];
  gin.vx[j] = bvj[0] + bu[0];
  gin.vy[j] = bvj[1] + bu[1];
  gin.vz[j] = bvj[2] + bu[2];
  return eb;
}

// Reverse-mode derivative of one step with the pair set fixed (caller order).
// Forward quantities of a pair (i, j) from i's side, as in resolve_one:
//   d = x_j - x_i (minimum image), u = v_j - v_i, t = contact time, w = d + t u,
//   n = w / s, g = u . n, c = m_r (1 + e), J = c g,
//   vi' = v_i + (J/m_i) n,  vj' = v_j - (J/m_j) n,
//   xi' = x_i + t v_i + (dt - t) vi',  xj' = x_j + t v_j + (dt - t) vj'.
// The contact time depends on (d, u) through |d + t u| = s:  dt/dd = -n/g,
// dt/du = -t n/g.  Given the gradients G of the loss with respect to the
// end-of-step state of i and j, the sweep of adjoints below returns the
// gradients with respect to both start states.  The thread of the smaller index
// does the pair: the partner's 14 values lie anywhere in 14 arrays, and reading
// them from one side only, with six scattered writes, beats each thread reading
// the other's (127 us at 1M spheres, 57% of them in pairs).
// Spheres without a collision: x' = x + dt v gives gx = Gx, gv = Gv + dt Gx.
// The e-gradients are summed per workgroup by a fixed tree into epart, one value
// per workgroup, which k_sum_det adds up: one workgroup reading all n of them
// took 243 us at 1M spheres (8 MB through one CU), against 4 us for 3907 sums.
__global__ __launch_bounds__(256) void k_step_backward(int n, const double *x, const double *y,
                                                       const double *z, const double *vx,
                                                       const double *vy, const double *vz,
                                                       const double *r, const double *m, Grid G,
                                                       double dt, double e, const int *partner,
                                                       const double *tcoll, StateGrad gout,
                                                       StateGrad gin, double *epart) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  const double eb = i < n ? backward_sphere(i, x, y, z, vx, vy, vz, r, m, G, dt, e, partner, tcoll,
                                            gout, gin)
                          : 0.0;
  __shared__ double part[256 / WAVE];
  double acc = eb;
  for (int o = WAVE / 2; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
  if (__lane_id() == 0) part[threadIdx.x / WAVE] = acc;
  __syncthreads();
  if (threadIdx.x == 0) epart[blockIdx.x] = (part[0] + part[1]) + (part[2] + part[3]);
}
// deterministic sum of v[0..n) (fixed tree order) added to *out; one block
__global__ __launch_bounds__(1024) void k_sum_det(const double *v, int n, double *out) {
  __shared__ double part[1024];
  double acc = 0.0;
  for (int k = threadIdx.x; k < n; k += 1024) acc += v[k];
  part[threadIdx.x] = acc;
  __syncthreads();
  for (int o = 512; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) part[threadIdx.x] += part[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out += part[0];
}

hipError_t launch_step_backward(hipStream_t s, const Particles &P, const Grid &G, double dt,
                                double e, const int *partner, const double *tcoll,
                                const StateGrad &gout, const StateGrad &gin, double *epart,
                                double *ge) {
  const int n = (int)P.n;
  if (n <= 0) return hipSuccess;
  const int nb = (n + 255) / 256;
  hipLaunchKernelGGL(k_step_backward, dim3(nb), dim3(256), 0, s, n, P.x, P.y, P.z, P.vx, P.vy, P.vz,
                     P.r, P.m, G, dt, e, partner, tcoll, gout, gin, epart);
  hipLaunchKernelGGL(k_sum_det, dim3(1), dim3(1024), 0, s, epart, nb, ge);
  return hipGetLastError();
}

}  // namespace pcol

namespace pcol {

// ---------------------------------------------------------------- batched form

// box id of every sphere (caller order), one workgroup per box
__global__ __launch_bounds__(256) void k_fill_box_of(const int64_t *box_off, int *box_of) {
  const int b = blockIdx.x;
  for (int64_t i = box_off[b] + threadIdx.x; i < box_off[b + 1]; i += 256) box_of[i] = b;
}

hipError_t launch_fill_box_of(hipStream_t s, int nbox, const int64_t *box_off, int *box_of) {
  if (nbox <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_box_of, dim3(nbox), dim3(256), 0, s, box_off, box_of);
  return hipGetLastError();
}

// a1 per box: data validity, reach = 2 max r + 2 max|v| dt (stored), the box
// check L > 2 reach, and whether the planned cells are still at least the reach
// wide (else the host re-plans before any state changes).  Boxes are cut into
// chunks of at most BREACH_CHUNK spheres, one workgroup each, which merge their
// maxima into the box's BoxMax; k_breach_fin then takes one box per thread
// and clears its BoxMax for the next pass.
// BIN: the same pass also takes each sphere's global cell (the box's first
// cell + its cell on the box's planned grid) and its slot in that cell, before
// k_breach_fin has checked the data and the plan: cell coordinates are
// clamped, so every count stays inside the plan's cells, and a failed check
// stops every kernel after it.
template <bool BIN>
__global__ __launch_bounds__(256) void k_breach(Particles P, BatchDev B, int *cid, int *slot,
                                                int *count) {
  const int b = B.chunk_box[blockIdx.x];
  const Grid &G = B.gtab[b];
  const int64_t lo = B.chunk_lo[blockIdx.x];
  const int64_t hi = lo + BREACH_CHUNK < B.box_off[b + 1] ? lo + BREACH_CHUNK : B.box_off[b + 1];
  double v2 = 0.0, rm = 0.0;
  unsigned int bad = 0u;
  for (int64_t i = lo + threadIdx.x; i < hi; i += 256) {
    const double x = P.x[i], y = P.y[i], z = P.z[i];
    const double vx = P.vx[i], vy = P.vy[i], vz = P.vz[i];
    const double r = P.r[i], m = P.m[i];
    const double w = (vx * vx + vy * vy) + vz * vz;
    const bool fin = isfinite(x) && isfinite(y) && isfinite(z) && isfinite(w) && isfinite(r) &&
                     isfinite(m);
    if (!fin || !(r > 0.0) || !(m > 0.0)) bad |= ERR_INVALID;
    if (!(x >= 0.0 && x < G.L[0]) || !(y >= 0.0 && y < G.L[1]) || !(z >= 0.0 && z < G.L[2]))
      bad |= ERR_INVALID;
    if (fin) {
      v2 = w > v2 ? w : v2;
      rm = r > rm ? r : rm;
    }
    if (BIN) {
      const int cx = cell_coord(x, G.inv_h[0], G.nc[0]);
      const int cy = cell_coord(y, G.inv_h[1], G.nc[1]);
      const int cz = cell_coord(z, G.inv_h[2], G.nc[2]);
      const int c = B.cell_base[b] + (cz * G.nc[1] + cy) * G.nc[0] + cx;
      cid[i] = c;
      slot[i] = atomicAdd(&count[c], 1);
    }
  }
  __shared__ double sv[4], sr[4];
  __shared__ unsigned int sb[4];
  for (int o = WAVE / 2; o > 0; o >>= 1) {
    const double a = __shfl_xor(v2, o), c = __shfl_xor(rm, o);
    v2 = a > v2 ? a : v2;
    rm = c > rm ? c : rm;
    bad |= __shfl_xor(bad, o);
  }
  const int w = threadIdx.x / WAVE;
  if (__lane_id() == 0) {
    sv[w] = v2;
    sr[w] = rm;
    sb[w] = bad;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int k = 1; k < 4; ++k) {
      v2 = sv[k] > v2 ? sv[k] : v2;
      rm = sr[k] > rm ? sr[k] : rm;
      bad |= sb[k];
    }
    atomicMax(&B.bmax[b].v2, dbits(v2));
    atomicMax(&B.bmax[b].rm, dbits(rm));
    if (bad) atomicOr(&B.bmax[b].bad, bad);
  }
}

__global__ __launch_bounds__(256) void k_breach_fin(BatchDev B, double dt, int check_plan) {
  const int b = blockIdx.x * 256 + threadIdx.x;
  if (b >= B.nbox) return;
  const BoxMax mx = B.bmax[b];
  B.bmax[b] = BoxMax{0ull, 0ull, 0u, 0u};
  const double v2 = __longlong_as_double((long long)mx.v2);
  const double rm = __longlong_as_double((long long)mx.rm);
  unsigned int bad = mx.bad;
  const Grid &G = B.gtab[b];
  const double reach = 2.0 * rm + 2.0 * sqrt(v2) * dt;
  B.breach[b] = reach;
  for (int a = 0; a < 3; ++a) {
    if (!(G.L[a] > 2.0 * reach)) bad |= ERR_BOX;
    if (check_plan && !(reach * (1.0 + 1e-9) <= G.L[a] / G.nc[a])) bad |= ERR_REPLAN;
  }
  if (bad) atomicOr(&B.flags[FLAG_ERR], bad);
}

hipError_t launch_breach(hipStream_t s, const Particles &P, const BatchDev &B, double dt,
                         int check_plan, int *cid, int *slot, int *count) {
  if (B.nbox <= 0) return hipSuccess;
  if (B.nchunk > 0) {
    if (count)
      hipLaunchKernelGGL(k_breach<true>, dim3(B.nchunk), dim3(256), 0, s, P, B, cid, slot, count);
    else
      hipLaunchKernelGGL(k_breach<false>, dim3(B.nchunk), dim3(256), 0, s, P, B, nullptr, nullptr,
                         nullptr);
  }
  hipLaunchKernelGGL(k_breach_fin, dim3((B.nbox + 255) / 256), dim3(256), 0, s, B, dt, check_plan);
  return hipGetLastError();
}

hipError_t launch_detect_batched(hipStream_t s, const DetectArgs &A, const BatchDev &B,
                                 int total_cells, int cpw) {
  if (cpw < 1 || total_cells <= 0) return cpw < 1 ? hipErrorInvalidValue : hipSuccess;
  hipLaunchKernelGGL(k_detect_batched, dim3((unsigned)((total_cells + cpw - 1) / cpw)), dim3(WAVE),
                     0, s, A, B, cpw);
  return hipGetLastError();
}

}  // namespace pcol

// ---------------------------------------------------------------- deposition
//
// Sec. "Dispersed Phase" (projection operator) and Sec. "Deposition": each
// sphere's source components are imposed linearly on the eight corner nodes of
// its host cell of a periodic Cartesian grid (deposition radius = cell side;
// on equal cells the C0 inverse-distance weights are the trilinear ones), and
// every node receives the sum over spheres.  The paper accumulates with atomic
// adds; on this GPU FP64 atomics to HBM run at about 23e9 per second, so 32 per
// sphere would bound the operator at 0.7e9 spheres/s whatever the memory
// order.  Instead the spheres are counted and scattered by element (a counting
// sort, one integer atomic per sphere), each element sums its spheres' corner
// contributions in caller-index order, and each node adds the corner sums of
// its eight elements in a fixed order, in the shared memory of the workgroup
// that owns the node's tile: no floating-point atomics, and the result is the
// same bit for bit on every run.  Nodes are stored node-major:
// out[node * comp + q], node = (k nc1 + j) nc0 + i; element e has the node of
// the same number as its corner (0, 0, 0).
namespace pcol {

namespace {

// Members of an element are taken in caller-index order (a selection over the
// element's records) up to DEP_SORT_MAX; a larger element sums in scatter
// order.  Up to DEP_REG members the selection runs on caller indices held in
// registers (an element holds 3.9 spheres on average in the 16M workload).
constexpr int DEP_SORT_MAX = 64;
constexpr int DEP_REG = 16;

template <int COMP>
struct alignas(16) DepRec {
  double p[3];
  double a[COMP];
  long long o;  // caller index
};

// Host cell and local coordinate of p on one axis: s = p / h, c = floor(s)
// (at most nc - 1), f = s - c in [0, 1].
__device__ __forceinline__ int dep_cell(double p, double h, int nc, double &f) {
  const double s = p / h;
  int c = (int)floor(s);
  c = c > nc - 1 ? nc - 1 : c;
  f = s - (double)c;
  return c;
}

// Zero element counts, scan words and position flag.
__global__ __launch_bounds__(256) void k_dep_clear(DepositArgs D, int words) {
  const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const int64_t step = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = t; i < D.nnode; i += step) D.cnt[i] = 0;
  for (int64_t i = t; i < words; i += step) D.scan->word[i] = 0ull;
  if (t == 0) {
    D.scan->ticket = 0;
    *D.flag = 0u;
  }
}

// Element of every sphere and its slot among the element's spheres.  A
// position outside [0, L) or not finite raises bit 0 of *flag and is not
// counted (the kernels behind do nothing then).  Consecutive
// lanes of one element (spheres stored in element order) take their slots with
// one atomic per run.
__global__ __launch_bounds__(256) void k_dep_count(DepositArgs D) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int e = -1;  // -1: no element (past the end, or a bad position)
  bool bad = false;
  if (i < D.n) {
    const double p0 = D.x[i], p1 = D.y[i], p2 = D.z[i];
    bad = !(p0 >= 0.0 && p0 < D.L[0]) || !(p1 >= 0.0 && p1 < D.L[1]) ||
          !(p2 >= 0.0 && p2 < D.L[2]);
    if (!bad) {
      double f;
      const int c0 = dep_cell(p0, D.h[0], D.nc[0], f);
      const int c1 = dep_cell(p1, D.h[1], D.nc[1], f);
      const int c2 = dep_cell(p2, D.h[2], D.nc[2], f);
      e = (c2 * D.nc[1] + c1) * D.nc[0] + c0;
    }
  }
  const int lane = (int)__lane_id();
  const unsigned long long badm = __ballot(bad);
  if (badm != 0ull && lane == __ffsll((long long)badm) - 1) atomicOr(D.flag, 1u);
  const int sl = run_slot(e, D.cnt);
  if (e >= 0) {
    D.eid[i] = e;
    D.slot[i] = sl;
  }
}

// one record per sphere at its element-sorted position (caller arrays read
// coalesced)
template <int COMP>
__global__ __launch_bounds__(256) void k_dep_scatter(DepositArgs D) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (D.flag_host && i == 0) *D.flag_host = *D.flag;
  if (*D.flag) return;
  __shared__ Stage<sizeof(DepRec<COMP>) / 16> stage[256 / WAVE];
  DepRec<COMP> r{};
  int pos = -1;
  if (i < D.n) {
    r.p[0] = D.x[i];
    r.p[1] = D.y[i];
    r.p[2] = D.z[i];
#pragma unroll
    for (int q = 0; q < COMP; ++q) r.a[q] = D.a[(int64_t)q * D.n + i];
    r.o = i;
    pos = D.start[D.eid[i]] + D.slot[i];
  }
  store_records(r, pos, reinterpret_cast<DepRec<COMP> *>(D.rec), stage[threadIdx.x / WAVE]);
}

// The eight corner sums of element e's spheres, each a sum in caller-index
// order of w_b a_q with the trilinear weight
// w_b = ((b0 ? f0 : 1 - f0) (b1 ? f1 : 1 - f1)) (b2 ? f2 : 1 - f2).
template <int COMP>
__device__ __forceinline__ void elem_sums(const DepositArgs &D, int64_t e, double (&acc)[8][COMP]) {
  const DepRec<COMP> *R = reinterpret_cast<const DepRec<COMP> *>(D.rec);
  const int m0 = D.start[e], m1 = D.start[e + 1];
  const bool ordered = m1 - m0 <= DEP_SORT_MAX;
#pragma unroll
  for (int b = 0; b < 8; ++b)
#pragma unroll
    for (int q = 0; q < COMP; ++q) acc[b][q] = 0.0;
  auto add = [&](const DepRec<COMP> &r) {
    double f0, f1, f2;
    (void)dep_cell(r.p[0], D.h[0], D.nc[0], f0);
    (void)dep_cell(r.p[1], D.h[1], D.nc[1], f1);
    (void)dep_cell(r.p[2], D.h[2], D.nc[2], f2);
    const double g0 = 1.0 - f0, g1 = 1.0 - f1, g2 = 1.0 - f2;
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const double w = (((b & 1) ? f0 : g0) * ((b & 2) ? f1 : g1)) * ((b & 4) ? f2 : g2);
#pragma unroll
      for (int q = 0; q < COMP; ++q) acc[b][q] += w * r.a[q];
    }
  };
  const int m = m1 - m0;
  if (m <= DEP_REG) {
    int oreg[DEP_REG];  // caller indices (< 2^31) of the members, in slot order
#pragma unroll
    for (int u = 0; u < DEP_REG; ++u) oreg[u] = u < m ? (int)R[m0 + u].o : 0x7fffffff;
    int last = -1;
    for (int t = 0; t < m; ++t) {  // the next caller index after `last`
      int best = 0x7fffffff, k = 0;
#pragma unroll
      for (int u = 0; u < DEP_REG; ++u) {
        const bool take = oreg[u] > last && oreg[u] < best;
        best = take ? oreg[u] : best;
        k = take ? u : k;
      }
      last = best;
      add(R[m0 + k]);
    }
  } else {
    long long last = -1;
    for (int t = m0; t < m1; ++t) {
      int k = t;
      if (ordered) {  // the next caller index after `last`, read from the records
        long long best = 0x7fffffffffffffffll;
        for (int u = m0; u < m1; ++u) {
          const long long o = R[u].o;
          if (o > last && o < best) {
            best = o;
            k = u;
          }
        }
        last = best;
      }
      add(R[k]);
    }
  }
}

// Node sums over a tile of DEP_TN^3 nodes: node (i, j, k) is corner b of
// element (i - b0, j - b1, k - b2) (periodic), and receives the eight corner
// sums in the order b = 0..7.  One thread per element of the tile's
// (DEP_TN + 1)^3 elements (the tile's own and one layer below it on each axis)
// forms its element's eight corner sums; then, phase b after phase b, every
// element adds its corner-b sum to the tile node it touches (within a phase no
// two elements share a node), so each node's sum is formed in the order b =
// 0..7 from zero, with no atomics and no corner-sum array in memory.  The
// elements of the lower layer are summed by two to eight tiles.
constexpr int DEP_TN = 7, DEP_TE = DEP_TN + 1, DEP_TILE_THREADS = DEP_TE * DEP_TE * DEP_TE;

template <int COMP>
__global__ __launch_bounds__(DEP_TILE_THREADS) void k_dep_tile(DepositArgs D, int ntx, int nty) {
  if (*D.flag) return;
  __shared__ double nacc[DEP_TN * DEP_TN * DEP_TN * COMP];
  const int tile = xcd_remap(blockIdx.x, gridDim.x);
  const int tx = tile % ntx, ty = (tile / ntx) % nty, tz = tile / (ntx * nty);
  const int i0 = tx * DEP_TN, j0 = ty * DEP_TN, k0 = tz * DEP_TN;
  const int t = threadIdx.x;
  const int ex = t % DEP_TE, ey = (t / DEP_TE) % DEP_TE, ez = t / (DEP_TE * DEP_TE);
  // the element's global cell, one below the tile's first node on each axis
  auto wrap = [](int c, int nc) { return c < 0 ? c + nc : (c >= nc ? c - nc : c); };
  const int gi = wrap(i0 - 1 + ex, D.nc[0]), gj = wrap(j0 - 1 + ey, D.nc[1]),
            gk = wrap(k0 - 1 + ez, D.nc[2]);
  for (int u = t; u < DEP_TN * DEP_TN * DEP_TN * COMP; u += DEP_TILE_THREADS) nacc[u] = 0.0;
  // every element of the tile's box touches a node of the tile, but past the
  // grid's last cell (a partial tile) it has no node to serve
  const bool live = i0 - 1 + ex < D.nc[0] && j0 - 1 + ey < D.nc[1] && k0 - 1 + ez < D.nc[2];
  double acc[8][COMP];
  if (live) {
    elem_sums<COMP>(D, ((int64_t)gk * D.nc[1] + gj) * D.nc[0] + gi, acc);
  } else {
#pragma unroll
    for (int b = 0; b < 8; ++b)
#pragma unroll
      for (int q = 0; q < COMP; ++q) acc[b][q] = 0.0;
  }
  __syncthreads();
#pragma unroll
  for (int b = 0; b < 8; ++b) {
    const int nx = ex - 1 + (b & 1), ny = ey - 1 + ((b >> 1) & 1), nz = ez - 1 + ((b >> 2) & 1);
    const bool hit = live && nx >= 0 && nx < DEP_TN && ny >= 0 && ny < DEP_TN && nz >= 0 &&
                     nz < DEP_TN && i0 + nx < D.nc[0] && j0 + ny < D.nc[1] && k0 + nz < D.nc[2];
    if (hit) {
      double *a = nacc + ((nz * DEP_TN + ny) * DEP_TN + nx) * COMP;
#pragma unroll
      for (int q = 0; q < COMP; ++q) a[q] += acc[b][q];
    }
    __syncthreads();
  }
  if (t < DEP_TN * DEP_TN * DEP_TN) {
    const int nx = t % DEP_TN, ny = (t / DEP_TN) % DEP_TN, nz = t / (DEP_TN * DEP_TN);
    if (i0 + nx < D.nc[0] && j0 + ny < D.nc[1] && k0 + nz < D.nc[2]) {
      const int64_t n = ((int64_t)(k0 + nz) * D.nc[1] + (j0 + ny)) * D.nc[0] + (i0 + nx);
#pragma unroll
      for (int q = 0; q < COMP; ++q) D.out[n * COMP + q] = nacc[t * COMP + q];
    }
  }
}

template <int COMP>
hipError_t deposit_sorted(hipStream_t s, const DepositArgs &D, hipEvent_t known) {
  const unsigned gn = (unsigned)((D.n + 255) / 256);
  if (D.n > 0) hipLaunchKernelGGL(k_dep_scatter<COMP>, dim3(gn), dim3(256), 0, s, D);
  if (known) {
    const hipError_t e = hipEventRecord(known, s);
    if (e != hipSuccess) return e;
  }
  const int ntx = (D.nc[0] + DEP_TN - 1) / DEP_TN, nty = (D.nc[1] + DEP_TN - 1) / DEP_TN,
            ntz = (D.nc[2] + DEP_TN - 1) / DEP_TN;
  hipLaunchKernelGGL(k_dep_tile<COMP>, dim3((unsigned)(ntx * nty * ntz)), dim3(DEP_TILE_THREADS),
                     0, s, D, ntx, nty);
  return hipGetLastError();
}

}  // namespace

int64_t deposit_record_bytes(int comp) { return ((int64_t)(4 + comp) * 8 + 15) / 16 * 16; }

hipError_t launch_deposit_count(hipStream_t s, const DepositArgs &D) {
  const int words = scan_tiles(D.nnode) + 1;
  hipLaunchKernelGGL(k_dep_clear, dim3(fill_grid(D.nnode)), dim3(256), 0, s, D, words);
  if (D.n > 0)
    hipLaunchKernelGGL(k_dep_count, dim3((unsigned)((D.n + 255) / 256)), dim3(256), 0, s, D);
  return hipGetLastError();
}

hipError_t launch_deposit(hipStream_t s, const DepositArgs &D, hipEvent_t known) {
  switch (D.comp) {
    case 1: return deposit_sorted<1>(s, D, known);
    case 2: return deposit_sorted<2>(s, D, known);
    case 3: return deposit_sorted<3>(s, D, known);
    case 4: return deposit_sorted<4>(s, D, known);
    case 5: return deposit_sorted<5>(s, D, known);
    case 6: return deposit_sorted<6>(s, D, known);
    case 7: return deposit_sorted<7>(s, D, known);
    case 8: return deposit_sorted<8>(s, D, known);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace pcol
