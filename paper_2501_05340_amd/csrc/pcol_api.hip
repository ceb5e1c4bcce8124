// C-ABI layer of the pcol library: argument checks, the context and its
// device scratch, the grid choice, and the sweep driver of pcol_step.
#include <math.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <cstdlib>
#include <fstream>
#include <mutex>
#include <new>
#include <sstream>
#include <string>
#include <vector>

#include "../../include/pcol.h"
#include "pcol_internal.h"

using namespace pcol;

struct pcol_ctx {
  int64_t n_max = 0;
  hipStream_t stream = nullptr;
  pcol_opts opts{};
  std::string err;
  int K = 12;

  // cell-sorted state of the last pcol_bin
  Rec *rec = nullptr;
  int *rank = nullptr;  // caller index -> sorted position
  int *cid = nullptr;
  int *slot = nullptr;
  int *count = nullptr;
  int *start = nullptr;
  ScanState *scan = nullptr;
  int64_t cell_cap = 0;
  bool counts_dirty = false;  // a call stopped between counting the cells and their scan

  // sweep state
  int *cnt = nullptr;
  double *slot_t = nullptr;
  int *slot_j = nullptr;
  int *key_j = nullptr;
  double *key_t = nullptr;
  uint8_t *status = nullptr;
  int *ovf = nullptr;  // spheres with more contacts than slots, then the sweeps' second keys
  int *list_a = nullptr;  // spheres still to act after sweep 1
  OutRec *out = nullptr;
  int *partner_tmp = nullptr;
  double *tcoll_tmp = nullptr;
  ReachScratch reach{};
  SweepCounters *ctr_d = nullptr;
  StepPlan *plan_d = nullptr;  // the plan of the last binning, made on the device,
  StepPlan *plan_h = nullptr;  // and in page-locked host memory
  StepReport *rep = nullptr;  // page-locked host memory that the step's last kernel writes
  int exact_sweeps = 0;       // some step's contacts overflowed the slots: sweeps that can search
  int sweep_guess = 5;        // sweeps the last step took: so many are queued, and one more
  hipEvent_t ev[8] = {};

  bool binned = false;
  int64_t binned_n = -1;
  double binned_dt = 0.0;
  StepPlan plan{};                 // the last binning's, once the host has waited for it
  const Spin *spin = nullptr;      // set by pcol_step_spin for the step: its spins are validated
  int walls = 0;                   // set by pcol_step_walls for the step: bit k = walls on axis k
  // pcol_deposit: position check flag, and the element sort's scratch with its capacities
  unsigned int *dep_flag_h = nullptr;
  hipEvent_t dep_known = nullptr;      // the flag has been written
  hipStream_t dep_stream = nullptr;    // of the last deposition, whose node sums may still run
  unsigned char *dep_buf = nullptr;  // carved by deposit_layout
  int64_t dep_cap = 0;
  // The last two plans of a shape (sphere count, box, step, walls): the kernels of
  // a step are sized by the last one, and if both gave one grid the reach pass of
  // a large step counts the spheres on it.
  bool shape_valid = false, steady = false;
  bool many_cells = false;  // some plan of the shape was not one for k_bin_small
  bool split_seen = false;  // some plan of the shape split: the wide search is queued every time
  int64_t shape_n = -1;
  double shape_L[3] = {0, 0, 0}, shape_dt = 0.0;
  int shape_walls = 0;
  bool detect_timed = false;
  unsigned long long *crank = nullptr;  // literal order (opts.order = 1): curve rank per sorted sphere
  struct BatchPlan *bp = nullptr;  // batched form (pcol_step_batched)
};

// State of the batched form: per-box grids on the host and device, the
// captured step graph and what it was captured for.
struct BatchPlan {
  // layout the tables were built for
  int nbox = 0;
  int64_t n = 0;
  std::vector<int64_t> box_off;
  std::vector<double> len;  // 3 per box
  // device tables
  Grid *gtab = nullptr;
  int *cell_base = nullptr;
  int *box_of = nullptr;
  int64_t *box_off_d = nullptr;
  double *breach = nullptr;
  int *chunk_box = nullptr;               // chunks of the reach pass (BREACH_CHUNK spheres)
  int64_t *chunk_lo = nullptr;
  BoxMax *bmax = nullptr;                 // [nbox], zero between passes
  int nchunk = 0, cap_chunk = 0;
  std::vector<int> chunk_box_h;
  std::vector<int64_t> chunk_lo_h;
  unsigned int *flags = nullptr;          // FLAG_* words
  int cap_box = 0;
  int64_t cap_n = 0;
  unsigned int *flags_h = nullptr;        // pinned read-back of the flags
  std::vector<double> breach_h;
  std::vector<Grid> gtab_h;
  std::vector<int> cell_base_h;
  int total_cells = 0;
  bool tables = false;  // grids planned for the current layout
  // tuning choice
  double cell_mult = 1.0;
  int cpw = 4;           // home cells per workgroup of the pair-test launch
  bool tuned = false;
  int kmax = 12;        // sweeps captured in the graph
  // captured graph and its arguments
  hipStream_t gstream = nullptr;
  hipGraphExec_t exec = nullptr;
  bool captured = false;
  int cap_exact = 0;  // its sweeps can search
  const void *cap_ptr[8] = {};
  const void *cap_part = nullptr, *cap_tc = nullptr;
  double cap_dt = 0.0, cap_e = 0.0;
  // tuning scratch
  double *tune_buf = nullptr;
  int64_t tune_cap = 0;
};

namespace {

pcol_status fail(pcol_ctx *c, pcol_status st, const char *what) {
  if (c) c->err = what;
  return st;
}

pcol_status hip_fail(pcol_ctx *c, hipError_t e, const char *where) {
  if (c) {
    c->err = std::string(where) + ": " + hipGetErrorString(e);
  }
  return PCOL_E_HIP;
}

#define PCOL_HIP(call)                                   \
  do {                                                   \
    hipError_t e_ = (call);                              \
    if (e_ != hipSuccess) return hip_fail(ctx, e_, #call); \
  } while (0)

template <typename T>
hipError_t dalloc(T **p, size_t count) {
  return hipMalloc((void **)p, (count ? count : 1) * sizeof(T));
}

bool finite_pos(double v) { return isfinite(v) && v > 0.0; }

pcol_status check_common(pcol_ctx *ctx, const pcol_particles *p, const pcol_box *box, double dt) {
  if (!ctx) return PCOL_E_INVALID;
  if (!p || !box) return fail(ctx, PCOL_E_INVALID, "null particles or box");
  if (p->n < 0 || p->n > ctx->n_max) return fail(ctx, PCOL_E_INVALID, "n outside [0, n_max]");
  if (p->n > 0 && (!p->x || !p->y || !p->z || !p->vx || !p->vy || !p->vz || !p->r || !p->m))
    return fail(ctx, PCOL_E_INVALID, "null particle array");
  for (int a = 0; a < 3; ++a)
    if (!finite_pos(box->len[a])) return fail(ctx, PCOL_E_INVALID, "box side not finite positive");
  if (!finite_pos(dt)) return fail(ctx, PCOL_E_INVALID, "dt not finite positive");
  return PCOL_OK;
}

Particles to_dev(const pcol_particles *p) {
  Particles P;
  P.n = p->n;
  P.x = p->x;
  P.y = p->y;
  P.z = p->z;
  P.vx = p->vx;
  P.vy = p->vy;
  P.vz = p->vz;
  P.r = p->r;
  P.m = p->m;
  return P;
}

// (re)allocate *p for at least `want` elements when its capacity `cap` is short
template <typename T>
hipError_t grow(T **p, int64_t &cap, int64_t want) {
  if (*p && cap >= want) return hipSuccess;
  if (*p) (void)hipFree(*p);
  *p = nullptr;
  cap = 0;
  const hipError_t e = hipMalloc((void **)p, (size_t)(want > 0 ? want : 1) * sizeof(T));
  if (e == hipSuccess) cap = want;
  return e;
}

double ms_between(hipEvent_t a, hipEvent_t b) {
  float ms = 0.f;
  if (hipEventElapsedTime(&ms, a, b) != hipSuccess) return 0.0;
  return (double)ms;
}

// ---------------------------------------------------------------- deposition scratch

// The deposition's scratch carved out of one buffer, each part on a 256-B
// boundary: element id and slot per sphere, the element-sorted records, the
// per-element counts and starts, the scan's words and the position flag.
struct DepositLayout {
  int64_t eid, slot, rec, cnt, start, scan, flag, bytes;
};

DepositLayout deposit_layout(int64_t n, int64_t ne, int comp) {
  DepositLayout L{};
  int64_t at = 0;
  auto take = [&at](int64_t bytes) {
    const int64_t here = at;
    at += (bytes + 255) / 256 * 256;
    return here;
  };
  L.eid = take(n * (int64_t)sizeof(int));
  L.slot = take(n * (int64_t)sizeof(int));
  L.rec = take(n * deposit_record_bytes(comp));
  L.cnt = take((ne + 1) * (int64_t)sizeof(int));
  L.start = take((ne + 1) * (int64_t)sizeof(int));
  // 8 bytes a tile; not less than the 4 bytes a tile and 8,232 that the size limit
  // of the fixed scratch is stated with
  const int64_t words = (ne / SCAN_B + 2) * 8 + (int64_t)sizeof(ScanState);
  const int64_t least = ((ne / 4096 + 2) * 4 + 255) / 256 * 256 + 8448;
  L.scan = take(words > least ? words : least);
  L.flag = take((int64_t)sizeof(unsigned int));
  L.bytes = at;
  return L;
}

// Argument checks of the deposition (no device access); fills D but its
// scratch pointers.
pcol_status deposit_args(const double *x, const double *y, const double *z, int64_t n,
                         const double *a, int comp, const int32_t nc[3], const double len[3],
                         double *out, DepositArgs &D, const char *&why) {
  if (n < 0 || n > INT32_MAX) return why = "n outside [0, 2^31 - 1]", PCOL_E_INVALID;
  if (comp < 1 || comp > 8) return why = "comp outside [1, 8]", PCOL_E_INVALID;
  if (!nc || !len || !out) return why = "null grid or output", PCOL_E_INVALID;
  if (n > 0 && (!x || !y || !z || !a)) return why = "null array", PCOL_E_INVALID;
  D.x = x;
  D.y = y;
  D.z = z;
  D.a = a;
  D.n = n;
  D.comp = comp;
  D.out = out;
  D.nnode = 1;
  for (int d = 0; d < 3; ++d) {
    if (nc[d] < 1 || nc[d] > (1 << 20)) return why = "nc outside [1, 2^20]", PCOL_E_INVALID;
    if (!(len[d] > 0.0) || !isfinite(len[d])) return why = "box side <= 0", PCOL_E_INVALID;
    D.nc[d] = nc[d];
    D.L[d] = len[d];
    D.h[d] = len[d] / nc[d];
    D.nnode *= nc[d];
    if (D.nnode > INT32_MAX) return why = "more than 2^31 - 1 elements", PCOL_E_INVALID;
  }
  return PCOL_OK;
}

// The deposition on stream s with its scratch at base (laid out by Lo).  The count
// checks every position, and the kernels behind it do nothing if one is bad, so
// all are queued at once and the flag is read behind them (into flag_h, host
// memory); st receives PCOL_E_INVALID for a bad position, else PCOL_OK.  known
// given: flag_h is page-locked, the scatter writes it, and the host waits for this
// event behind the scatter only, not for the node sums (waiting for them too, 300,000
// spheres onto 32^3 elements took 174 us a call among others, now 156, and a caller
// could do nothing meanwhile).
hipError_t deposit_run(DepositArgs &D, const DepositLayout &Lo, unsigned char *base, hipStream_t s,
                       unsigned int *flag_h, hipEvent_t known, pcol_status &st) {
  st = PCOL_OK;
  D.eid = (int *)(base + Lo.eid);
  D.slot = (int *)(base + Lo.slot);
  D.rec = base + Lo.rec;
  D.cnt = (int *)(base + Lo.cnt);
  D.start = (int *)(base + Lo.start);
  D.scan = (ScanState *)(base + Lo.scan);
  D.flag = (unsigned int *)(base + Lo.flag);
  D.flag_host = known ? flag_h : nullptr;
  hipError_t e = launch_deposit_count(s, D);
  if (e == hipSuccess)
    e = launch_scan(s, D.cnt, (int)D.nnode, nullptr, D.start, D.scan, nullptr, false);
  if (e == hipSuccess) e = launch_deposit(s, D, D.n > 0 ? known : nullptr);
  if (e != hipSuccess || D.n == 0) return e;
  if (known) {
    e = hipEventSynchronize(known);
  } else {
    e = hipMemcpyAsync(flag_h, D.flag, sizeof(unsigned int), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
  }
  if (e == hipSuccess && *flag_h) st = PCOL_E_INVALID;
  return e;
}

}  // namespace

// ---------------------------------------------------------------- static scratch

// Device scratch of pcol_deposit_noalloc: one copy per GPU, held until the
// process ends.  Host code never passes `scratch` itself to a kernel (its host
// name is a stand-in, not a device address): the device address of each GPU's
// copy comes from hipGetSymbolAddress, taken once per device on the first call
// with that device current.
static __device__ __align__(256) unsigned char scratch[PCOL_NOALLOC_SCRATCH_BYTES];

static constexpr int MAX_DEVICES = 64;
static std::mutex scratch_mu;
static unsigned char *scratch_ptr[MAX_DEVICES] = {};

static hipError_t static_scratch(unsigned char **out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= MAX_DEVICES) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(scratch_mu);
  if (!scratch_ptr[dev]) {
    void *p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    scratch_ptr[dev] = (unsigned char *)p;
  }
  *out = scratch_ptr[dev];
  return hipSuccess;
}


extern "C" {

void pcol_default_opts(pcol_opts *o) {
  if (!o) return;
  memset(o, 0, sizeof(*o));
  o->cell_mult = 1.0;
  o->max_sweeps = 0;
  o->home_cells = 0;
  o->contact_slots = 12;
  o->filter = 0;
  o->band_rel = 1e-4;
  o->timing = 0;
  o->autotune = 1;
  o->split_quantile = 0.999;
  o->order = 0;
}

const char *pcol_last_error(const pcol_ctx *ctx) {
  if (!ctx) return "null context";
  return ctx->err.c_str();
}

pcol_status pcol_set_stream(pcol_ctx *ctx, void *hip_stream) {
  if (!ctx) return PCOL_E_INVALID;
  ctx->stream = (hipStream_t)hip_stream;
  return PCOL_OK;
}

void pcol_destroy(pcol_ctx *ctx) {
  if (!ctx) return;
  void *dev[] = {ctx->rec,    ctx->rank,   ctx->cid,         ctx->slot,
                 ctx->count,  ctx->start,  ctx->scan, ctx->cnt,      ctx->slot_t,
                 ctx->slot_j, ctx->key_j,  ctx->key_t,  ctx->status,      ctx->out,
                 ctx->ovf,    ctx->partner_tmp, ctx->tcoll_tmp, ctx->list_a,
                 ctx->ctr_d, ctx->dep_buf, ctx->crank, ctx->reach.parts, ctx->reach.hist,
                 ctx->plan_d};
  for (void *p : dev)
    if (p) (void)hipFree(p);
  if (ctx->plan_h) (void)hipHostFree(ctx->plan_h);
  if (ctx->rep) (void)hipHostFree(ctx->rep);
  if (ctx->dep_flag_h) (void)hipHostFree(ctx->dep_flag_h);
  if (ctx->dep_known) (void)hipEventDestroy(ctx->dep_known);
  for (hipEvent_t &e : ctx->ev)
    if (e) (void)hipEventDestroy(e);
  if (BatchPlan *bp = ctx->bp) {
    void *bd[] = {bp->gtab,    bp->cell_base, bp->box_of, bp->box_off_d, bp->breach,
                  bp->chunk_box, bp->chunk_lo, bp->bmax,  bp->flags,     bp->tune_buf};
    for (void *q : bd)
      if (q) (void)hipFree(q);
    if (bp->flags_h) (void)hipHostFree(bp->flags_h);
    if (bp->exec) (void)hipGraphExecDestroy(bp->exec);
    if (bp->gstream) (void)hipStreamDestroy(bp->gstream);
    delete bp;
  }
  delete ctx;
}

pcol_status pcol_create(pcol_ctx **out, int64_t n_max, void *hip_stream, const pcol_opts *opts) {
  if (!out) return PCOL_E_INVALID;
  *out = nullptr;
  if (n_max < 0 || n_max > 0x7fffffffLL) return PCOL_E_INVALID;
  pcol_ctx *ctx = new (std::nothrow) pcol_ctx();
  if (!ctx) return PCOL_E_NOMEM;
  pcol_default_opts(&ctx->opts);
  if (opts) ctx->opts = *opts;
  if (!(ctx->opts.cell_mult >= 1.0) || !isfinite(ctx->opts.cell_mult) ||
      ctx->opts.max_sweeps < 0 || ctx->opts.contact_slots < 0 || ctx->opts.contact_slots > 64 ||
      ctx->opts.home_cells < 0 || ctx->opts.home_cells > 16 ||
      ctx->opts.order < 0 || ctx->opts.order > 1 ||
      !(ctx->opts.band_rel >= 0.0) ||
      !(ctx->opts.split_quantile >= 0.0 && ctx->opts.split_quantile <= 1.0) ||
      ctx->opts.filter < 0 || ctx->opts.filter > 1) {
    delete ctx;
    return PCOL_E_INVALID;
  }
  ctx->K = ctx->opts.contact_slots > 0 ? ctx->opts.contact_slots : 12;
  ctx->n_max = n_max;
  ctx->stream = (hipStream_t)hip_stream;
  const size_t n = (size_t)n_max;
  hipError_t e = hipSuccess;
  auto A = [&](hipError_t r) {
    if (e == hipSuccess && r != hipSuccess) e = r;
  };
  const size_t lists = n + (size_t)(NSHARD + 1) * 256;  // every shard has whole workgroups
  A(dalloc(&ctx->rec, n));
  A(dalloc(&ctx->rank, n));
  A(dalloc(&ctx->cid, lists));
  A(dalloc(&ctx->slot, n));
  A(dalloc(&ctx->cnt, n));
  A(dalloc(&ctx->slot_t, n * (size_t)ctx->K));
  A(dalloc(&ctx->slot_j, n * (size_t)ctx->K));
  A(dalloc(&ctx->key_j, n));
  A(dalloc(&ctx->key_t, n));
  A(dalloc(&ctx->status, n));
  A(dalloc(&ctx->out, n));
  A(dalloc(&ctx->ovf, n));
  A(dalloc(&ctx->list_a, lists));
  A(dalloc(&ctx->partner_tmp, n));
  A(dalloc(&ctx->tcoll_tmp, n));
  if (ctx->opts.order == 1) A(dalloc(&ctx->crank, n));
  A(dalloc(&ctx->plan_d, 1));
  A(dalloc(&ctx->reach.parts, REACH_BLOCKS));
  A(dalloc(&ctx->reach.hist, RHO_BINS));
  A(dalloc(&ctx->ctr_d, 1));
  if (e == hipSuccess) e = hipHostMalloc((void **)&ctx->plan_h, sizeof(StepPlan));
  if (e == hipSuccess) e = hipHostMalloc((void **)&ctx->rep, sizeof(StepReport));
  for (hipEvent_t &ev : ctx->ev)
    if (e == hipSuccess) e = hipEventCreate(&ev);
  if (e != hipSuccess) {
    pcol_destroy(ctx);
    return e == hipErrorOutOfMemory ? PCOL_E_NOMEM : PCOL_E_HIP;
  }
  *out = ctx;
  return PCOL_OK;
}

// The cell arrays for `cells` cells (of both layers), with room for a grid a
// little finer; the counts start at zero, and so does the extent histogram with
// the first ones (a context that only deposits needs none of them: clearing the
// histogram in pcol_create, and waiting for that, took 50 us).
static pcol_status grow_cells(pcol_ctx *ctx, int64_t cells) {
  if (cells + 2 <= ctx->cell_cap) return PCOL_OK;
  const bool first = ctx->cell_cap == 0;
  PCOL_HIP(hipStreamSynchronize(ctx->stream));
  if (ctx->count) (void)hipFree(ctx->count);
  if (ctx->start) (void)hipFree(ctx->start);
  if (ctx->scan) (void)hipFree(ctx->scan);
  ctx->count = ctx->start = nullptr;
  ctx->scan = nullptr;
  ctx->cell_cap = 0;
  if (ctx->bp) ctx->bp->captured = false;  // its graph holds the old cell arrays
  const int64_t cap = cells + cells / 4 + 64;
  hipError_t e = dalloc(&ctx->count, (size_t)cap);
  if (e == hipSuccess) e = dalloc(&ctx->start, (size_t)cap + 1);
  if (e == hipSuccess)
    e = hipMalloc((void **)&ctx->scan, sizeof(ScanState) + (size_t)(cap / SCAN_B + 2) * 8);
  if (e == hipSuccess) e = hipMemsetAsync(ctx->count, 0, (size_t)cap * sizeof(int), ctx->stream);
  if (e == hipSuccess)
    e = hipMemsetAsync(ctx->scan, 0, sizeof(ScanState) + (size_t)(cap / SCAN_B + 2) * 8,
                       ctx->stream);
  if (e == hipSuccess && first)
    e = hipMemsetAsync(ctx->reach.hist, 0, RHO_BINS * sizeof(unsigned int), ctx->stream);
  if (e != hipSuccess) return fail(ctx, PCOL_E_NOMEM, "cell arrays");
  ctx->cell_cap = cap;
  ctx->counts_dirty = false;
  return PCOL_OK;
}

static bool same_grid(const StepPlan &a, const StepPlan &b) {
  return a.G.nc[0] == b.G.nc[0] && a.G.nc[1] == b.G.nc[1] && a.G.nc[2] == b.G.nc[2] &&
         a.G.layer2 == b.G.layer2 && (!a.split || a.rho_c == b.rho_c);
}

// The host's turn after a wait: the plan's verdict and, if it stands, the plan.
static pcol_status take_plan(pcol_ctx *ctx) {
  const unsigned int err = ctx->plan_h->err;
  if (err & PLAN_INVALID) return fail(ctx, PCOL_E_INVALID, "non-finite value, r <= 0 or m <= 0");
  if (err & PLAN_POSITION) return fail(ctx, PCOL_E_INVALID, "position outside [0, L)");
  if (err & PLAN_BOX)
    return fail(ctx, PCOL_E_BOX, "box side <= 2 * reach: minimum image not unique");
  ctx->steady = ctx->shape_valid && same_grid(ctx->plan, *ctx->plan_h);
  ctx->plan = *ctx->plan_h;
  ctx->shape_valid = true;
  ctx->split_seen = ctx->split_seen || ctx->plan.split;
  ctx->binned = true;
  return PCOL_OK;
}

// Enqueue the binning of p.  ahead: everything at once, for a caller that looks
// at the plan after its next wait (take_plan; PLAN_AGAIN asks it to bin once more
// without `ahead`), if the last call says how large the kernels behind the plan
// have to be: the same shape and no small grid, whose kernels are others.
// Otherwise (ahead then false) it waits for the plan, checks it and makes room for
// its cells before it queues the rest.
// few: let one workgroup bin the box if that can be done ahead (then still set).
static pcol_status bin_queue(pcol_ctx *ctx, const pcol_particles *p, const pcol_box *box, double dt,
                             bool &ahead, bool &few) {
  ctx->binned = false;
  Particles P = to_dev(p);
  if (ctx->spin) {
    P.wx = ctx->spin->wx;
    P.wy = ctx->spin->wy;
    P.wz = ctx->spin->wz;
  }
  hipStream_t s = ctx->stream;
  // room for a usual grid: a cell holds some 13 spheres, and a split grid has two layers
  if (ctx->cell_cap == 0) {
    const pcol_status st = grow_cells(ctx, p->n / 4);
    if (st != PCOL_OK) return st;
  }
  if (ctx->counts_dirty) {
    PCOL_HIP(hipMemsetAsync(ctx->count, 0, (size_t)ctx->cell_cap * sizeof(int), s));
    ctx->counts_dirty = false;
  }
  const bool shape = ctx->shape_valid && ctx->shape_n == p->n && ctx->shape_dt == dt &&
                     ctx->shape_walls == ctx->walls && ctx->shape_L[0] == box->len[0] &&
                     ctx->shape_L[1] == box->len[1] && ctx->shape_L[2] == box->len[2];
  if (!shape) ctx->shape_valid = ctx->steady = ctx->split_seen = ctx->many_cells = false;
  ahead = ahead && ctx->shape_valid && !ctx->plan.small && p->n > 0;
  ctx->shape_n = p->n;
  ctx->shape_dt = dt;
  ctx->shape_walls = ctx->walls;
  for (int a = 0; a < 3; ++a) ctx->shape_L[a] = box->len[a];
  ctx->binned_n = p->n;
  ctx->binned_dt = dt;
  PlanArgs A{};
  A.n = p->n;
  A.cell_cap = ctx->cell_cap;
  for (int a = 0; a < 3; ++a) A.L[a] = box->len[a];
  A.dt = dt;
  A.cell_mult = ctx->opts.cell_mult;
  A.band_rel = ctx->opts.band_rel;
  A.quantile = ctx->opts.split_quantile;
  A.home_cells = ctx->opts.home_cells;
  A.fp32 = ctx->opts.filter == 1;
  A.walls = ctx->walls;
  A.curve = ctx->opts.order == 1;
  A.allow_small = !ahead;
  A.allow_split = !ahead || ctx->split_seen;
  A.tried_rho_c = INFINITY;
  // Counting in the reach pass saves reading the spheres once more (0.66 ms for both
  // at 16M spheres in random order, against 0.22 + 0.64 apart) but is thrown away
  // if the grid changes, so only where the last two steps had the same one, and
  // where a pass over the spheres costs more than a launch.  It pays where the state
  // is restored or changes little: in a box of 1M spheres that goes on, whose grid
  // follows its fastest sphere, two equal grids in a row say little, and the counts of
  // every second step are thrown away (60 + 43 us, against 27 + 43; 18 us of a step's
  // 410).
  const bool tried = ctx->steady && p->n >= (1 << 18) && ctx->plan.cells + 2 <= ctx->cell_cap;
  const StepPlan last = ctx->plan;
  if (tried) {
    A.tried = 1;
    for (int a = 0; a < 3; ++a) A.tried_nc[a] = last.G.nc[a];
    A.tried_layer2 = last.G.layer2;
    A.tried_rho_c = last.rho_c;
  }
  // the extent histogram only picks the split extent: above 2^20 spheres it
  // samples one sphere in 16 (the quantile of a million samples is as good)
  const int hist_shift = p->n >= (1 << 20) ? 4 : 0;
  few = few && ahead && !ctx->many_cells;
  if (few) {  // counts in LDS: the context's stay clean
    A.allow_split = 0;
    PCOL_HIP(launch_bin_small(s, P, A, ctx->ctr_d, ctx->plan_d, ctx->plan_h, ctx->start, ctx->rec,
                              ctx->rank, ctx->cnt, ctx->crank));
    return PCOL_OK;
  }
  ctx->counts_dirty = true;  // until the scan is queued behind a plan that stands
  if (tried)
    PCOL_HIP(launch_reach(s, P, dt, hist_shift, A, ctx->reach, ctx->ctr_d, ctx->scan, ctx->plan_d,
                          ctx->plan_h, &last.G, last.rho_c, ctx->cid, ctx->slot, ctx->count));
  else
    PCOL_HIP(launch_reach(s, P, dt, hist_shift, A, ctx->reach, ctx->ctr_d, ctx->scan, ctx->plan_d,
                          ctx->plan_h));
  int cells = last.cells;
  if (!ahead) {
    PCOL_HIP(hipStreamSynchronize(s));
    if (ctx->plan_h->err == PLAN_AGAIN) {  // more cells than there is room for
      const pcol_status st = grow_cells(ctx, ctx->plan_h->cells);
      if (st != PCOL_OK) return st;
      ctx->steady = false;
      return bin_queue(ctx, p, box, dt, ahead, few);
    }
    const pcol_status st = take_plan(ctx);
    if (st != PCOL_OK) return st;
    cells = ctx->plan.cells;
  }
  // a2-a4: counting sort into cell-sorted records
  PCOL_HIP(launch_cell_hist(s, P, ctx->plan_d, dt, tried ? last.cells : 0, ctx->cid, ctx->slot,
                            ctx->count));
  PCOL_HIP(launch_scan(s, ctx->count, cells, ctx->plan_d, ctx->start, ctx->scan,
                       &ctx->ctr_d->maxcell, true));
  ctx->counts_dirty = ahead;
  PCOL_HIP(launch_scatter(s, P, ctx->cid, ctx->slot, ctx->start, ctx->rec, ctx->rank, ctx->cnt,
                          nullptr, &ctx->plan_d->err));
  if (ctx->opts.order == 1)
    PCOL_HIP(launch_curve_rank(s, ctx->rec, (int)p->n, ctx->plan_d, ctx->crank));
  return PCOL_OK;
}

pcol_status pcol_bin(pcol_ctx *ctx, const pcol_particles *p, const pcol_box *box, double dt) {
  pcol_status st = check_common(ctx, p, box, dt);
  if (st != PCOL_OK) return st;
  bool ahead = false, few = false;
  return bin_queue(ctx, p, box, dt, ahead, few);
}

static pcol_status check_binned(pcol_ctx *ctx, const pcol_particles *p, const pcol_box *box,
                                double dt) {
  if (!ctx->binned || ctx->binned_n != p->n)
    return fail(ctx, PCOL_E_STATE, "pcol_bin must run first on the same particle set");
  if (ctx->plan.G.walls) return fail(ctx, PCOL_E_STATE, "the last binning was for a box with walls");
  if (dt != ctx->binned_dt) return fail(ctx, PCOL_E_STATE, "dt differs from pcol_bin");
  for (int a = 0; a < 3; ++a)
    if (box->len[a] != ctx->plan.G.L[a]) return fail(ctx, PCOL_E_STATE, "box differs from pcol_bin");
  return PCOL_OK;
}

// sweep 1: keys of all spheres (all active) into ctx->key_j / key_t (sorted
// order); crank given: the literal order's partners instead of rule 2's
// The spheres whose contacts overflowed their slots get no key (overflow_search).
// contacts_only: the pair tests alone; masked: if a masked detect takes them.
static pcol_status detect_all(pcol_ctx *ctx, double dt, const unsigned long long *crank,
                              bool contacts_only = false, bool masked = false) {
  hipStream_t s = ctx->stream;
  const int n = (int)ctx->binned_n;
  // sized by the last plan that the host has seen: this binning's, or for a step
  // that has not waited yet the one before it (which then had no small grid, and
  // some plan of the shape a split one if this one has)
  const StepPlan &pl = ctx->plan;
  const unsigned int *err = &ctx->plan_d->err;
  const Grid *G = &ctx->plan_d->G;
  if (!pl.small) {
    DetectArgs A{};
    A.rec = ctx->rec;
    A.start = ctx->start;
    A.cnt = ctx->cnt;
    A.slot_t = ctx->slot_t;
    A.slot_j = ctx->slot_j;
    A.ctr = ctx->ctr_d;
    A.n = n;
    A.K = ctx->K;
    A.plan = ctx->plan_d;
    A.err = err;
    A.masked = masked;
    A.dt = dt;
    A.dt2 = 2.0 * dt * (1.0 + 0x1.0p-20);
    if (ctx->opts.timing) PCOL_HIP(hipEventRecord(ctx->ev[5], s));
    PCOL_HIP(launch_detect_half(s, A, ctx->opts.filter == 1,
                                (pl.G.ncell + pl.cpw - 1) / (pl.cpw > 0 ? pl.cpw : 1)));
    // spheres of large extent: exact search of their wider neighbourhood
    if (ctx->split_seen) PCOL_HIP(launch_detect_wide(s, A));
    if (ctx->opts.timing) PCOL_HIP(hipEventRecord(ctx->ev[6], s));
    ctx->detect_timed = true;
    if (contacts_only) return PCOL_OK;
    PCOL_HIP(launch_slot_min(s, n, ctx->cnt, ctx->slot_t, ctx->slot_j, ctx->K, ctx->rec,
                             ctx->key_j, ctx->key_t, ctx->ovf, ctx->ctr_d, err, G, crank));
  } else {
    // fewer than 3 cells on some axis: exact search for every sphere
    PCOL_HIP(launch_gather_exact(s, nullptr, n, nullptr, ctx->rec, ctx->start, G, dt, ctx->key_j,
                                 ctx->key_t, nullptr, err, crank));
  }
  return PCOL_OK;
}

// Keys, by the exact search, of the spheres that detect_all left out.
static pcol_status overflow_search(pcol_ctx *ctx, double dt, const unsigned long long *crank) {
  PCOL_HIP(launch_gather_exact(ctx->stream, ctx->ovf, (int)ctx->binned_n, &ctx->ctr_d->n_overflow,
                               ctx->rec, ctx->start, &ctx->plan_d->G, dt, ctx->key_j, ctx->key_t,
                               nullptr, &ctx->plan_d->err, crank));
  return PCOL_OK;
}

pcol_status pcol_detect(pcol_ctx *ctx, const pcol_particles *p, const pcol_box *box, double dt,
                        const uint8_t *active, uint64_t *key_out, double *tmin_out) {
  pcol_status st = check_common(ctx, p, box, dt);
  if (st != PCOL_OK) return st;
  if ((st = check_binned(ctx, p, box, dt)) != PCOL_OK) return st;
  if (p->n > 0 && !key_out) return fail(ctx, PCOL_E_INVALID, "key_out is null");
  hipStream_t s = ctx->stream;
  const int n = (int)p->n;
  if (n == 0) return PCOL_OK;
  if (!active) {
    // cleared by kernels: the call waits for nothing, so a caller may capture it, and
    // memset nodes of a graph are not relied on
    PCOL_HIP(launch_fill_u32(s, (unsigned int *)ctx->ctr_d, 0u, sizeof(SweepCounters) / 4));
    PCOL_HIP(launch_fill_i32(s, ctx->cnt, 0, n));
    if ((st = detect_all(ctx, dt, nullptr)) != PCOL_OK) return st;
    if (!ctx->plan.small && (st = overflow_search(ctx, dt, nullptr)) != PCOL_OK) return st;
  } else {
    // the pair tests of all spheres if many of them are active, else the exact search
    // of each active one: the device decides.  The search alone on a small grid, and
    // below SMALL_N spheres, where the launches count: 19 us at 3,000 spheres with few
    // active and 25 with all, against 21 for either with the pair tests queued before it
    // (10,000: 19 and 49, against 21 and 22).
    const bool pairs = !ctx->plan.small && n >= SMALL_N;
    PCOL_HIP(launch_status_from_active(s, active, ctx->rec, n, ctx->status, ctx->cnt, ctx->ctr_d));
    if (pairs && (st = detect_all(ctx, dt, nullptr, true, true)) != PCOL_OK) return st;
    PCOL_HIP(launch_masked_keys(s, ctx->ctr_d, n, pairs, ctx->K, ctx->cnt, ctx->slot_t, ctx->slot_j,
                                ctx->rec, ctx->start, &ctx->plan_d->G, dt, ctx->status, ctx->key_j,
                                ctx->key_t));
  }
  PCOL_HIP(launch_export_keys(s, n, ctx->rec, ctx->key_j, ctx->key_t,
                              active ? ctx->status : nullptr, ctx->ctr_d, key_out, tmin_out));
  return PCOL_OK;
}

pcol_status pcol_resolve(pcol_ctx *ctx, pcol_particles *p, const pcol_box *box, double dt,
                         double e, const uint64_t *key, uint8_t *active, int32_t *partner,
                         double *tcoll, int64_t *n_pairs_dev) {
  pcol_status st = check_common(ctx, p, box, dt);
  if (st != PCOL_OK) return st;
  if (!(e >= 0.0 && e <= 1.0)) return fail(ctx, PCOL_E_INVALID, "e outside [0, 1]");
  if ((st = check_binned(ctx, p, box, dt)) != PCOL_OK) return st;
  if (p->n > 0 && (!key || !active)) return fail(ctx, PCOL_E_INVALID, "key or active is null");
  PCOL_HIP(launch_resolve_public(ctx->stream, (int)p->n, ctx->rec, ctx->rank, ctx->plan.G, dt, e, key,
                                 to_dev(p), active, partner, tcoll, (long long *)n_pairs_dev));
  return PCOL_OK;
}

pcol_status pcol_advance(pcol_ctx *ctx, pcol_particles *p, const pcol_box *box, double dt,
                         const int32_t *partner) {
  pcol_status st = check_common(ctx, p, box, dt);
  if (st != PCOL_OK) return st;
  if (p->n > 0 && !partner) return fail(ctx, PCOL_E_INVALID, "partner is null");
  PCOL_HIP(launch_advance(ctx->stream, to_dev(p), partner, dt, box->len));
  return PCOL_OK;
}

}  // extern "C"

// What the sweeps of a step need from the context.
static SweepArgs sweep_args(const pcol_ctx *ctx, const Particles &P, double dt, double e) {
  SweepArgs W{};
  W.n = (int)P.n;
  W.K = ctx->K;
  W.small = ctx->plan.small;
  W.exact = ctx->plan.small || ctx->exact_sweeps;
  W.rec = ctx->rec;
  W.start = ctx->start;
  W.G = &ctx->plan_d->G;
  W.err = &ctx->plan_d->err;
  W.dt = dt;
  W.e = e;
  W.mass = P.m;
  W.cnt = ctx->cnt;
  W.slot_j = ctx->slot_j;
  W.slot_t = ctx->slot_t;
  W.key_t = ctx->key_t;
  W.status = ctx->status;
  W.out = ctx->out;
  W.list[0] = ctx->list_a;
  W.list[1] = ctx->cid;  // the cell numbers are done with once the spheres are sorted
  W.ctr = ctx->ctr_d;
  sweep_shards(W);
  return W;
}

// Queue the sweeps before place `end` of the counters on s.  first: from the
// first sweep on (place 0), keys in ctx->key_j, and the list is made; else more
// of them, from place 1.  The keys alternate between ctx->key_j and ctx->ovf; W
// counts the turns from one group to the next.
static hipError_t queue_sweeps(pcol_ctx *ctx, SweepArgs &W, hipStream_t s, int end, bool first) {
  hipError_t e = hipSuccess;
  if (first) {
    if ((e = launch_sweep_first(s, W, ctx->key_j)) != hipSuccess) return e;
    W.turn = 0;
    // a first group of one: the next one starts with the rekey
    W.rekeyed = end > 1;
    if (end > 1 && (e = launch_rekey(s, W, ctx->key_j)) != hipSuccess) return e;
  } else if (!W.rekeyed) {
    if ((e = launch_rekey(s, W, ctx->key_j)) != hipSuccess) return e;
    W.rekeyed = 1;
  }
  for (int k = 1; k < end; ++k) {
    int *in = W.turn & 1 ? ctx->ovf : ctx->key_j, *out = W.turn & 1 ? ctx->key_j : ctx->ovf;
    if ((e = launch_sweep(s, W, in, out, k, k == 1, W.turn)) != hipSuccess) return e;
    ++W.turn;
  }
  return e;
}

// The whole step of pcol_step and pcol_step_spin (spin: nullptr for none).
static pcol_status step_impl(pcol_ctx *ctx, pcol_particles *p, const pcol_box *box, double dt,
                             double e, int32_t *partner, double *tcoll, pcol_stats *stats,
                             const Spin *spin) {
  pcol_status st = check_common(ctx, p, box, dt);
  if (st != PCOL_OK) return st;
  if (!(e >= 0.0 && e <= 1.0)) return fail(ctx, PCOL_E_INVALID, "e outside [0, 1]");
  if (ctx->opts.order == 1 && (spin || ctx->walls))
    return fail(ctx, PCOL_E_INVALID, "the literal order (opts.order = 1) is built for pcol_step only");
  // the literal order's ranks (set by the binning), else rule 2
  const unsigned long long *crank = ctx->opts.order == 1 ? ctx->crank : nullptr;
  hipStream_t s = ctx->stream;
  const bool timing = ctx->opts.timing != 0;
  if (timing) PCOL_HIP(hipEventRecord(ctx->ev[0], s));
  // The binning is queued ahead of its plan where that can be done.  If the plan
  // turns out not to fit, nothing has run, and the step is queued again behind a
  // wait.
  // Few spheres: one workgroup before the pair tests and, of fewer still, one after
  // them, unless slots have overflowed.
  bool ahead = true, few = p->n < SMALL_N;
  if ((st = bin_queue(ctx, p, box, dt, ahead, few)) != PCOL_OK) return st;
  if (timing) PCOL_HIP(hipEventRecord(ctx->ev[1], s));
  const int n = (int)p->n;
  int32_t *part = partner ? partner : ctx->partner_tmp;
  double *tc = tcoll ? tcoll : ctx->tcoll_tmp;
  const Particles P = to_dev(p);
  int64_t pairs = 0, sweeps = 0, ovf_total = 0;
  unsigned long long contacts = 0ull, recheck = 0ull, tests = 0ull;
  double ms_detect = 0.0;
  if (n > 0) {
    // sweep 1: every contact within dt, then the earliest partner of each sphere
    ctx->detect_timed = false;
    // (the friction resolve needs the registers of a whole workgroup of 1024 twice)
    bool one_tail = few && n <= SMALL_TAIL && !spin && !timing && !ctx->exact_sweeps;
    if ((st = detect_all(ctx, dt, crank, one_tail)) != PCOL_OK) return st;
    if (timing) PCOL_HIP(hipEventRecord(ctx->ev[2], s));
    SweepArgs W = sweep_args(ctx, P, dt, e);
    W.crank = crank;
    if (spin) W.spin = *spin;
    // sweeps that cannot search stop at an overflow, so only the others need its keys
    const unsigned int *err = &ctx->plan_d->err;
    if (W.exact && !ctx->plan.small &&
        (st = overflow_search(ctx, dt, crank)) != PCOL_OK)
      return st;
    // The plan did not fit what was queued behind it, and nothing has run: once more,
    // behind a wait.  The events of the binning and the pair tests are taken again.
    const auto start_over = [&]() -> pcol_status {
      few = one_tail = false;
      pcol_status again = bin_queue(ctx, p, box, dt, ahead, few);
      if (again != PCOL_OK) return again;
      if (timing) PCOL_HIP(hipEventRecord(ctx->ev[1], s));
      ctx->detect_timed = false;
      if ((again = detect_all(ctx, dt, crank)) != PCOL_OK) return again;
      if (timing) PCOL_HIP(hipEventRecord(ctx->ev[2], s));
      W = sweep_args(ctx, P, dt, e);
      W.crank = crank;
      if (spin) W.spin = *spin;
      return W.exact && !ctx->plan.small ? overflow_search(ctx, dt, crank) : PCOL_OK;
    };
    // All the sweeps that the step is likely to take, and the free flight behind
    // them, are queued at once: a sweep runs if the one before it resolved a pair,
    // the free flight if the last one resolved none.  Steps that need more are
    // continued below, one wait for each group.
    const int cap = ctx->opts.max_sweeps;
    if (one_tail) {
      PCOL_HIP(launch_sweeps_small(s, W, P, part, tc, cap, ctx->rep));
      PCOL_HIP(hipStreamSynchronize(s));
      ahead = false;
      if (ctx->plan_h->err == PLAN_AGAIN) {  // too many cells, or a grid of another kind
        ctx->many_cells = ctx->plan_h->cells > SMALL_CELLS;
        if ((st = start_over()) != PCOL_OK) return st;
      } else {
        if ((st = take_plan(ctx)) != PCOL_OK) return st;
        if (ctx->rep->n_overflow) {  // nothing ran: sweeps that can search
          one_tail = false;
          W.exact = ctx->exact_sweeps = 1;
          PCOL_HIP(launch_slot_min(s, n, ctx->cnt, ctx->slot_t, ctx->slot_j, ctx->K, ctx->rec,
                                   ctx->key_j, ctx->key_t, ctx->ovf, ctx->ctr_d, err,
                                   &ctx->plan_d->G, crank));
          if ((st = overflow_search(ctx, dt, crank)) != PCOL_OK) return st;
        } else {
          pairs = (int64_t)ctx->rep->small_pairs;
          sweeps = ctx->rep->small_sweeps;
          if (!ctx->rep->small_done)
            return fail(ctx, PCOL_E_SWEEPS, "sweep cap reached with pairs still resolving");
        }
      }
    }
    int group = ctx->sweep_guess + 1;
    if (group < 4) group = 4;
    bool first = true;
    while (!one_tail) {
      if (group > MAX_QUEUE - 1) group = MAX_QUEUE - 1;
      if (cap > 0 && group > cap - (int)sweeps) group = cap - (int)sweeps;
      if (!first) PCOL_HIP(hipMemsetAsync(ctx->ctr_d->pairs, 0, sizeof(ctx->ctr_d->pairs), s));
      const int begin = first ? 0 : 1, end = begin + group;
      PCOL_HIP(queue_sweeps(ctx, W, s, end, first));
      if (timing) PCOL_HIP(hipEventRecord(ctx->ev[3], s));
      PCOL_HIP(launch_finish(s, P, ctx->rank, ctx->out, ctx->status, part, tc, dt, ctx->plan_d,
                             ctx->start, nullptr, ctx->ctr_d, end, W.exact != 0,
                             err, ctx->rep));
      PCOL_HIP(hipStreamSynchronize(s));
      if (ahead) {
        ahead = false;
        if (ctx->plan_h->err == PLAN_AGAIN) {
          ctx->many_cells = few && ctx->plan_h->cells > SMALL_CELLS;
          if ((st = start_over()) != PCOL_OK) return st;
          continue;
        }
        if ((st = take_plan(ctx)) != PCOL_OK) return st;
        if (!few) ctx->counts_dirty = false;
      }
      if (!W.exact && ctx->rep->n_overflow) {  // nothing ran: again, with the exact search
        W.exact = ctx->exact_sweeps = 1;
        if ((st = overflow_search(ctx, dt, crank)) != PCOL_OK) return st;
        continue;
      }
      bool done = false;
      for (int k = begin; k < end && !done; ++k) {
        ++sweeps;
        pairs += (int64_t)ctx->rep->pairs[k];
        done = ctx->rep->pairs[k] == 0ull;
      }
      if (done) break;
      if (cap > 0 && sweeps >= cap)
        return fail(ctx, PCOL_E_SWEEPS, "sweep cap reached with pairs still resolving");
      group = first ? 4 : 2 * group;
      first = false;
    }
    ctx->sweep_guess = (int)std::min(sweeps, (int64_t)MAX_QUEUE);
    contacts = ctx->rep->contacts / 2ull;
    recheck = ctx->rep->recheck;
    tests = ctx->rep->tests;
    ovf_total = ctx->rep->n_overflow;
    if (timing) {
      PCOL_HIP(hipEventRecord(ctx->ev[4], s));
      PCOL_HIP(hipEventSynchronize(ctx->ev[4]));
      ms_detect = ctx->detect_timed ? ms_between(ctx->ev[5], ctx->ev[6])
                                    : ms_between(ctx->ev[1], ctx->ev[2]);
    }
  }
  if (stats) {
    memset(stats, 0, sizeof(*stats));
    stats->n_pairs = pairs;
    stats->n_sweeps = sweeps;
    stats->contacts = (int64_t)contacts;
    stats->n_overflow = ovf_total;
    stats->n_recheck = (int64_t)recheck;
    const StepPlan &pl = ctx->plan;
    stats->band = pl.band;
    for (int a = 0; a < 3; ++a) {
      stats->nc[a] = pl.G.nc[a];
      stats->h[a] = pl.G.h[a];
    }
    stats->max_cell = n > 0 ? (int)ctx->rep->maxcell : 0;
    stats->home_cells = n > 0 ? pl.cpw : 0;
    stats->reach = pl.reach;
    stats->n_wide = n > 0 ? n - ctx->rep->wide_first : 0;
    stats->rho_c = pl.split ? pl.rho_c : 0.0;
    stats->pair_tests = (int64_t)tests;
    if (timing && n > 0) {
      stats->ms_bin = ms_between(ctx->ev[0], ctx->ev[1]);
      stats->ms_detect = ms_detect;
      stats->ms_sweeps = ms_between(ctx->ev[2], ctx->ev[3]);
      stats->ms_advance = ms_between(ctx->ev[3], ctx->ev[4]);
    }
  }
  return PCOL_OK;
}

extern "C" {

pcol_status pcol_step(pcol_ctx *ctx, pcol_particles *p, const pcol_box *box, double dt, double e,
                      int32_t *partner, double *tcoll, pcol_stats *stats) {
  return step_impl(ctx, p, box, dt, e, partner, tcoll, stats, nullptr);
}

pcol_status pcol_step_spin(pcol_ctx *ctx, pcol_particles *p, double *wx, double *wy, double *wz,
                           const pcol_box *box, double dt, double e, double mu,
                           int32_t *partner, double *tcoll, pcol_stats *stats) {
  if (!ctx) return PCOL_E_INVALID;
  if (!(mu >= 0.0) || !isfinite(mu)) return fail(ctx, PCOL_E_INVALID, "mu negative or not finite");
  if (p && p->n > 0 && (!wx || !wy || !wz)) return fail(ctx, PCOL_E_INVALID, "null spin array");
  const Spin sp{wx, wy, wz, mu};
  ctx->spin = &sp;  // the binning validates the spins with the other inputs
  const pcol_status st = step_impl(ctx, p, box, dt, e, partner, tcoll, stats, &sp);
  ctx->spin = nullptr;
  return st;
}

pcol_status pcol_step_spin_walls(pcol_ctx *ctx, pcol_particles *p, double *wx, double *wy,
                                 double *wz, const pcol_box *box, const int32_t walls[3],
                                 double dt, double e, double mu, int32_t *partner, double *tcoll,
                                 pcol_stats *stats) {
  if (!ctx) return PCOL_E_INVALID;
  if (!walls) return fail(ctx, PCOL_E_INVALID, "null walls");
  int mask = 0;
  for (int a = 0; a < 3; ++a)
    if (walls[a]) mask |= 1 << a;
  ctx->walls = mask;
  const pcol_status st = pcol_step_spin(ctx, p, wx, wy, wz, box, dt, e, mu, partner, tcoll, stats);
  ctx->walls = 0;
  return st;
}

pcol_status pcol_step_walls(pcol_ctx *ctx, pcol_particles *p, const pcol_box *box,
                            const int32_t walls[3], double dt, double e, int32_t *partner,
                            double *tcoll, pcol_stats *stats) {
  if (!ctx) return PCOL_E_INVALID;
  if (!walls) return fail(ctx, PCOL_E_INVALID, "null walls");
  int mask = 0;
  for (int a = 0; a < 3; ++a)
    if (walls[a]) mask |= 1 << a;
  ctx->walls = mask;  // the binning builds its grid with these walls
  const pcol_status st = step_impl(ctx, p, box, dt, e, partner, tcoll, stats, nullptr);
  ctx->walls = 0;
  return st;
}

pcol_status pcol_step_backward(pcol_ctx *ctx, const pcol_particles *start, const pcol_box *box,
                               double dt, double e, const int32_t *partner, const double *tcoll,
                               const pcol_state_grad *g_out, pcol_state_grad *g_in, double *ge) {
  pcol_status st = check_common(ctx, start, box, dt);
  if (st != PCOL_OK) return st;
  if (!(e >= 0.0 && e <= 1.0)) return fail(ctx, PCOL_E_INVALID, "e outside [0, 1]");
  if (!g_out || !g_in || !ge) return fail(ctx, PCOL_E_INVALID, "null gradient argument");
  if (start->n > 0 && (!partner || !tcoll || !g_out->x || !g_out->y || !g_out->z || !g_out->vx ||
                       !g_out->vy || !g_out->vz || !g_in->x || !g_in->y || !g_in->z ||
                       !g_in->vx || !g_in->vy || !g_in->vz))
    return fail(ctx, PCOL_E_INVALID, "null array");
  Grid G{};
  for (int a = 0; a < 3; ++a) {
    G.L[a] = box->len[a];
    G.halfL[a] = 0.5 * box->len[a];
    G.sL[a] = box->len[a];
  }
  StateGrad go{g_out->x, g_out->y, g_out->z, g_out->vx, g_out->vy, g_out->vz};
  StateGrad gi{g_in->x, g_in->y, g_in->z, g_in->vx, g_in->vy, g_in->vz};
  PCOL_HIP(launch_step_backward(ctx->stream, to_dev(start), G, dt, e, partner, tcoll, go, gi,
                                ctx->key_t, ge));
  return PCOL_OK;
}

pcol_status pcol_deposit(pcol_ctx *ctx, const double *x, const double *y, const double *z,
                         int64_t n, const double *a, int comp, const int32_t nc[3],
                         const double len[3], double *out) {
  if (!ctx) return PCOL_E_INVALID;
  DepositArgs D{};
  const char *why = nullptr;
  pcol_status st = deposit_args(x, y, z, n, a, comp, nc, len, out, D, why);
  if (st != PCOL_OK) return fail(ctx, st, why);
  hipStream_t s = ctx->stream;
  const DepositLayout Lo = deposit_layout(D.n, D.nnode, comp);
  // the last deposition's node sums read the scratch on another stream
  if (ctx->dep_flag_h && ctx->dep_stream != s) PCOL_HIP(hipDeviceSynchronize());
  ctx->dep_stream = s;
  if (ctx->dep_cap < Lo.bytes || !ctx->dep_known) {
    PCOL_HIP(hipStreamSynchronize(s));  // the free below waits for nothing queued
    hipError_t e = grow(&ctx->dep_buf, ctx->dep_cap, Lo.bytes);
    if (e == hipSuccess && !ctx->dep_flag_h)
      e = hipHostMalloc((void **)&ctx->dep_flag_h, sizeof(unsigned int));
    if (e == hipSuccess && !ctx->dep_known)
      e = hipEventCreateWithFlags(&ctx->dep_known, hipEventDisableTiming);
    if (e != hipSuccess) {
      (void)hipGetLastError();
      return fail(ctx, e == hipErrorOutOfMemory ? PCOL_E_NOMEM : PCOL_E_HIP,
                  "deposition scratch allocation failed");
    }
  }
  hipError_t e = deposit_run(D, Lo, ctx->dep_buf, s, ctx->dep_flag_h, ctx->dep_known, st);
  if (e != hipSuccess) return hip_fail(ctx, e, "pcol_deposit");
  if (st != PCOL_OK) return fail(ctx, st, "position outside [0, L) or not finite");
  return PCOL_OK;
}

pcol_status pcol_deposit_noalloc(const double *x, const double *y, const double *z, int64_t n,
                                 const double *a, int comp, const int32_t nc[3],
                                 const double len[3], double *out, void *hip_stream) {
  DepositArgs D{};
  const char *why = nullptr;
  pcol_status st = deposit_args(x, y, z, n, a, comp, nc, len, out, D, why);
  if (st != PCOL_OK) return st;
  const DepositLayout Lo = deposit_layout(D.n, D.nnode, comp);
  if (Lo.bytes > (int64_t)PCOL_NOALLOC_SCRATCH_BYTES) return PCOL_E_SCRATCH;
  unsigned char *base = nullptr;
  if (static_scratch(&base) != hipSuccess) return PCOL_E_HIP;
  unsigned int flag_h = 0u;  // pageable host word: no pinned allocation
  if (deposit_run(D, Lo, base, (hipStream_t)hip_stream, &flag_h, nullptr, st) != hipSuccess)
    return PCOL_E_HIP;
  return st;
}

}  // extern "C"

// ---------------------------------------------------------------- batched form

namespace {

BatchDev batch_dev(const BatchPlan *bp) {
  BatchDev B{};
  B.gtab = bp->gtab;
  B.cell_base = bp->cell_base;
  B.box_of = bp->box_of;
  B.box_off = bp->box_off_d;
  B.breach = bp->breach;
  B.nchunk = bp->nchunk;
  B.chunk_box = bp->chunk_box;
  B.chunk_lo = bp->chunk_lo;
  B.bmax = bp->bmax;
  B.flags = bp->flags;
  B.nbox = bp->nbox;
  return B;
}

// Grid of one box: cell side >= reach * mult * 1.05 per axis (the slack lets
// the reach grow a little over later steps before a re-plan), no more cells
// than max(27, n_b / 8) for a box of n_b spheres (sparse boxes get cells of
// about 8 spheres: the per-cell work of the pair tests outweighs the extra
// pairs), and at least 3 cells per axis (else the box is rejected).
bool box_grid(const double len[3], int64_t nb, double reach, double mult, Grid &G) {
  double cell = reach * mult * 1.05;
  const double vol = len[0] * len[1] * len[2];
  const double most = (double)nb / 8.0 > 27.0 ? (double)nb / 8.0 : 27.0;
  const double floor_side = cbrt(vol / most);
  if (!(cell >= floor_side)) cell = floor_side;
  for (int a = 0; a < 3; ++a) {
    double q = floor(len[a] / (cell * (1.0 + 1e-9)));
    if (q > 1024.0) q = 1024.0;
    if (q < 3.0) {
      // fall back to exactly 3 cells when they are still at least the reach wide
      if (len[a] / 3.0 >= reach * (1.0 + 1e-9))
        q = 3.0;
      else
        return false;
    }
    G.nc[a] = (int)q;
    G.L[a] = len[a];
    G.halfL[a] = 0.5 * len[a];
    G.sL[a] = len[a];
    G.inv_h[a] = q / len[a];
    G.h[a] = len[a] / q;
  }
  G.ncell = G.nc[0] * G.nc[1] * G.nc[2];
  G.inv_row = 1.0 / G.nc[0];
  G.inv_layer = 1.0 / ((double)G.nc[0] * G.nc[1]);
  return true;
}

template <typename T>
hipError_t regrow(T **p, int64_t want) {
  if (*p) (void)hipFree(*p);
  *p = nullptr;
  return hipMalloc((void **)p, (size_t)(want > 0 ? want : 1) * sizeof(T));
}

// read back the flags of the last batched run (its report is there with them)
hipError_t batch_readback(pcol_ctx *ctx, BatchPlan *bp) {
  hipError_t e = hipMemcpyAsync(bp->flags_h, bp->flags, 4 * sizeof(unsigned int),
                                hipMemcpyDeviceToHost, ctx->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
  return e;
}

}  // namespace

// (Re)build the per-box tables for this layout and the current data: per-box
// reach on the device, then grids and cell numbering on the host.
static pcol_status batch_plan(pcol_ctx *ctx, int nbox, const int64_t *box_off,
                              const pcol_box *boxes, const Particles &P, double dt, double mult) {
  BatchPlan *bp = ctx->bp;
  hipStream_t s = ctx->stream;
  hipError_t e = hipSuccess;
  if (nbox > bp->cap_box) {
    if ((e = regrow(&bp->gtab, nbox)) != hipSuccess ||
        (e = regrow(&bp->cell_base, nbox + 1)) != hipSuccess ||
        (e = regrow(&bp->box_off_d, nbox + 1)) != hipSuccess ||
        (e = regrow(&bp->breach, nbox)) != hipSuccess ||
        (e = regrow(&bp->bmax, nbox)) != hipSuccess)
      return fail(ctx, PCOL_E_NOMEM, "batched tables");
    bp->cap_box = nbox;
  }
  // chunks of the reach pass: each box cut into pieces of BREACH_CHUNK spheres
  std::vector<int> &cbox = bp->chunk_box_h;
  std::vector<int64_t> &clo = bp->chunk_lo_h;
  cbox.clear();
  clo.clear();
  for (int b = 0; b < nbox; ++b)
    for (int64_t lo = box_off[b]; lo < box_off[b + 1]; lo += BREACH_CHUNK) {
      cbox.push_back(b);
      clo.push_back(lo);
    }
  if ((int)cbox.size() > bp->cap_chunk) {
    if ((e = regrow(&bp->chunk_box, (int64_t)cbox.size())) != hipSuccess ||
        (e = regrow(&bp->chunk_lo, (int64_t)cbox.size())) != hipSuccess)
      return fail(ctx, PCOL_E_NOMEM, "batched tables");
    bp->cap_chunk = (int)cbox.size();
  }
  bp->nchunk = (int)cbox.size();
  if (!cbox.empty()) {
    PCOL_HIP(hipMemcpyAsync(bp->chunk_box, cbox.data(), cbox.size() * sizeof(int),
                            hipMemcpyHostToDevice, s));
    PCOL_HIP(hipMemcpyAsync(bp->chunk_lo, clo.data(), clo.size() * sizeof(int64_t),
                            hipMemcpyHostToDevice, s));
  }
  PCOL_HIP(hipMemsetAsync(bp->bmax, 0, (size_t)nbox * sizeof(BoxMax), s));
  if (P.n > bp->cap_n) {
    if ((e = regrow(&bp->box_of, P.n)) != hipSuccess)
      return fail(ctx, PCOL_E_NOMEM, "batched tables");
    bp->cap_n = P.n;
  }
  if (!bp->flags) {
    if (hipMalloc((void **)&bp->flags, 16 * sizeof(unsigned int)) != hipSuccess ||
        hipHostMalloc((void **)&bp->flags_h, 16 * sizeof(unsigned int)) != hipSuccess)
      return fail(ctx, PCOL_E_NOMEM, "batched flags");
  }
  bp->nbox = nbox;
  bp->n = P.n;
  bp->box_off.assign(box_off, box_off + nbox + 1);
  bp->len.resize((size_t)3 * nbox);
  bp->gtab_h.assign(nbox, Grid{});
  for (int b = 0; b < nbox; ++b)
    for (int a = 0; a < 3; ++a) {
      bp->len[3 * b + a] = boxes[b].len[a];
      bp->gtab_h[b].L[a] = boxes[b].len[a];
      bp->gtab_h[b].nc[a] = 1;
    }
  PCOL_HIP(hipMemcpyAsync(bp->box_off_d, box_off, (nbox + 1) * sizeof(int64_t),
                          hipMemcpyHostToDevice, s));
  PCOL_HIP(hipMemcpyAsync(bp->gtab, bp->gtab_h.data(), nbox * sizeof(Grid), hipMemcpyHostToDevice, s));
  PCOL_HIP(launch_fill_box_of(s, nbox, bp->box_off_d, bp->box_of));
  PCOL_HIP(launch_fill_u32(s, bp->flags, 0u, 16));
  PCOL_HIP(launch_breach(s, P, batch_dev(bp), dt, 0));
  bp->breach_h.resize(nbox);
  PCOL_HIP(hipMemcpyAsync(bp->breach_h.data(), bp->breach, nbox * sizeof(double),
                          hipMemcpyDeviceToHost, s));
  PCOL_HIP(batch_readback(ctx, bp));
  const unsigned int err = bp->flags_h[FLAG_ERR];
  if (err & ERR_INVALID) return fail(ctx, PCOL_E_INVALID, "non-finite value, r <= 0, m <= 0 or position outside its box");
  if (err & ERR_BOX) return fail(ctx, PCOL_E_BOX, "a box side <= 2 * reach");
  bp->cell_base_h.assign(nbox + 1, 0);
  int64_t total = 0;
  for (int b = 0; b < nbox; ++b) {
    double len[3] = {boxes[b].len[0], boxes[b].len[1], boxes[b].len[2]};
    if (!box_grid(len, box_off[b + 1] - box_off[b], bp->breach_h[b], mult, bp->gtab_h[b]))
      return fail(ctx, PCOL_E_BOX, "batched form needs 3 cells of at least the reach per axis");
    bp->cell_base_h[b] = (int)total;
    total += bp->gtab_h[b].ncell;
    if (total > (1 << 28)) return fail(ctx, PCOL_E_BOX, "too many cells in the batch");
  }
  bp->cell_base_h[nbox] = (int)total;
  bp->total_cells = (int)total;
  PCOL_HIP(hipMemcpyAsync(bp->gtab, bp->gtab_h.data(), nbox * sizeof(Grid), hipMemcpyHostToDevice, s));
  PCOL_HIP(hipMemcpyAsync(bp->cell_base, bp->cell_base_h.data(), (nbox + 1) * sizeof(int),
                          hipMemcpyHostToDevice, s));
  const pcol_status room = grow_cells(ctx, total);
  if (room != PCOL_OK) return room;
  PCOL_HIP(hipStreamSynchronize(s));
  bp->tables = true;
  bp->cell_mult = mult;
  return PCOL_OK;
}

static SweepArgs batch_sweep_args(const pcol_ctx *ctx, const Particles &P, double dt, double e) {
  SweepArgs W = sweep_args(ctx, P, dt, e);
  W.small = 0;
  W.exact = ctx->exact_sweeps;
  W.G = nullptr;  // periodic boxes; each sphere's grid is its box's
  W.B = batch_dev(ctx->bp);
  W.err = ctx->bp->flags + FLAG_ERR;
  return W;
}

// Keys, by the exact search, of the spheres whose contacts overflowed their slots.
static hipError_t batch_overflow_search(pcol_ctx *ctx, hipStream_t s, const BatchDev &B, int n,
                                        double dt) {
  return launch_gather_exact(s, ctx->ovf, n, &ctx->ctr_d->n_overflow, ctx->rec, ctx->start, nullptr,
                             dt, ctx->key_j, ctx->key_t, &B, ctx->bp->flags + FLAG_ERR);
}

// Enqueue the whole batched step on stream s (captured into a graph).
static pcol_status batch_enqueue(pcol_ctx *ctx, hipStream_t s, const Particles &P, int32_t *part,
                                 double *tc, double dt, double e, int kmax, int cpw) {
  BatchPlan *bp = ctx->bp;
  const BatchDev B = batch_dev(bp);
  const int n = (int)P.n;
  const int ncell = bp->total_cells;
  PCOL_HIP(launch_fill_u32(s, bp->flags, 0u, 16));
  PCOL_HIP(launch_fill_u32(s, (unsigned int *)ctx->ctr_d, 0u, sizeof(SweepCounters) / 4));
  // reach check and cell ids in one pass over the spheres (the counts are
  // discarded with everything else if the check fails)
  PCOL_HIP(launch_fill_i32(s, ctx->count, 0, ncell));
  PCOL_HIP(launch_fill_u32(s, (unsigned int *)ctx->scan, 0u,
                           2 + 2 * ((int64_t)scan_tiles(ncell) + 1)));
  PCOL_HIP(launch_breach(s, P, B, dt, 1, ctx->cid, ctx->slot, ctx->count));
  PCOL_HIP(launch_scan(s, ctx->count, ncell, nullptr, ctx->start, ctx->scan, nullptr, true));
  PCOL_HIP(launch_scatter(s, P, ctx->cid, ctx->slot, ctx->start, ctx->rec, ctx->rank, ctx->cnt, &B,
                          bp->flags + FLAG_ERR));
  DetectArgs A{};
  A.rec = ctx->rec;
  A.start = ctx->start;
  A.cnt = ctx->cnt;
  A.slot_t = ctx->slot_t;
  A.slot_j = ctx->slot_j;
  A.ctr = ctx->ctr_d;
  A.n = n;
  A.dt = dt;
  A.dt2 = 2.0 * dt * (1.0 + 0x1.0p-20);
  // Filter tolerance (see the single-box detect) from bounds that hold for any
  // data the graph accepts: the re-plan check stops the step unless every
  // box's reach 2 rmax + 2 vmax dt is at most its cell side, so with hmax the
  // largest cell side, reach <= hmax, 2 rmax <= hmax and 2 vmax <= hmax / dt.
  double hmax = 0.0;
  for (const Grid &G : bp->gtab_h)
    for (int a = 0; a < 3; ++a) hmax = G.h[a] > hmax ? G.h[a] : hmax;
  {
    // reach <= hmax, 2 r_max <= hmax and 2 v_max dt <= hmax in every box (see above)
    double Lmax = 0.0, X = 0.0;
    for (const Grid &G : bp->gtab_h) {
      X = std::max(X, grid_norm(G));
      for (int a = 0; a < 3; ++a) Lmax = G.L[a] > Lmax ? G.L[a] : Lmax;
    }
    A.tol64 = gram64_tolerance(X, hmax, hmax, hmax / (2.0 * dt), 0.5 * hmax, Lmax, A.dt2);
  }
  A.K = ctx->K;
  PCOL_HIP(launch_detect_batched(s, A, B, bp->total_cells, cpw));
  PCOL_HIP(launch_slot_min(s, n, ctx->cnt, ctx->slot_t, ctx->slot_j, ctx->K, ctx->rec, ctx->key_j,
                           ctx->key_t, ctx->ovf, ctx->ctr_d, bp->flags + FLAG_ERR));
  SweepArgs W = batch_sweep_args(ctx, P, dt, e);
  if (W.exact) PCOL_HIP(batch_overflow_search(ctx, s, B, n, dt));
  PCOL_HIP(queue_sweeps(ctx, W, s, kmax, true));
  PCOL_HIP(launch_finish(s, P, ctx->rank, ctx->out, ctx->status, part, tc, dt, nullptr,
                         nullptr, &B, ctx->ctr_d, kmax, W.exact != 0, bp->flags + FLAG_ERR,
                         ctx->rep));
  return PCOL_OK;
}

static pcol_status batch_capture(pcol_ctx *ctx, const Particles &P, int32_t *part, double *tc,
                                 double dt, double e, int kmax, int cpw, hipGraphExec_t *exec) {
  BatchPlan *bp = ctx->bp;
  if (!bp->gstream) PCOL_HIP(hipStreamCreateWithFlags(&bp->gstream, hipStreamNonBlocking));
  PCOL_HIP(hipStreamBeginCapture(bp->gstream, hipStreamCaptureModeRelaxed));
  pcol_status st = batch_enqueue(ctx, bp->gstream, P, part, tc, dt, e, kmax, cpw);
  hipGraph_t g = nullptr;
  hipError_t ee = hipStreamEndCapture(bp->gstream, &g);
  if (st != PCOL_OK) {
    if (g) (void)hipGraphDestroy(g);
    return st;
  }
  if (ee != hipSuccess) return hip_fail(ctx, ee, "hipStreamEndCapture");
  ee = hipGraphInstantiate(exec, g, nullptr, nullptr, 0);
  (void)hipGraphDestroy(g);
  if (ee != hipSuccess) return hip_fail(ctx, ee, "hipGraphInstantiate");
  return PCOL_OK;
}

// Continue a step whose captured sweeps ran out (the graph then skipped the free
// flight and the copy back): more sweeps, a wait for each group.
static pcol_status batch_finish(pcol_ctx *ctx, const Particles &P, int32_t *part, double *tc,
                                double dt, double e, int64_t &pairs, int64_t &sweeps) {
  BatchPlan *bp = ctx->bp;
  const BatchDev B = batch_dev(bp);
  hipStream_t s = ctx->stream;
  SweepArgs W = batch_sweep_args(ctx, P, dt, e);
  W.rekeyed = bp->kmax > 1;
  W.turn = bp->kmax - 1;
  for (int end = 5;; end = std::min(2 * end, MAX_QUEUE)) {
    PCOL_HIP(hipMemsetAsync(ctx->ctr_d->pairs, 0, sizeof(ctx->ctr_d->pairs), s));
    PCOL_HIP(queue_sweeps(ctx, W, s, end, false));
    PCOL_HIP(launch_finish(s, P, ctx->rank, ctx->out, ctx->status, part, tc, dt, nullptr,
                           nullptr, &B, ctx->ctr_d, end, W.exact != 0, bp->flags + FLAG_ERR,
                           ctx->rep));
    PCOL_HIP(hipStreamSynchronize(s));
    for (int k = 1; k < end; ++k) {
      ++sweeps;
      pairs += (int64_t)ctx->rep->pairs[k];
      if (ctx->rep->pairs[k] == 0ull) return PCOL_OK;
    }
  }
}

static std::string tune_key(int nbox, int64_t n, const int64_t *box_off, const pcol_box *boxes,
                            double dt) {
  hipDeviceProp_t prop{};
  int dev = 0;
  (void)hipGetDevice(&dev);
  (void)hipGetDeviceProperties(&prop, dev);
  double vol = 0.0;
  for (int b = 0; b < nbox; ++b) vol += boxes[b].len[0] * boxes[b].len[1] * boxes[b].len[2];
  std::ostringstream k;
  k << "c" << prop.gcnArchName << "|n" << (int)round(log2((double)(n > 0 ? n : 1))) << "|b"
    << (int)round(log2((double)nbox)) << "|rho" << (int)round(4.0 * log2(n / vol + 1e-300))
    << "|dt" << dt;
  (void)box_off;
  std::string key = k.str();
  for (char &c : key)
    if (c == ' ') c = '_';
  return key;
}

static std::string tune_path() {
  const char *p = getenv("PCOL_TUNE_CACHE");
  if (p && *p) return p;
  const char *h = getenv("HOME");
  return std::string(h ? h : ".") + "/.cache/pcol_tune.txt";
}

static bool tune_lookup(const std::string &key, double &mult, int &cpw) {
  std::ifstream f(tune_path());
  std::string k;
  double m;
  int w;
  bool found = false;
  while (f >> k >> m >> w)
    if (k == key) {
      mult = m;
      cpw = w;
      found = true;
    }
  return found;
}

static void tune_store(const std::string &key, double mult, int cpw) {
  std::ofstream f(tune_path(), std::ios::app);
  if (f) f << key << " " << mult << " " << cpw << "\n";
}

// Time candidate (cell size factor, home cells per workgroup) pairs on scratch
// copies of the input; keep the fastest.  Every candidate computes the same
// step (the result does not depend on the cell size or the launch shape).
static pcol_status batch_autotune(pcol_ctx *ctx, int nbox, const int64_t *box_off,
                                  const pcol_box *boxes, const Particles &P, double dt,
                                  double e) {
  BatchPlan *bp = ctx->bp;
  hipStream_t s = ctx->stream;
  const int64_t n = P.n;
  if (bp->tune_cap < n) {
    if (bp->tune_buf) (void)hipFree(bp->tune_buf);
    bp->tune_buf = nullptr;
    if (hipMalloc((void **)&bp->tune_buf, (size_t)(n > 0 ? n : 1) * 6 * sizeof(double)) != hipSuccess)
      return fail(ctx, PCOL_E_NOMEM, "tuning scratch");
    bp->tune_cap = n;
  }
  Particles T = P;
  double *src[6] = {P.x, P.y, P.z, P.vx, P.vy, P.vz};
  double *dst[6];
  for (int k = 0; k < 6; ++k) dst[k] = bp->tune_buf + (size_t)k * n;
  T.x = dst[0];
  T.y = dst[1];
  T.z = dst[2];
  T.vx = dst[3];
  T.vy = dst[4];
  T.vz = dst[5];
  const double mults[3] = {1.0, 1.15, 1.3};
  const int shapes[3] = {2, 4, 8};  // home cells per workgroup
  double best = 1e300, best_mult = 1.0;
  int best_cpw = 4;
  for (double mult : mults) {
    pcol_status st = batch_plan(ctx, nbox, box_off, boxes, P, dt, mult);
    if (st == PCOL_E_BOX) continue;  // this cell size leaves some box under 3 cells
    if (st != PCOL_OK) return st;
    for (int c = 0; c < 3; ++c) {
      const int cpw = shapes[c];
      hipGraphExec_t ex = nullptr;
      if ((st = batch_capture(ctx, T, ctx->partner_tmp, ctx->tcoll_tmp, dt, e, bp->kmax, cpw,
                              &ex)) != PCOL_OK)
        return st;
      float times[3];
      for (int rep = 0; rep < 3; ++rep) {
        for (int k = 0; k < 6; ++k)
          PCOL_HIP(hipMemcpyAsync(dst[k], src[k], n * sizeof(double), hipMemcpyDeviceToDevice, s));
        PCOL_HIP(hipEventRecord(ctx->ev[0], s));
        PCOL_HIP(hipGraphLaunch(ex, s));
        PCOL_HIP(hipEventRecord(ctx->ev[1], s));
        PCOL_HIP(hipEventSynchronize(ctx->ev[1]));
        (void)hipEventElapsedTime(&times[rep], ctx->ev[0], ctx->ev[1]);
      }
      (void)hipGraphExecDestroy(ex);
      // Slots overflowed: the sweeps stopped before they began.  The contacts are the
      // same for every candidate, so this is the first one; it is timed again.
      if (!ctx->exact_sweeps && ctx->rep->n_overflow) {
        ctx->exact_sweeps = 1;
        --c;
        continue;
      }
      std::sort(times, times + 3);
      if (times[1] < best) {
        best = times[1];
        best_mult = mult;
        best_cpw = cpw;
      }
    }
  }
  bp->cell_mult = best_mult;
  bp->cpw = best_cpw;
  bp->tuned = true;
  bp->tables = false;
  return PCOL_OK;
}

extern "C" pcol_status pcol_step_batched(pcol_ctx *ctx, int32_t nbox, const int64_t *box_off,
                                         const pcol_box *boxes, pcol_particles *p, double dt,
                                         double e, int32_t *partner, double *tcoll,
                                         pcol_batch_stats *stats) {
  if (!ctx) return PCOL_E_INVALID;
  if (ctx->opts.order == 1)
    return fail(ctx, PCOL_E_INVALID, "the literal order (opts.order = 1) is built for pcol_step only");
  if (nbox < 1 || !box_off || !boxes || !p) return fail(ctx, PCOL_E_INVALID, "bad batch arguments");
  pcol_box any{{1.0, 1.0, 1.0}};
  pcol_status st = check_common(ctx, p, &any, dt);
  if (st != PCOL_OK) return st;
  if (!(e >= 0.0 && e <= 1.0)) return fail(ctx, PCOL_E_INVALID, "e outside [0, 1]");
  if (box_off[0] != 0 || box_off[nbox] != p->n)
    return fail(ctx, PCOL_E_INVALID, "box_off must run from 0 to n");
  for (int b = 0; b < nbox; ++b) {
    if (box_off[b + 1] < box_off[b]) return fail(ctx, PCOL_E_INVALID, "box_off not increasing");
    for (int a = 0; a < 3; ++a)
      if (!finite_pos(boxes[b].len[a])) return fail(ctx, PCOL_E_INVALID, "box side not finite positive");
  }
  ctx->binned = false;  // the batch's spheres and cells take the place of the last binning's
  if (!ctx->bp) {
    ctx->bp = new (std::nothrow) BatchPlan();
    if (!ctx->bp) return PCOL_E_NOMEM;
    if (ctx->opts.max_sweeps > 0) ctx->bp->kmax = std::min(ctx->opts.max_sweeps, MAX_QUEUE);
  }
  BatchPlan *bp = ctx->bp;
  const Particles P = to_dev(p);
  int32_t *part = partner ? partner : ctx->partner_tmp;
  double *tc = tcoll ? tcoll : ctx->tcoll_tmp;
  const void *ptrs[8] = {p->x, p->y, p->z, p->vx, p->vy, p->vz, p->r, p->m};
  bool same_layout = bp->tables && bp->nbox == nbox && bp->n == p->n &&
                     std::equal(box_off, box_off + nbox + 1, bp->box_off.begin());
  for (int b = 0; same_layout && b < nbox; ++b)
    for (int a = 0; a < 3; ++a)
      if (bp->len[3 * b + a] != boxes[b].len[a]) same_layout = false;
  int replanned = 0, tuned = 0, host_finish = 0;
  if (!same_layout && !bp->tuned && ctx->opts.autotune) {
    const std::string key = tune_key(nbox, p->n, box_off, boxes, dt);
    double m;
    int w;
    if (tune_lookup(key, m, w)) {
      bp->cell_mult = m;
      bp->cpw = w;
      bp->tuned = true;
    } else {
      if ((st = batch_autotune(ctx, nbox, box_off, boxes, P, dt, e)) != PCOL_OK) return st;
      tune_store(key, bp->cell_mult, bp->cpw);
      tuned = 1;
    }
  }
  if (!ctx->opts.autotune && !bp->tuned) {
    bp->cell_mult = ctx->opts.cell_mult;
    bp->cpw = 4;
  }
  for (int attempt = 0;; ++attempt) {
    if (!same_layout || !bp->tables) {
      if ((st = batch_plan(ctx, nbox, box_off, boxes, P, dt, bp->cell_mult)) != PCOL_OK) return st;
      same_layout = true;
      bp->captured = false;
      replanned = 1;
    }
    bool recapture = !bp->captured || bp->cap_dt != dt || bp->cap_e != e || bp->cap_part != part ||
                     bp->cap_tc != tc;
    for (int k = 0; k < 8 && !recapture; ++k) recapture = bp->cap_ptr[k] != ptrs[k];
    if (recapture) {
      if (bp->exec) (void)hipGraphExecDestroy(bp->exec);
      bp->exec = nullptr;
      if ((st = batch_capture(ctx, P, part, tc, dt, e, bp->kmax, bp->cpw, &bp->exec)) != PCOL_OK)
        return st;
      bp->captured = true;
      bp->cap_exact = ctx->exact_sweeps;
      bp->cap_dt = dt;
      bp->cap_e = e;
      bp->cap_part = part;
      bp->cap_tc = tc;
      for (int k = 0; k < 8; ++k) bp->cap_ptr[k] = ptrs[k];
    }
    PCOL_HIP(hipGraphLaunch(bp->exec, ctx->stream));
    PCOL_HIP(batch_readback(ctx, bp));
    const unsigned int err = bp->flags_h[FLAG_ERR];
    if (err & ERR_INVALID)
      return fail(ctx, PCOL_E_INVALID, "non-finite value, r <= 0, m <= 0 or position outside its box");
    if (err & ERR_BOX) return fail(ctx, PCOL_E_BOX, "a box side <= 2 * reach");
    if (err & ERR_REPLAN) {  // reach outgrew the planned cells; nothing was written
      if (attempt > 0) return fail(ctx, PCOL_E_HIP, "batched re-plan did not settle");
      bp->tables = false;
      continue;
    }
    break;
  }
  if (!bp->cap_exact && ctx->rep->n_overflow) {
    // no sweep ran: queue them here with the exact search, and capture it next time
    ctx->exact_sweeps = 1;
    bp->captured = false;
    SweepArgs W = batch_sweep_args(ctx, P, dt, e);
    const BatchDev B = batch_dev(bp);
    PCOL_HIP(batch_overflow_search(ctx, ctx->stream, B, W.n, dt));
    PCOL_HIP(queue_sweeps(ctx, W, ctx->stream, bp->kmax, true));
    PCOL_HIP(launch_finish(ctx->stream, P, ctx->rank, ctx->out, ctx->status, part, tc, dt, nullptr,
                           nullptr, &B, ctx->ctr_d, bp->kmax, true, bp->flags + FLAG_ERR,
                           ctx->rep));
    PCOL_HIP(hipStreamSynchronize(ctx->stream));
  }
  int64_t pairs = 0, sweeps = 0;
  bool done = false;
  for (int k = 0; k < bp->kmax && !done; ++k) {
    ++sweeps;
    pairs += (int64_t)ctx->rep->pairs[k];
    done = ctx->rep->pairs[k] == 0ull;
  }
  if (!done) {
    if ((st = batch_finish(ctx, P, part, tc, dt, e, pairs, sweeps)) != PCOL_OK) return st;
    host_finish = 1;
    if (ctx->opts.max_sweeps == 0) {  // capture enough sweeps next time
      bp->kmax = (int)std::min(sweeps + 4, (int64_t)MAX_QUEUE);
      bp->captured = false;
    }
  } else if (ctx->opts.max_sweeps == 0 && bp->kmax > (int)sweeps + 4) {
    // far more sweep slots than the step used: each empty slot still launches
    // its kernel (an early exit), so capture fewer next time, keeping room for
    // two more sweeps than this step took
    bp->kmax = (int)sweeps + 2;
    bp->captured = false;
  }
  if (stats) {
    memset(stats, 0, sizeof(*stats));
    stats->n_pairs = pairs;
    stats->n_sweeps = sweeps;
    stats->contacts = (int64_t)(ctx->rep->contacts / 2ull);
    stats->n_overflow = (int64_t)ctx->rep->n_overflow;
    stats->total_cells = bp->total_cells;
    stats->replanned = replanned;
    stats->finished_on_host = host_finish;
    stats->tuned = tuned;
    stats->home_cells = bp->cpw;
    stats->cell_mult = bp->cell_mult;
  }
  return PCOL_OK;
}
