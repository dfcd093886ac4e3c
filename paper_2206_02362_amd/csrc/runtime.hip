// Host runtime of the FWIME hot-path library: the C ABI of include/fwime.h.
//
// Responsibilities: input validation (including the CFL test, which needs the
// velocity range and therefore one small device reduction), the context's
// device-memory arena under an HBM budget, the per-tile source/receiver tables
// consumed by the stencil kernel, shot batching, and the time loops with
// sqrt(nt) wavefield checkpointing for the adjoint-state operators.
//
// Time bookkeeping (equation n = 0 .. nt-2 advances u^n -> u^{n+1}):
//   - forward: the kernel of equation n reads u^n, u^{n-1}, writes u^{n+1},
//     injects f^n and records u^n at the receivers; u^{nt-1} is gathered after
//     the loop;
//   - adjoint: the kernel of index k = nt-1 .. 1 reads lambda_k, lambda_{k+1},
//     writes lambda_{k-1} and injects the adjoint source of time k;
//   - segments of K = ceil(sqrt(nt - 1)) equations: the forward pass stores
//     (u^{n0-1}, u^{n0}) at each segment start n0; the backward pass recomputes
//     one segment from its checkpoint, keeping T2u_n = V (L u^n + f^n) for the
//     segment, while the adjoint fields live in rings of K + 2 time slots.
#include "../../include/fwime.h"
#include "internal.h"
#include "line_search.h"

#include <algorithm>
#include <atomic>
#include <cstdint>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <vector>

using namespace fw;

struct fwime_ctx {
  int device = 0;
  size_t budget = 0;
  std::string err;
  void *arena = nullptr;
  size_t arena_bytes = 0;
  double *host_red = nullptr;   // pinned: reduction results
  size_t host_red_n = 0;        // doubles it holds
  int tile_x = 32;
  bool two_step = true;         // two or four time steps per launch (else one)
  int steps = 0;                // 2 or 4: steps per launch whatever the size (0: chosen by size)
  bool frugal = false;          // a call that did not fit runs again with less scratch (see or_frugally)
  size_t tape_bytes = 0;        // device memory held by live tapes
  // memory held for histories: of live tapes, the arena and the solver's buffer
  size_t tape_hist = 0, arena_hist = 0, vp_hist = 0;
  // memory of the largest tape freed so far, for the next one: a tape of whole
  // histories is up to gigabytes, allocated and released on every call else
  // (data and gradient through autograd on 100 x 200, one shot, a tape of
  // 0.65 GB: 13.4 ms with an allocation per call, 12.9 ms without).
  // One buffer at most, none under a budget; counted as free memory, and given
  // back when one of the context's allocations fails or a history needs the
  // room, by fwime_ctx_trim and with the context.
  // Tapes are freed on any thread, and after their context if need be: tape_mu
  // guards tape_bytes, tape_hist, tapes, spare and spare_bytes.
  mutable std::mutex tape_mu;
  std::vector<fwime_tape *> tapes;        // live ones
  void *spare = nullptr;
  size_t spare_bytes = 0;
  // calls that could keep histories so far, and the last of them that kept one
  // in the arena, in the solver's buffer and in the spare (see hist_batch)
  std::atomic<long> calls{0}, spare_use{0};
  long arena_use = 0, vp_use = 0;
  size_t last_arena_request = 0;
  hipStream_t capture = nullptr;          // private stream used only to record graphs
  std::map<std::string, int> tuned;       // batch signature -> tile width
  int last_batch_tile = 0;
  int graph_steps = 64;                   // steps per captured graph
  hipGraph_t graph = nullptr;             // last batch graph, released after the
  hipGraphExec_t graph_exec = nullptr;    // next stream synchronization
  void *vp = nullptr;                     // variable-projection solver vectors, background history
  size_t vp_bytes = 0;
  bool vp_busy = false;                   // while the solver runs
  // optional timing of the stencil launch loop of the modeling calls: two
  // events recorded on the call's stream around its launches
  bool timing = false;
  hipEvent_t tev[2] = {nullptr, nullptr};
  long timed_launches = -1;               // launches between the events of the last timed call
  // while set, the call's scratch is carved from this fixed device buffer
  // instead of the arena, and nothing is allocated (fwime_model_static)
  char *fixed = nullptr;
  size_t fixed_bytes = 0;
  char *static_scratch = nullptr;         // device address of the static scratch array on `device`
};

static void detach_tapes(fwime_ctx_t *ctx);   // live tapes outlive the context

static void release_graph(fwime_ctx_t *ctx) {
  if (ctx->graph_exec) (void)hipGraphExecDestroy(ctx->graph_exec);
  if (ctx->graph) (void)hipGraphDestroy(ctx->graph);
  ctx->graph_exec = nullptr;
  ctx->graph = nullptr;
}

namespace {

constexpr int kSplineMaxNodes = 1 << 24;  // spline nodes per axis
constexpr int kLbfgsMaxPairs = 256;    // L-BFGS pairs accepted by fwime_lbfgs_direction
constexpr int kGxPad = 64;              // zero taper entries past NX read by the last x-tile
constexpr int kGraphMaxTiles = 16384;   // batches above this many tiles launch directly
constexpr double kW[5] = {-205.0 / 72.0, 8.0 / 5.0, -1.0 / 5.0, 8.0 / 315.0, -1.0 / 560.0};

int set_err(fwime_ctx_t *ctx, int code, const std::string &msg) {
  if (ctx) ctx->err = msg;
  return code;
}

#define HIPCHK(expr)                                                                   \
  do {                                                                                 \
    hipError_t e_ = (expr);                                                            \
    if (e_ != hipSuccess)                                                              \
      return set_err(ctx, FWIME_EHIP, std::string(#expr) + ": " + hipGetErrorString(e_)); \
  } while (0)

// Events around a call's stencil launch loop (fwime_ctx_set_timing).
hipError_t timing_begin(fwime_ctx_t *ctx, hipStream_t st) {
  if (!ctx->timing) return hipSuccess;
  ctx->timed_launches = -1;
  return hipEventRecord(ctx->tev[0], st);
}
hipError_t timing_end(fwime_ctx_t *ctx, hipStream_t st, long launches) {
  if (!ctx->timing) return hipSuccess;
  hipError_t e = hipEventRecord(ctx->tev[1], st);
  if (e == hipSuccess) ctx->timed_launches = launches;
  return e;
}

double cfl_limit(double dz, double dx) {
  double nyq = -(kW[0] + 2.0 * (-kW[1] + kW[2] - kW[3] + kW[4]));
  return 2.0 / std::sqrt(nyq * (1.0 / (dz * dz) + 1.0 / (dx * dx)));
}

struct Dims {
  int nz, nx, nb, nt, NZ, NX, LZ, ntz, ntx, TX;
  int ntz2;     // 56-row tiles of the two-step kernel
  // tiles of the four-step kernel, used instead of the two-step one when T = 4
  int ntz4, ntx4, TX4, T;
  long field;   // NX * LZ
};

Dims make_dims(const fwime_grid_t *g, int tx) {
  Dims d;
  d.nz = g->nz;
  d.nx = g->nx;
  d.nb = g->nb;
  d.nt = g->nt;
  d.NZ = g->nz + 2 * g->nb;
  d.NX = g->nx + 2 * g->nb;
  d.LZ = (d.NZ + 4 + 63) / 64 * 64;   // >= 4 zero rows below the grid in every column
  d.TX = tx;
  d.ntz = (d.NZ + kTZ - 1) / kTZ;
  d.ntz2 = (d.NZ + kTZ2 - 1) / kTZ2;
  d.ntx = (d.NX + tx - 1) / tx;
  d.ntz4 = (d.NZ + kTZ4 - 1) / kTZ4;
  d.T = 2;
  d.TX4 = d.ntx4 = 0;
  d.field = (long)d.NX * d.LZ;
  return d;
}

// Steps per launch of the two-step path for batches of S shots.  A launch of
// few workgroups costs its latency, not its work: four steps per launch then
// take little longer than two.  The bounds are in two-step workgroups (56 x 32
// cells of every shot); the extended-precision kernels (df), with more than
// twice the instructions per cell, fill the device sooner.  Measured over 400
// steps, two against four per launch: modeling 36 workgroups 1.65 / 0.86 ms,
// 288 1.79 / 1.48, 330 1.91 / 1.85, 432 1.92 / 2.13; gradient 288 9.9 / 8.6,
// 440 11.6 / 13.1; Born pair 36 11.1 / 5.9, 144 12.2 / 11.2, 220 13.1 / 16.3.
// Tiles are eight columns wide while one round of them fits the 256 compute
// units (one 100 x 200 shot: 0.86 against 0.93 ms; two: 1.01 against 0.96).
constexpr int kStep4MaxTiles = 320, kStep4MaxTilesDF = 160, kStep4MaxNarrow = 256;

void choose_steps(const fwime_ctx_t *ctx, Dims &d, int S, bool df) {
  if (!ctx->two_step || ctx->frugal) return;
  const long tiles = (long)d.ntz2 * d.ntx * S;
  if (ctx->steps ? ctx->steps != 4 : tiles > (df ? kStep4MaxTilesDF : kStep4MaxTiles)) return;
  if ((long)d.ntz4 * ((d.NX + 7) / 8) * S + 8 >= (1L << 20)) return;   // the kernel's tile arithmetic
  d.T = 4;
  d.TX4 = (long)d.ntz4 * ((d.NX + 7) / 8) * S <= kStep4MaxNarrow ? 8 : 16;
  d.ntx4 = (d.NX + d.TX4 - 1) / d.TX4;
}

// ---------------------------------------------------------------------------
// Arena: one device allocation carved into aligned pieces for one call.
// ---------------------------------------------------------------------------
struct Carve {
  std::vector<std::pair<void **, size_t>> items;
  size_t total = 0;
  template <class T>
  void add(T **p, size_t count) {
    size_t bytes = (count * sizeof(T) + 255) / 256 * 256;
    items.push_back({(void **)p, bytes});
    total += bytes;
  }
  // point every piece into `base` (at least `total` bytes)
  void assign(void *base) const {
    char *p = (char *)base;
    for (const auto &it : items) {
      *it.first = p;
      p += it.second;
    }
  }
};

// Frees the spare tape memory (idle since its tape was freed).
void release_spare(fwime_ctx_t *ctx) {
  std::lock_guard<std::mutex> lock(ctx->tape_mu);
  if (ctx->spare) (void)hipFree(ctx->spare);
  ctx->spare = nullptr;
  ctx->spare_bytes = 0;
}

size_t spare_bytes(fwime_ctx_t *ctx) {
  std::lock_guard<std::mutex> lock(ctx->tape_mu);
  return ctx->spare_bytes;
}

size_t tape_hist_bytes(const fwime_ctx_t *ctx) {
  std::lock_guard<std::mutex> lock(ctx->tape_mu);
  return ctx->tape_hist;
}

size_t live_tape_bytes(const fwime_ctx_t *ctx) {
  std::lock_guard<std::mutex> lock(ctx->tape_mu);
  return ctx->tape_bytes;
}

// Frees what the context holds between calls: the spare, the solver's buffer
// and the arena, except the buffer of `owner`.  Between the input checks of a
// call, which wait for the stream, and its own use of them they are idle.
void release_vp(fwime_ctx_t *ctx) {
  if (ctx->vp) (void)hipFree(ctx->vp);
  ctx->vp = nullptr;
  ctx->vp_bytes = ctx->vp_hist = 0;
}
void release_arena(fwime_ctx_t *ctx) {
  if (ctx->arena) (void)hipFree(ctx->arena);
  ctx->arena = nullptr;
  ctx->arena_bytes = ctx->arena_hist = 0;
  ctx->last_arena_request = 0;             // the next one is as large as it needs to be
}
void release_idle(fwime_ctx_t *ctx, void **owner) {
  release_spare(ctx);
  if (!ctx->vp_busy && owner != &ctx->vp) release_vp(ctx);
  if (owner != &ctx->arena) release_arena(ctx);
}

// hipMalloc that gives back what is held idle when memory is short
hipError_t device_alloc(fwime_ctx_t *ctx, void **p, size_t bytes) {
  hipError_t e = hipMalloc(p, bytes);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    release_idle(ctx, p);
    e = hipMalloc(p, bytes);
  }
  return e;
}

int arena_get(fwime_ctx_t *ctx, Carve &cv) {
  if (ctx->fixed) {
    if (cv.total > ctx->fixed_bytes)
      return set_err(ctx, FWIME_ENOMEM, "the call needs " + std::to_string(cv.total) +
                                            " bytes of scratch; the static scratch array holds " +
                                            std::to_string(ctx->fixed_bytes));
    cv.assign(ctx->fixed);
    return FWIME_OK;
  }
  if (cv.total > ctx->arena_bytes) {
    if (ctx->budget && cv.total > ctx->budget)
      return set_err(ctx, FWIME_ENOMEM, "request of " + std::to_string(cv.total) + " bytes exceeds the HBM budget");
    if (ctx->arena) {
      // the context's work runs on one stream, which every call synchronizes
      // during its input checks: the old arena is idle here
      HIPCHK(hipFree(ctx->arena));
      ctx->arena = nullptr;
      ctx->arena_bytes = 0;
    }
    // grow geometrically (within the budget, by 4 GiB at most) so that a
    // sequence of slightly larger calls does not reallocate every time
    const size_t last = ctx->last_arena_request;
    size_t want = std::max(cv.total, last + std::min(last / 2, (size_t)4 << 30));
    if (ctx->budget) want = std::min(want, ctx->budget);
    want = std::max(want, cv.total);
    hipError_t e = device_alloc(ctx, &ctx->arena, want);
    if (e != hipSuccess) {
      (void)hipGetLastError();
      want = cv.total;
      e = device_alloc(ctx, &ctx->arena, want);
    }
    if (e != hipSuccess) {
      ctx->arena = nullptr;
      (void)hipGetLastError();
      return set_err(ctx, FWIME_ENOMEM, "hipMalloc of " + std::to_string(cv.total) + " bytes failed");
    }
    ctx->arena_bytes = want;
  }
  ctx->last_arena_request = std::max(ctx->last_arena_request, cv.total);
  char *p = (char *)ctx->arena;
  for (auto &it : cv.items) {
    *it.first = p;
    p += it.second;
  }
  return FWIME_OK;
}

// Result rc of a call's allocations, or, where they did not fit (rc is
// FWIME_ENOMEM; nothing is written yet) and the call can do with less scratch,
// of the call made again with less: checkpoints instead of whole histories
// (their size goes by what was free, not by what one allocation finds), and two
// steps per launch, whose source and receiver lists take up to 52 bytes a
// receiver against 76 with four.
template <class Call>
int or_frugally(fwime_ctx_t *ctx, int rc, bool less, Call call) {
  if (rc != FWIME_ENOMEM || !less || ctx->frugal) return rc;
  struct Guard {
    fwime_ctx_t *c;
    ~Guard() { c->frugal = false; }
  } guard{ctx};
  ctx->frugal = true;
  return call();
}

// ---------------------------------------------------------------------------
// Validation
// ---------------------------------------------------------------------------
int check_grid(fwime_ctx_t *ctx, const fwime_grid_t *g) {
  if (!g) return set_err(ctx, FWIME_EINVAL, "grid is null");
  if (g->nz < 1 || g->nx < 1 || g->nb < 0 || g->nt < 2)
    return set_err(ctx, FWIME_EINVAL, "grid needs nz, nx >= 1, nb >= 0, nt >= 2");
  if (!(g->dz > 0 && g->dx > 0 && g->dt > 0) || !std::isfinite(g->dz) || !std::isfinite(g->dx) ||
      !std::isfinite(g->dt))
    return set_err(ctx, FWIME_EINVAL, "dz, dx, dt must be positive and finite");
  if (!(g->sponge_alpha >= 0) || !std::isfinite(g->sponge_alpha))
    return set_err(ctx, FWIME_EINVAL, "sponge_alpha must be >= 0");
  if (g->free_surface && g->nb < kR)
    return set_err(ctx, FWIME_EINVAL, "a free surface needs nb >= 4 (the mirrored stencil rows)");
  const long NZ = (long)g->nz + 2L * g->nb, NX = (long)g->nx + 2L * g->nb;
  const long LZ = (NZ + 4 + 63) / 64 * 64;
  // kernels address one shot's field with 32-bit byte offsets
  if ((NX + 256) * LZ * 4 >= (1L << 31)) return set_err(ctx, FWIME_EINVAL, "padded grid too large");
  return FWIME_OK;
}

int check_geom(fwime_ctx_t *ctx, const fwime_grid_t *g, const fwime_geom_t *geo) {
  if (!geo) return set_err(ctx, FWIME_EINVAL, "geometry is null");
  if (geo->nshots < 1 || geo->nrec < 1) return set_err(ctx, FWIME_EINVAL, "need nshots >= 1 and nrec >= 1");
  if (!geo->src_iz || !geo->src_ix || !geo->rec_iz || !geo->rec_ix || !geo->wavelet)
    return set_err(ctx, FWIME_EINVAL, "geometry pointer is null");
  for (int s = 0; s < geo->nshots; ++s) {
    if (geo->src_iz[s] < 0 || geo->src_iz[s] >= g->nz || geo->src_ix[s] < 0 || geo->src_ix[s] >= g->nx)
      return set_err(ctx, FWIME_EINVAL, "source " + std::to_string(s) + " outside the model grid");
  }
  const long n = (long)geo->nshots * geo->nrec;
  for (long i = 0; i < n; ++i) {
    if (geo->rec_iz[i] < 0 || geo->rec_iz[i] >= g->nz || geo->rec_ix[i] < 0 || geo->rec_ix[i] >= g->nx)
      return set_err(ctx, FWIME_EINVAL, "receiver " + std::to_string(i) + " outside the model grid");
  }
  return FWIME_OK;
}

int check_nh(fwime_ctx_t *ctx, const fwime_grid_t *g, int nh) {
  if (nh < 1 || nh % 2 == 0 || nh > 2 * g->nx - 1)
    return set_err(ctx, FWIME_EINVAL, "nh must be odd with 1 <= nh <= 2 nx - 1");
  return FWIME_OK;
}

// Pinned host space for at least n doubles of reduction results.
int host_red_reserve(fwime_ctx_t *ctx, size_t n) {
  if (n <= ctx->host_red_n) return FWIME_OK;
  if (ctx->fixed) return set_err(ctx, FWIME_ENOMEM, "too many arrays to validate without allocating");
  if (ctx->host_red) HIPCHK(hipHostFree(ctx->host_red));
  ctx->host_red = nullptr;
  ctx->host_red_n = 0;
  const size_t want = std::max<size_t>(n, 64);
  HIPCHK(hipHostMalloc((void **)&ctx->host_red, want * sizeof(double), hipHostMallocDefault));
  ctx->host_red_n = want;
  return FWIME_OK;
}

// min / max / non-finite count of several device arrays: one launch for up to
// kRangeArrays of them, whose workgroups write their triples to pinned host
// memory, and one stream synchronization.  out[3 k .. 3 k + 2] describe array k.
constexpr int kRangeBlocks = 2048;       // workgroups for all arrays, and one more per array
int device_ranges(fwime_ctx_t *ctx, const std::vector<std::pair<const float *, long>> &arrays, hipStream_t st,
                  std::vector<double> &out) {
  const size_t n = arrays.size();
  double all = 0.0;
  for (auto &a : arrays) {
    if (!a.first) return set_err(ctx, FWIME_EINVAL, "input pointer is null");
    all += (double)a.second;
  }
  int rc;
  if ((rc = host_red_reserve(ctx, 3 * (kRangeBlocks + n)))) return rc;
  std::vector<int> first(n + 1, 0);      // workgroups before array k
  for (size_t k = 0; k < n; ++k) {
    const long share = (long)(kRangeBlocks * ((double)arrays[k].second / std::max(all, 1.0)));
    first[k + 1] = first[k] + (int)std::max(1L, std::min(share, (arrays[k].second + 2047) / 2048));
  }
  for (size_t k0 = 0; k0 < n; k0 += kRangeArrays) {
    RangeArgs r;
    r.count = (int)std::min<size_t>(kRangeArrays, n - k0);
    for (int k = 0; k < r.count; ++k) {
      r.a[k] = arrays[k0 + k].first;
      r.n[k] = arrays[k0 + k].second;
      r.block0[k] = first[k0 + k] - first[k0];
    }
    r.block0[r.count] = first[k0 + r.count] - first[k0];
    HIPCHK(launch_ranges(r, ctx->host_red + 3L * first[k0], st));
  }
  HIPCHK(hipStreamSynchronize(st));
  out.resize(3 * n);
  for (size_t k = 0; k < n; ++k) {
    double mn = INFINITY, mx = -INFINITY, bad = 0.0;
    for (int b = first[k]; b < first[k + 1]; ++b) {
      mn = std::min(mn, ctx->host_red[3 * b]);
      mx = std::max(mx, ctx->host_red[3 * b + 1]);
      bad += ctx->host_red[3 * b + 2];
    }
    out[3 * k] = mn;
    out[3 * k + 1] = mx;
    out[3 * k + 2] = bad;
  }
  return FWIME_OK;
}

// Velocity range (positive, finite, CFL) from its min / max / non-finite triple.
int check_velocity_range(fwime_ctx_t *ctx, const fwime_grid_t *g, const double *r) {
  if (r[2] > 0) return set_err(ctx, FWIME_ENONFINITE, "vel has non-finite values");
  if (!(r[0] > 0)) return set_err(ctx, FWIME_EINVAL, "velocity must be positive");
  if (r[1] * g->dt > cfl_limit(g->dz, g->dx) * (1 + 1e-12))
    return set_err(ctx, FWIME_EINVAL, "CFL condition violated: v_max dt = " + std::to_string(r[1] * g->dt) +
                                          " > " + std::to_string(cfl_limit(g->dz, g->dx)));
  return FWIME_OK;
}

// Common prologue: validates velocity (positive, finite, CFL), the wavelets
// and the other float inputs in one device pass and one synchronization;
// runs before any output is touched.
int check_inputs(fwime_ctx_t *ctx, const fwime_grid_t *g, const float *vel, const fwime_geom_t *geo,
                 std::vector<std::pair<const float *, long>> extra, hipStream_t st) {
  if (!vel) return set_err(ctx, FWIME_EINVAL, "vel is null");
  std::vector<std::pair<const float *, long>> arrays{{vel, (long)g->nx * g->nz},
                                                     {geo->wavelet, (long)geo->nshots * g->nt}};
  arrays.insert(arrays.end(), extra.begin(), extra.end());
  std::vector<double> r;
  int rc = device_ranges(ctx, arrays, st, r);
  if (rc) return rc;
  if ((rc = check_velocity_range(ctx, g, r.data()))) return rc;
  for (size_t k = 1; k < arrays.size(); ++k)
    if (r[3 * k + 2] > 0) return set_err(ctx, FWIME_ENONFINITE, "input array has non-finite values");
  return FWIME_OK;
}

// ---------------------------------------------------------------------------
// Geometry tables for one batch of shots [s0, s0 + S).  Indices stored in the
// tables are batch-local (shot s, receiver s * nrec + r); callers offset the
// wavelet and data pointers to the batch start.
// ---------------------------------------------------------------------------
// One-step tiling (64-row tiles): src / rinj lists per (tile, wave) on the
// tile, rext per tile.  Two-step tiling (56-row tiles): src / rinj are the
// step-2 lists on the tile, src1 / rinj1 the step-1 lists over the tile plus
// a 4-cell halo, rext per tile.
struct HostTables {
  std::vector<int> src_ptr, rext_ptr, rinj_ptr, cells, src1_ptr, rinj1_ptr;
  std::vector<int2> src_ent, rext_ent, rinj_ent, src1_ent, rinj1_ent;
};

struct DevTables {
  int *src_ptr, *rext_ptr, *rinj_ptr, *cells, *src1_ptr, *rinj1_ptr;
  int2 *src_ent, *rext_ent, *rinj_ent, *src1_ent, *rinj1_ent;
};

void csr_build(std::vector<int> &ptr, std::vector<int2> &ent, long nbucket,
               const std::vector<std::pair<long, int2>> &items) {
  ptr.assign(nbucket + 1, 0);
  for (auto &it : items) ptr[it.first + 1]++;
  for (long b = 0; b < nbucket; ++b) ptr[b + 1] += ptr[b];
  ent.resize(items.size());
  std::vector<int> fill(ptr.begin(), ptr.end() - 1);
  for (auto &it : items) ent[fill[it.first]++] = it.second;
  // inject lists are consumed in column order by each wave
  for (long b = 0; b < nbucket; ++b)
    std::stable_sort(ent.begin() + ptr[b], ent.begin() + ptr[b + 1],
                     [](const int2 &a, const int2 &c) { return (a.x >> 6) < (c.x >> 6); });
}

// kInjRepeat on every entry of a bucket that names a cell twice (buckets are
// sorted by column: only entries of one column can name the same cell)
void mark_repeats(const std::vector<int> &ptr, std::vector<int2> &ent) {
  for (size_t b = 0; b + 1 < ptr.size(); ++b) {
    bool repeat = false;
    uint64_t rows = 0;
    for (int e = ptr[b]; e < ptr[b + 1]; ++e) {
      if (e > ptr[b] && (ent[e].x >> 6) != (ent[e - 1].x >> 6)) rows = 0;
      const uint64_t bit = 1ull << (ent[e].x & 63);
      repeat = repeat || (rows & bit);
      rows |= bit;
    }
    if (repeat)
      for (int e = ptr[b]; e < ptr[b + 1]; ++e) ent[e].x |= kInjRepeat;
  }
}

HostTables build_tables(const Dims &d, const fwime_geom_t *geo, int s0, int S) {
  HostTables t;
  const int CPW = d.TX / kWaves;
  const long ntiles = (long)d.ntz * d.ntx * S;
  auto locate = [&](int s, int px, int pz, long &tile, int &lx, int &lz) {
    const int txi = px / d.TX, tzi = pz / kTZ;
    tile = tile_index(txi, tzi, s, d.ntz, d.ntx, S);
    lx = px - txi * d.TX;
    lz = pz - tzi * kTZ;
  };
  std::vector<std::pair<long, int2>> src, rext, rinj;
  for (int s = 0; s < S; ++s) {
    const int sg = s0 + s;
    long tile;
    int lx, lz;
    locate(s, geo->src_ix[sg] + d.nb, geo->src_iz[sg] + d.nb, tile, lx, lz);
    src.push_back({tile * kWaves + lx / CPW, make_int2(((lx % CPW) << 6) | lz, s)});
    for (int r = 0; r < geo->nrec; ++r) {
      const long ir = (long)sg * geo->nrec + r;      // global receiver (geometry lookup)
      const int il = s * geo->nrec + r;              // batch-local receiver (table index)
      const int px = geo->rec_ix[ir] + d.nb, pz = geo->rec_iz[ir] + d.nb;
      locate(s, px, pz, tile, lx, lz);
      rext.push_back({tile, make_int2((lx << 6) | lz, il)});
      rinj.push_back({tile * kWaves + lx / CPW, make_int2(((lx % CPW) << 6) | lz, il)});
      t.cells.push_back(px * d.LZ + pz);
    }
  }
  csr_build(t.src_ptr, t.src_ent, ntiles * kWaves, src);
  csr_build(t.rext_ptr, t.rext_ent, ntiles, rext);
  csr_build(t.rinj_ptr, t.rinj_ent, ntiles * kWaves, rinj);
  return t;
}

// Two-step tiling: a cell (px, pz) lies on the tile (txi, tzi) with
// txi = px / TX, tzi = pz / 56, and in the step-1 region (tile plus 4-cell
// halo) of every tile whose [x0 - 4, x0 + TX + 4) x [z0 - 4, z0 + 60) holds it.
HostTables build_tables2(const Dims &d, const fwime_geom_t *geo, int s0, int S) {
  HostTables t;
  const int W1 = (d.TX + 2 * kR) / kWaves, W2 = d.TX / kWaves;
  const long ntiles = (long)d.ntz2 * d.ntx * S;
  auto tile_of = [&](int s, int txi, int tzi) { return tile_index(txi, tzi, s, d.ntz2, d.ntx, S); };
  std::vector<std::pair<long, int2>> src1, src2, rext, rinj1, rinj2;
  auto add_inject = [&](int s, int px, int pz, int idx, std::vector<std::pair<long, int2>> &l1,
                        std::vector<std::pair<long, int2>> &l2) {
    const int txi = px / d.TX, tzi = pz / kTZ2;
    {
      const int lx = px - txi * d.TX, lane = pz - tzi * kTZ2 + kR;
      l2.push_back({tile_of(s, txi, tzi) * kWaves + lx / W2, make_int2(((lx % W2) << 6) | lane, idx)});
    }
    // candidate neighbours: the own tile and the ones before / after it
    for (int tx = std::max(0, txi - 1); tx <= std::min(d.ntx - 1, txi + 1); ++tx)
      for (int tz = std::max(0, tzi - 1); tz <= std::min(d.ntz2 - 1, tzi + 1); ++tz) {
        const int jj = px - (tx * d.TX - kR), lane = pz - (tz * kTZ2 - kR);
        if (jj < 0 || jj >= d.TX + 2 * kR || lane < 0 || lane >= 64) continue;
        l1.push_back({tile_of(s, tx, tz) * kWaves + jj / W1, make_int2(((jj % W1) << 6) | lane, idx)});
      }
  };
  for (int s = 0; s < S; ++s) {
    const int sg = s0 + s;
    add_inject(s, geo->src_ix[sg] + d.nb, geo->src_iz[sg] + d.nb, s, src1, src2);
    for (int r = 0; r < geo->nrec; ++r) {
      const long ir = (long)sg * geo->nrec + r;
      const int il = s * geo->nrec + r;
      const int px = geo->rec_ix[ir] + d.nb, pz = geo->rec_iz[ir] + d.nb;
      const int txi = px / d.TX, tzi = pz / kTZ2;
      rext.push_back({tile_of(s, txi, tzi), make_int2(((px - txi * d.TX) << 6) | (pz - tzi * kTZ2), il)});
      add_inject(s, px, pz, il, rinj1, rinj2);
      t.cells.push_back(px * d.LZ + pz);
    }
  }
  csr_build(t.src1_ptr, t.src1_ent, ntiles * kWaves, src1);
  csr_build(t.src_ptr, t.src_ent, ntiles * kWaves, src2);
  csr_build(t.rext_ptr, t.rext_ent, ntiles, rext);
  csr_build(t.rinj1_ptr, t.rinj1_ent, ntiles * kWaves, rinj1);
  csr_build(t.rinj_ptr, t.rinj_ent, ntiles * kWaves, rinj2);
  mark_repeats(t.src1_ptr, t.src1_ent);
  mark_repeats(t.src_ptr, t.src_ent);
  mark_repeats(t.rinj1_ptr, t.rinj1_ent);
  mark_repeats(t.rinj_ptr, t.rinj_ent);
  return t;
}

// Four-step tiling: one list per (tile, wave) for every step, over the tile plus
// the kHalo4 cells around it that the first step computes; rext per tile.
HostTables build_tables4(const Dims &d, const fwime_geom_t *geo, int s0, int S) {
  HostTables t;
  const int W = (d.TX4 + 2 * kHalo4) / kWaves4;
  const long ntiles = (long)d.ntz4 * d.ntx4 * S;
  auto tile_of = [&](int s, int txi, int tzi) { return tile_index4(txi, tzi, s, d.ntz4, d.ntx4); };
  std::vector<std::pair<long, int2>> src, rext, rinj;
  auto add_inject = [&](int s, int px, int pz, int idx, std::vector<std::pair<long, int2>> &l) {
    const int rx = (kHalo4 + d.TX4 - 1) / d.TX4, txi = px / d.TX4, tzi = pz / kTZ4;   // the halo reaches rx tiles
    for (int tx = std::max(0, txi - rx); tx <= std::min(d.ntx4 - 1, txi + rx); ++tx)
      for (int tz = std::max(0, tzi - 1); tz <= std::min(d.ntz4 - 1, tzi + 1); ++tz) {
        const int jj = px - (tx * d.TX4 - kHalo4), lane = pz - (tz * kTZ4 - kHalo4);
        if (jj < 0 || jj >= d.TX4 + 2 * kHalo4 || lane < 0 || lane >= 64) continue;
        l.push_back({tile_of(s, tx, tz) * kWaves4 + jj / W, make_int2(((jj % W) << 6) | lane, idx)});
      }
  };
  for (int s = 0; s < S; ++s) {
    const int sg = s0 + s;
    add_inject(s, geo->src_ix[sg] + d.nb, geo->src_iz[sg] + d.nb, s, src);
    for (int r = 0; r < geo->nrec; ++r) {
      const long ir = (long)sg * geo->nrec + r;
      const int il = s * geo->nrec + r;
      const int px = geo->rec_ix[ir] + d.nb, pz = geo->rec_iz[ir] + d.nb;
      const int txi = px / d.TX4, tzi = pz / kTZ4;
      rext.push_back({tile_of(s, txi, tzi), make_int2(((px - txi * d.TX4) << 6) | (pz - tzi * kTZ4), il)});
      add_inject(s, px, pz, il, rinj);
      t.cells.push_back(px * d.LZ + pz);
    }
  }
  csr_build(t.src_ptr, t.src_ent, ntiles * kWaves4, src);
  csr_build(t.rext_ptr, t.rext_ent, ntiles, rext);
  csr_build(t.rinj_ptr, t.rinj_ent, ntiles * kWaves4, rinj);
  mark_repeats(t.src_ptr, t.src_ent);
  mark_repeats(t.rinj_ptr, t.rinj_ent);
  return t;
}

size_t tables_ints(const HostTables &t) {
  return t.src_ptr.size() + t.rext_ptr.size() + t.rinj_ptr.size() + t.cells.size() + t.src1_ptr.size() +
         t.rinj1_ptr.size() +
         2 * (t.src_ent.size() + t.rext_ent.size() + t.rinj_ent.size() + t.src1_ent.size() + t.rinj1_ent.size()) +
         11 * 64;
}

// Lay out all batch tables into one host blob and one device buffer.
struct TableSet {
  std::vector<HostTables> host;
  std::vector<DevTables> dev;
  std::vector<int> blob;
};

TableSet build_table_set(const Dims &d, const fwime_geom_t *geo, const std::vector<std::pair<int, int>> &batches,
                         bool two_step = false) {
  TableSet ts;
  for (auto &b : batches)
    ts.host.push_back(!two_step    ? build_tables(d, geo, b.first, b.second)
                      : d.T == 4 ? build_tables4(d, geo, b.first, b.second)
                                 : build_tables2(d, geo, b.first, b.second));
  return ts;
}

size_t table_set_ints(const TableSet &ts) {
  size_t n = 0;
  for (auto &t : ts.host) n += tables_ints(t);
  return n;
}

// Appends the tables to `blob` (pieces on 64-int boundaries) and points
// ts.dev into its device copy, whose first int is at `dev`.
void layout_tables(TableSet &ts, std::vector<int> &blob, int *dev) {
  ts.dev.clear();
  auto put = [&](const void *src, size_t nint) -> int * {
    const size_t off = (blob.size() + 63) / 64 * 64;
    blob.resize(off + nint);
    if (nint) std::memcpy(blob.data() + off, src, nint * sizeof(int));
    return dev + off;
  };
  for (auto &t : ts.host) {
    DevTables dt;
    dt.src_ptr = put(t.src_ptr.data(), t.src_ptr.size());
    dt.rext_ptr = put(t.rext_ptr.data(), t.rext_ptr.size());
    dt.rinj_ptr = put(t.rinj_ptr.data(), t.rinj_ptr.size());
    dt.cells = put(t.cells.data(), t.cells.size());
    dt.src_ent = (int2 *)put(t.src_ent.data(), 2 * t.src_ent.size());
    dt.rext_ent = (int2 *)put(t.rext_ent.data(), 2 * t.rext_ent.size());
    dt.rinj_ent = (int2 *)put(t.rinj_ent.data(), 2 * t.rinj_ent.size());
    dt.src1_ptr = put(t.src1_ptr.data(), t.src1_ptr.size());
    dt.src1_ent = (int2 *)put(t.src1_ent.data(), 2 * t.src1_ent.size());
    dt.rinj1_ptr = put(t.rinj1_ptr.data(), t.rinj1_ptr.size());
    dt.rinj1_ent = (int2 *)put(t.rinj1_ent.data(), 2 * t.rinj1_ent.size());
    ts.dev.push_back(dt);
  }
}

// sync = false: the copy may still read ts.blob after the call returns, so
// the caller keeps ts alive until the stream has passed the copy.
int upload_tables(fwime_ctx_t *ctx, TableSet &ts, int *dev, hipStream_t st, bool sync = true) {
  ts.blob.clear();
  layout_tables(ts, ts.blob, dev);
  // With sync the blob is copied synchronously (pageable memory): the call
  // owns no host staging that could outlive it.
  HIPCHK(hipMemcpyAsync(dev, ts.blob.data(), ts.blob.size() * sizeof(int), hipMemcpyHostToDevice, st));
  if (sync) HIPCHK(hipStreamSynchronize(st));
  return FWIME_OK;
}

// ---------------------------------------------------------------------------
// Shared per-call state
// ---------------------------------------------------------------------------
struct Common {
  Dims d;
  float *V = nullptr, *gz = nullptr, *gx = nullptr;
  int *tables = nullptr;
  StepArgs base;
};

void taper_host(int n, int nb, double alpha, int len, std::vector<float> &out) {
  out.assign(len, 0.f);
  for (int i = 0; i < n + 2 * nb; ++i) {
    int k = 0;
    if (i < nb) k = nb - i;
    else if (i >= nb + n) k = i - (nb + n - 1);
    const double a = nb > 0 ? alpha * k / nb : 0.0;
    out[i] = (float)std::exp(-a * a);
  }
}

// step arguments shared by every launch of a call
void common_args(Common &c, const fwime_grid_t *g) {
  const Dims &d = c.d;
  StepArgs &a = c.base;
  a = StepArgs();
  a.V = c.V;
  a.gz = c.gz;
  a.gx = c.gx;
  a.NZ = d.NZ;
  a.NX = d.NX;
  a.LZ = d.LZ;
  a.ntz = d.ntz;
  a.ntx = d.ntx;
  a.fs = g->free_surface ? d.nb : -1;
  const double idz2 = 1.0 / (g->dz * g->dz), idx2 = 1.0 / (g->dx * g->dx);
  for (int k = 0; k < kR; ++k) {
    a.cz[k] = (float)(kW[k + 1] * idz2);
    a.cx[k] = (float)(kW[k + 1] * idx2);
  }
}

int setup_common(fwime_ctx_t *ctx, Common &c, const fwime_grid_t *g, const float *vel, hipStream_t st) {
  const Dims &d = c.d;
  HIPCHK(launch_prep(vel, d.nz, d.nx, d.nb, d.NZ, d.NX, d.LZ, (float)g->dt, c.V, st));
  std::vector<float> gz, gx;
  taper_host(d.nz, d.nb, g->sponge_alpha, d.LZ, gz);
  taper_host(d.nx, d.nb, g->sponge_alpha, d.NX + kGxPad, gx);
  HIPCHK(hipMemcpyAsync(c.gz, gz.data(), gz.size() * sizeof(float), hipMemcpyHostToDevice, st));
  HIPCHK(hipMemcpyAsync(c.gx, gx.data(), gx.size() * sizeof(float), hipMemcpyHostToDevice, st));
  common_args(c, g);
  return FWIME_OK;
}

// Step-argument helpers for one batch.
StepArgs batch_args(const Common &c, int S, long sstride) {
  StepArgs a = c.base;
  a.nshots = S;
  a.sstride = sstride;
  return a;
}

void with_src_w(StepArgs &a, const DevTables &t, const float *wav_b, const fwime_grid_t *g, int n) {
  a.inj.ptr = t.src_ptr;
  a.inj.ent = t.src_ent;
  a.inj.val = wav_b;
  a.inj.stride_idx = g->nt;
  a.inj.t = n;
  a.inj.scale = (float)(1.0 / (g->dx * g->dz));
}

void with_src(StepArgs &a, const DevTables &t, const fwime_geom_t *geo, const fwime_grid_t *g, int s0, int n) {
  with_src_w(a, t, geo->wavelet + (long)s0 * g->nt, g, n);
}

void with_rec_inject(StepArgs &a, const DevTables &t, const float *data, int nt, int k) {
  a.inj.ptr = t.rinj_ptr;
  a.inj.ent = t.rinj_ent;
  a.inj.val = data;
  a.inj.stride_idx = nt;
  a.inj.t = k;
  a.inj.scale = 1.f;
}

void with_rec_extract(StepArgs &a, const DevTables &t, float *data, int nt, int n) {
  a.ext.ptr = t.rext_ptr;
  a.ext.ent = t.rext_ent;
  a.ext.out = data;
  a.ext.stride_idx = nt;
  a.ext.t = n;
}

// Four field buffers of one batch: prev = f[i], cur = f[i + 1]; a launch
// writes the last two fields it forms (its only one) to f[i + 2] and f[i + 3]
// (f[i + 2]) and advances i by as many.  No output buffer is read by that
// launch, and after it u^{n-1} and u^n are still in memory.
template <class T>
struct Ring4T {
  T *f[4];
  int i = 0;
  Ring4T(T *base, long stride) {
    for (int k = 0; k < 4; ++k) f[k] = base + k * stride;
  }
  T *at(int k) const { return f[(i + k) & 3]; }
  T *prev() const { return at(0); }
  T *cur() const { return at(1); }
  // outputs of a launch of k steps
  void outputs(T **out, int k) const {
    for (int q = 0; q < k; ++q) out[q] = q < k - 2 ? nullptr : at(q - std::max(0, k - 2) + 2);
  }
  void advance(int k) { i += std::min(k, 2); }
};
using Ring4 = Ring4T<float>;
using Ring4L = Ring4T<unsigned short>;   // BF16 low parts of an extended-precision field

// One launch of up to d.T time steps, whichever kernel runs it: fields, outputs
// and dense sources as in Step4Args, and what is injected and recorded.
struct Steps : Step4Args {
  const DevTables *tab = nullptr;        // the batch's lists
  enum { kNone, kSource, kReceivers } inject = kNone;
};

// point sources, from time n on
void with_src2(Steps &q, const DevTables &t, const float *wav_b, const fwime_grid_t *g, int n) {
  q.tab = &t;
  q.inject = Steps::kSource;
  q.inj.val = wav_b;
  q.inj.stride_idx = g->nt;
  q.inj.t = n;
  q.inj.scale = (float)(1.0 / (g->dx * g->dz));
  q.inj_dt = 1;
}

// the same for a two-step job descriptor: step-1 list at time n, step-2 list at time n + 1
void with_src2(Step2Args &p, const DevTables &t, const float *wav_b, const fwime_grid_t *g, int n) {
  with_src_w(p.a, t, wav_b, g, n);
  p.a.inj.ptr = t.src1_ptr;
  p.a.inj.ent = t.src1_ent;
  p.inj2 = p.a.inj;
  p.inj2.ptr = t.src_ptr;
  p.inj2.ent = t.src_ent;
  p.inj2.t = n + 1;
}

// receiver injection (adjoint sources): times k, k - 1, ... of `data`
void with_rec_inject2(Steps &q, const DevTables &t, const float *data, int nt, int k) {
  q.tab = &t;
  q.inject = Steps::kReceivers;
  q.inj.val = data;
  q.inj.stride_idx = nt;
  q.inj.t = k;
  q.inj.scale = 1.f;
  q.inj_dt = -1;
}

// records the fields of times n, n + 1, ... that the launch reads
void with_rec_extract(Steps &q, const DevTables &t, float *data, int nt, int n) {
  q.tab = &t;
  q.ext.out = data;
  q.ext.stride_idx = nt;
  q.ext.t = n;
}

// T2 output: slot `first` for the first step, the next slots (`slot` elements
// on) for the others; per-shot stride sstride
void with_t2(Steps &q, float *first, long slot, int k, long sstride) {
  for (int i = 0; i < k; ++i) q.t2[i] = first + i * slot;
  q.t2_sstride = sstride;
}

// rows and columns on which the offset scatter (or, with H = 0, the lag
// scatter) writes its output: the model's rows, the model's columns and the H
// columns on either side that lie on the grid
void with_dense_range(Steps &q, const ExtGeom &eg, int H) {
  q.ez0 = eg.nb;
  q.ez1 = eg.nb + eg.nz;
  q.ex0 = std::max(0, eg.nb - H);
  q.ex1 = std::min(eg.NX, eg.nb + eg.nx + H);
}

// dense source: slot `first` for the first step, the next slots for the others
void with_dsrc2(Steps &q, const float *first, long slot, int k, long sstride) {
  for (int i = 0; i < k; ++i) q.ds[i] = first + i * slot;
  q.ds_sstride = sstride;
}

// transposed second time difference of e as the source of the steps that read
// times k, k - 1, ...; slot(t): the e slot of time t
template <class Slot>
void with_nu(Steps &q, Slot slot, int k, int kk, long sstride) {
  for (int i = 0; i < kk + 2; ++i) q.ds[i] = slot(k + 1 - i);
  q.ds_sstride = sstride;
}

// Launches k steps for S shots.
hipError_t launch_steps(const Common &c, Steps &q, int S, long sstride, int k, int mode, hipStream_t st) {
  const Dims &d = c.d;
  const StepArgs &b = c.base;
  if (d.T == 4) {
    q.V = b.V;
    q.gz = b.gz;
    q.gx = b.gx;
    q.NZ = b.NZ;
    q.NX = b.NX;
    q.LZ = b.LZ;
    q.fs = b.fs;
    std::copy(b.cz, b.cz + kR, q.cz);
    std::copy(b.cx, b.cx + kR, q.cx);
    q.nshots = S;
    q.sstride = sstride;
    q.ntz = d.ntz4;
    q.ntx = d.ntx4;
    q.steps = k;
    if (q.inject != Steps::kNone) {
      q.inj.ptr = q.inject == Steps::kSource ? q.tab->src_ptr : q.tab->rinj_ptr;
      q.inj.ent = q.inject == Steps::kSource ? q.tab->src_ent : q.tab->rinj_ent;
    }
    if (q.ext.out) {
      q.ext.ptr = q.tab->rext_ptr;
      q.ext.ent = q.tab->rext_ent;
    }
    return launch_step4(q, d.TX4, mode, st);
  }
  Step2Args p;
  p.a = batch_args(c, S, sstride);
  p.a.ntz = d.ntz2;
  p.a.prev = q.prev;
  p.a.cur = q.cur;
  p.a.out = q.out[0];
  p.out2 = q.out[1];
  p.two = k == 2;
  p.lo_prev = q.lo_prev;
  p.lo_cur = q.lo_cur;
  p.lo_out = q.lo_out[0];
  p.lo_out2 = q.lo_out[1];
  p.a.t2 = q.t2[0];
  p.t2b = q.t2[1];
  p.a.t2_sstride = q.t2_sstride;
  if (mode & kModeDsrc) {
    p.a.dsrc = q.ds[0];
    p.dsrc2 = q.ds[1];
    p.a.dsrc_sstride = q.ds_sstride;
  } else if (mode & kModeNu) {
    p.a.nu = NuSource{q.ds[2], q.ds[1], q.ds[0], q.ds_sstride};
    if (k == 2) p.nu2 = NuSource{q.ds[3], q.ds[2], q.ds[1], q.ds_sstride};
  }
  p.a.ez0 = q.ez0;
  p.a.ez1 = q.ez1;
  p.a.ex0 = q.ex0;
  p.a.ex1 = q.ex1;
  if (q.inject != Steps::kNone) {
    const bool src = q.inject == Steps::kSource;
    p.a.inj = p.inj2 = q.inj;
    p.a.inj.ptr = src ? q.tab->src1_ptr : q.tab->rinj1_ptr;
    p.a.inj.ent = src ? q.tab->src1_ent : q.tab->rinj1_ent;
    p.inj2.ptr = src ? q.tab->src_ptr : q.tab->rinj_ptr;
    p.inj2.ent = src ? q.tab->src_ent : q.tab->rinj_ent;
    p.inj2.t = q.inj.t + q.inj_dt;
  }
  if (q.ext.out) {
    p.a.ext = q.ext;
    p.a.ext.ptr = q.tab->rext_ptr;
    p.a.ext.ent = q.tab->rext_ent;
  }
  return launch_step2(p, d.TX, mode, st);
}

// Advances ring f over the steps n0 .. n1 - 1 forward in time, d.T steps per
// launch and what is left in the last.  setup(q, n, k) adds the arguments of
// the launch that starts at step n and takes k steps.
// With lo != nullptr the field is carried in extended precision (mode gets
// kModeDF) and lo rotates with f.  Counts its launches in *launches.
template <class Setup>
int march2(fwime_ctx_t *ctx, const Common &c, Ring4 &f, int S, int n0, int n1, int mode, Setup setup,
           hipStream_t st, Ring4L *lo = nullptr, long *launches = nullptr) {
  for (int n = n0; n < n1;) {
    const int k = std::min(c.d.T, n1 - n);
    Steps q;
    q.prev = f.prev();
    q.cur = f.cur();
    f.outputs(q.out, k);
    if (lo) {
      q.lo_prev = lo->prev();
      q.lo_cur = lo->cur();
      lo->outputs(q.lo_out, k);
    }
    setup(q, n, k);
    HIPCHK(launch_steps(c, q, S, c.d.field, k, lo ? (mode | kModeDF) : mode, st));
    f.advance(k);
    if (lo) lo->advance(k);
    n += k;
    if (launches) ++*launches;
  }
  return FWIME_OK;
}

// u^{-1} = u^0 = 0: the two buffers of a four-buffer ring that the first launch reads
hipError_t zero_start(float *ring, const Dims &d, int S, hipStream_t st) {
  return launch_zero(ring, 2 * d.field * S, st);
}
hipError_t zero_start(unsigned short *ring_lo, const Dims &d, int S, hipStream_t st) {
  return launch_zero((float *)ring_lo, d.field * S, st);
}

// the fields of times nt - 1 and nt (the zero start of a backward recursion)
// in a ring of R slots
hipError_t zero_end(float *ring, long ring_stride, int R, const Dims &d, int S, hipStream_t st) {
  hipError_t e = launch_zero_fields(ring + (long)((d.nt - 1) % R) * d.field, ring_stride, S, d.field, st);
  return e != hipSuccess ? e : launch_zero_fields(ring + (long)(d.nt % R) * d.field, ring_stride, S, d.field, st);
}
hipError_t zero_end(unsigned short *ring, long ring_stride, int R, const Dims &d, int S, hipStream_t st) {
  hipError_t e = launch_zero_fields((float *)(ring + (long)((d.nt - 1) % R) * d.field), ring_stride / 2, S, d.field / 2, st);
  return e != hipSuccess ? e
                         : launch_zero_fields((float *)(ring + (long)(d.nt % R) * d.field), ring_stride / 2, S,
                                              d.field / 2, st);
}

// BF16 arrays copied as 32-bit words (fields hold an even number of cells)
hipError_t copy_lo(unsigned short *dst, long dst_sstride, const unsigned short *src, long src_sstride, int S, long n,
                   hipStream_t st) {
  return launch_copy_fields((float *)dst, dst_sstride / 2, (const float *)src, src_sstride / 2, S, n / 2, st);
}

// Adjoint recursion over a ring of R field slots (slot of time k: k % R),
// from time k = k1 down to k0 + 1, producing the fields of times k1 - 1 ..
// k0: d.T steps per launch (no more than the slots a launch does not read).
// setup(q, k, kk) adds the sources of the launch that starts at time k and
// takes kk steps.
// With lo != nullptr (a BF16 ring of the same shape) the field is carried in
// extended precision (mode gets kModeDF).
template <class Setup>
int march2_back_ring(fwime_ctx_t *ctx, const Common &c, float *ring, long ring_stride, int R, int S, int k0, int k1,
                     int mode, Setup setup, hipStream_t st, unsigned short *lo = nullptr) {
  const long F = c.d.field;
  const int most = std::min(c.d.T, R - 2);
  for (int k = k1; k >= k0 + 1;) {
    const int kk = std::min(most, k - k0);
    Steps q;
    q.cur = ring + (long)(k % R) * F;
    q.prev = ring + (long)((k + 1) % R) * F;
    for (int i = 0; i < kk; ++i) q.out[i] = ring + (long)((k - 1 - i) % R) * F;
    if (lo) {
      q.lo_cur = lo + (long)(k % R) * F;
      q.lo_prev = lo + (long)((k + 1) % R) * F;
      for (int i = 0; i < kk; ++i) q.lo_out[i] = lo + (long)((k - 1 - i) % R) * F;
    }
    setup(q, k, kk);
    HIPCHK(launch_steps(c, q, S, ring_stride, kk, lo ? (mode | kModeDF) : mode, st));
    k -= kk;
  }
  return FWIME_OK;
}

// lambda: receiver injection of `data` at the current time
int march2_back_lambda(fwime_ctx_t *ctx, const Common &c, float *ring, long ring_stride, int R, int S, int k0,
                       int k1, const DevTables &t, const float *data, int nt, hipStream_t st,
                       unsigned short *lo = nullptr) {
  return march2_back_ring(ctx, c, ring, ring_stride, R, S, k0, k1, kModePlain,
                          [&](Steps &q, int k, int) { with_rec_inject2(q, t, data, nt, k); }, st, lo);
}

int choose_batch(fwime_ctx_t *ctx, long per_shot_bytes, size_t fixed_bytes, int nshots) {
  size_t cap = 0;
  if (ctx->fixed) {
    cap = ctx->fixed_bytes;                // the static scratch array is all there is
  } else {
    size_t avail = 0, total = 0;
    if (hipMemGetInfo(&avail, &total) != hipSuccess) avail = 0;
    avail += ctx->arena_bytes + spare_bytes(ctx);   // the arena can be reused, the spare given back
    cap = (size_t)(avail * 0.85);
    if (ctx->budget && ctx->budget < cap) cap = ctx->budget;
  }
  if (cap <= fixed_bytes) return 1;
  long S = (long)((cap - fixed_bytes) / std::max<long>(per_shot_bytes, 1));
  S = std::max<long>(1, std::min<long>(S, nshots));
  return (int)S;
}

std::vector<std::pair<int, int>> split_batches(int nshots, int S) {
  std::vector<std::pair<int, int>> b;
  const int nb = (nshots + S - 1) / S;
  const int base = nshots / nb, extra = nshots % nb;   // balanced batch sizes
  int s0 = 0;
  for (int i = 0; i < nb; ++i) {
    const int n = base + (i < extra ? 1 : 0);
    b.push_back({s0, n});
    s0 += n;
  }
  return b;
}

// Segment length of the sqrt(nt) checkpointing, rounded up to an even count
// so two-step launches never straddle a segment start.
int seg_len(int nt) {
  int K = (int)std::ceil(std::sqrt((double)(nt - 1)));
  K = std::max(K, 1);
  return K + (K & 1);
}

// ---------------------------------------------------------------------------
// Whole T2 histories.  The adjoint-state operators need T2u_n (and T2du~_n)
// of every step backwards in time.  Where the memory is there, a batch keeps
// them whole instead of checkpointing the fields and propagating them again:
// the gradient then runs four propagations per shot instead of six and one
// offset scatter instead of two, the adjoint two instead of three.  Without
// checkpoints the segment length is free: long segments spread the offset
// kernels' weight loads over more time slots.  They hold whole checkpointed
// segments, and images and gradient sums are formed segment by segment inside
// them, so a result has the same bits with histories and with checkpoints.
//
// Only a context without a budget does so (one with a budget shares the device
// by exact footprints), and what it then holds for histories, in its arena, the
// solver's buffer, live tapes and the spare together, stays within a third of
// the device memory that others leave.  Where a history does not fit beside the
// others, the call checkpoints: allocating costs about 15 ms a gigabyte, ten
// times what a gigabyte of history saves a call, so buffers are not freed for
// one another from call to call.  One that the last kIdleCalls calls did
// without is.  All shots of the call must fit, or at least enough of them that a
// launch still fills the device.
// ---------------------------------------------------------------------------
constexpr long kIdleCalls = 16;
// Time slots (shots x steps) of a segment.  Measured, ms, with one checkpointed
// segment / 256 / 1024 / 4096 slots: gradient 300 x 1700, nh 61, 8 shots 140.6 /
// 137.0 / 133.8 / 129.5; Born pair 157.3 / 154.6 / 153.3 / 152.0; gradient 200 x 600,
// nh 11, 4 shots 34.1 / 34.1 / 34.0 / 34.0; autograd 100 x 200 14.5 / 13.4 / 13.4 /
// 13.3.  The rings of a segment take memory from the histories.
constexpr long kHistSlots = 1024;
// Two-step workgroups of a batch from which histories in several batches are
// taken rather than checkpoints in one, which fill the device better.  Measured,
// ms, gradient and Born adjoint, nt = 301: 300 x 1700, 12 shots, nh 61,
// checkpointed 93.5 and 55.7; batches of 784 workgroups 109.7 and 87.5, of 1176
// 89.9 and 68.4, of 1568 83.4 and 59.6, of 2352 72.4 and 49.4, all shots 64.0 and
// 40.2; 16 shots, nh 11, 106.1 and 65.6, batches of 1568 94.3 and 67.0, of 3136
// 79.8 and 52.4; 200 x 600, 24 shots, nh 41, 54.7 and 33.9, batches of 880 50.7
// and 37.2, of 1320 44.6 and 31.9.  The adjoint crosses last, near 1900; batches
// are evened out after the choice, to half of it at worst.
constexpr long kHistMinTiles = 3072;

// segment length for S shots: about kHistSlots slots in whole checkpointed
// segments, or the record (made even)
int hist_seg_len(int nt, int S) {
  const long seg = seg_len(nt), want = (kHistSlots + S - 1) / S;
  const long K = std::max(1L, (want + seg - 1) / seg) * seg;
  return (int)std::min<long>(K, (nt - 1) + ((nt - 1) & 1));
}

// Partial images of a launch that images a history segment of K steps, img
// cells an image: groups for every checkpointed segment in it, as far as 256 MB
// hold them.  (With one checkpointed segment to a launch, 100 x 200 and nh 11:
// autograd 13.66 instead of 13.29 ms, variable-projection step 41.8 instead of
// 41.1; 200 x 600 and larger the same to 0.2 %.)
constexpr long kHistPartsBytes = 256L << 20;
long hist_parts(int nt, int K, long img) {
  const long segs = (K + seg_len(nt) - 1) / seg_len(nt);
  return std::max<long>(kImageGroups, std::min<long>(segs * kImageGroups, kHistPartsBytes / (4 * img)));
}

// Shots per batch that keep whole histories (0: checkpoint instead).
// bytes(S): what the call holds for a batch of S shots; owner: the buffer that
// the history is held in (null: a tape of its own); in_arena: how much of all
// shots' is in the arena, with another owner.
template <class Bytes>
int hist_batch(fwime_ctx_t *ctx, int nshots, long tiles_per_shot, Bytes bytes, void **owner, size_t in_arena = 0) {
  if (ctx->fixed || ctx->budget || ctx->frugal) return 0;
  size_t avail = 0, total = 0;
  if (hipMemGetInfo(&avail, &total) != hipSuccess) return 0;
  if (!ctx->vp_busy) ++ctx->calls;                 // (the solver's calls are part of one)
  const size_t tapes = tape_hist_bytes(ctx), spare = spare_bytes(ctx);
  const size_t third = (avail + ctx->arena_bytes + ctx->vp_bytes + spare + live_tape_bytes(ctx)) / 3;
  // held for histories beside the call's own buffer (a tape takes the spare, a
  // small one leaves it alone), what is free or the call's own, and what of
  // the former the last calls did without
  const bool own_spare = !owner && bytes(nshots) >= spare / 4;
  const size_t arena = std::min(ctx->arena_bytes, owner == &ctx->arena ? ctx->arena_bytes : in_arena);
  const size_t idle[3] = {own_spare ? 0 : spare, owner == &ctx->vp || ctx->vp_busy ? 0 : ctx->vp_hist,
                          owner == &ctx->arena ? 0 : std::min(ctx->arena_hist, ctx->arena_bytes - arena)};
  const long now = ctx->calls, use[3] = {ctx->spare_use, ctx->vp_use, ctx->arena_use};
  size_t held = tapes + (ctx->vp_busy ? ctx->vp_hist : 0), old = 0;
  for (int i = 0; i < 3; ++i) (now - use[i] > kIdleCalls ? old : held) += idle[i];
  const size_t open = avail + old + arena + (owner == &ctx->vp ? ctx->vp_bytes : 0) + (own_spare ? spare : 0);
  const size_t cap = std::min(third > held ? third - held : 0, open / 2);   // half of it is left alone
  int S = nshots;
  if (bytes(nshots) > cap) {
    int lo = 0, hi = nshots;                       // largest S with bytes(S) <= cap
    while (hi - lo > 1) {
      const int mid = (lo + hi) / 2;
      (bytes(mid) <= cap ? lo : hi) = mid;
    }
    S = lo * tiles_per_shot >= kHistMinTiles ? lo : 0;
  }
  if (S > 0 && bytes(S) + old > cap)
    for (int i = 0; i < 3; ++i)
      if (idle[i] && now - use[i] > kIdleCalls)
        (i == 0 ? release_spare : i == 1 ? release_vp : release_arena)(ctx);
  if (S > 0 && owner == &ctx->arena) {
    ctx->arena_hist = std::max(ctx->arena_hist, bytes(S));
    if (!ctx->vp_busy) ctx->arena_use = now;
  }
  return S;
}

}  // namespace

// ===========================================================================
// C ABI
// ===========================================================================
extern "C" {

const char *fwime_strerror(int code) {
  switch (code) {
    case FWIME_OK: return "ok";
    case FWIME_EINVAL: return "invalid argument";
    case FWIME_ENOMEM: return "out of device memory or HBM budget";
    case FWIME_EHIP: return "HIP runtime error";
    case FWIME_ENONFINITE: return "non-finite input";
    default: return "unknown error";
  }
}

const char *fwime_last_error(const fwime_ctx_t *ctx) { return ctx ? ctx->err.c_str() : ""; }

}  // extern "C"

// ---------------------------------------------------------------------------
// Static scratch for the allocation-free entry point (fwime_model_static).
// In host code `scratch` names a host-side stand-in, not device memory: its
// device address is looked up once per device (fwime_ctx_create, with that
// device current) and only that address is ever passed to kernels or copies.
// Every call on a device shares its array.
// ---------------------------------------------------------------------------
static __device__ __align__(256) char scratch[FWIME_STATIC_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
char *g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on `device` (the current device).
int static_scratch_address(int device, char **out) {
  if (device < 0 || device >= kMaxDevices) return FWIME_EINVAL;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[device]) {
    void *p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
      (void)hipGetLastError();
      return FWIME_EHIP;
    }
    g_scratch_ptr[device] = (char *)p;
  }
  *out = g_scratch_ptr[device];
  return FWIME_OK;
}
}  // namespace

extern "C" {


int fwime_ctx_create(int device, size_t hbm_budget_bytes, fwime_ctx_t **out) {
  if (!out) return FWIME_EINVAL;
  *out = nullptr;
  int ndev = 0;
  if (hipGetDeviceCount(&ndev) != hipSuccess || device < 0 || device >= ndev) return FWIME_EINVAL;
  if (hipSetDevice(device) != hipSuccess) return FWIME_EHIP;
  fwime_ctx_t *ctx = new fwime_ctx_t();
  ctx->device = device;
  ctx->budget = hbm_budget_bytes;
  if (host_red_reserve(ctx, 3 * (kRangeBlocks + 64)) != FWIME_OK) {
    delete ctx;
    return FWIME_EHIP;
  }
  if (static_scratch_address(device, &ctx->static_scratch) != FWIME_OK) {
    (void)hipHostFree(ctx->host_red);
    delete ctx;
    return FWIME_EHIP;
  }
  const char *tx = std::getenv("FWIME_TILE_X");
  if (tx && step_tile_x_supported(std::atoi(tx))) ctx->tile_x = std::atoi(tx);
  // FWIME_STEP1=1: one time step per launch everywhere (same results, bit for bit)
  const char *s1 = std::getenv("FWIME_STEP1");
  if (s1 && std::atoi(s1) != 0) ctx->two_step = false;
  // FWIME_STEPS=2 or 4: that many per launch at every size (same results, bit for bit)
  const char *sn = std::getenv("FWIME_STEPS");
  if (sn && (std::atoi(sn) == 2 || std::atoi(sn) == 4)) ctx->steps = std::atoi(sn);
  *out = ctx;
  return FWIME_OK;
}

int fwime_ctx_trim(fwime_ctx_t *ctx, void *stream) {
  if (!ctx) return FWIME_EINVAL;
  if (hipSetDevice(ctx->device) != hipSuccess) return FWIME_EHIP;
  if (hipStreamSynchronize((hipStream_t)stream) != hipSuccess) return FWIME_EHIP;
  release_graph(ctx);
  if (ctx->arena && hipFree(ctx->arena) != hipSuccess) return FWIME_EHIP;
  ctx->arena = nullptr;
  release_arena(ctx);
  if (ctx->vp && hipFree(ctx->vp) != hipSuccess) return FWIME_EHIP;
  ctx->vp = nullptr;
  release_vp(ctx);
  release_spare(ctx);
  return FWIME_OK;
}

int fwime_ctx_info(const fwime_ctx_t *ctx, fwime_info_t *out) {
  if (!ctx || !out) return FWIME_EINVAL;
  out->arena_bytes = ctx->arena_bytes;
  out->tape_bytes = live_tape_bytes(ctx);
  out->tile_x = ctx->tile_x;
  out->last_batch_tile_x = ctx->last_batch_tile;
  out->tuned_signatures = (int32_t)ctx->tuned.size();
  out->last_stencil_launches = -1;
  out->last_stencil_ms = 0.0;
  if (ctx->timing && ctx->timed_launches >= 0) {
    if (hipSetDevice(ctx->device) != hipSuccess || hipEventSynchronize(ctx->tev[1]) != hipSuccess) return FWIME_EHIP;
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, ctx->tev[0], ctx->tev[1]) != hipSuccess) return FWIME_EHIP;
    out->last_stencil_launches = ctx->timed_launches;
    out->last_stencil_ms = ms;
  }
  return FWIME_OK;
}

int fwime_ctx_held(const fwime_ctx_t *ctx, size_t *bytes) {
  if (!ctx || !bytes) return FWIME_EINVAL;
  std::lock_guard<std::mutex> lock(ctx->tape_mu);
  *bytes = ctx->arena_bytes + ctx->vp_bytes + ctx->tape_bytes + ctx->spare_bytes;
  return FWIME_OK;
}

int fwime_ctx_set_timing(fwime_ctx_t *ctx, int32_t on) {
  if (!ctx) return FWIME_EINVAL;
  if (hipSetDevice(ctx->device) != hipSuccess) return FWIME_EHIP;
  if (on && !ctx->tev[0]) {
    for (auto &e : ctx->tev)
      if (hipEventCreate(&e) != hipSuccess) return set_err(ctx, FWIME_EHIP, "hipEventCreate failed");
  }
  ctx->timing = on != 0;
  ctx->timed_launches = -1;
  return FWIME_OK;
}

void fwime_ctx_destroy(fwime_ctx_t *ctx) {
  if (!ctx) return;
  (void)hipSetDevice(ctx->device);
  (void)hipDeviceSynchronize();
  release_graph(ctx);
  if (ctx->capture) (void)hipStreamDestroy(ctx->capture);
  if (ctx->arena) (void)hipFree(ctx->arena);
  if (ctx->vp) (void)hipFree(ctx->vp);
  release_spare(ctx);
  detach_tapes(ctx);
  if (ctx->host_red) (void)hipHostFree(ctx->host_red);
  for (auto &e : ctx->tev)
    if (e) (void)hipEventDestroy(e);
  delete ctx;
}

// ---------------------------------------------------------------------------
int fwime_model(fwime_ctx_t *ctx, const fwime_grid_t *g, const float *vel, const fwime_geom_t *geo, float *data,
                void *stream) {
  if (!ctx) return FWIME_EINVAL;
  ctx->err.clear();
  hipStream_t st = (hipStream_t)stream;
  int rc;
  if ((rc = check_grid(ctx, g)) || (rc = check_geom(ctx, g, geo))) return rc;
  if (!data) return set_err(ctx, FWIME_EINVAL, "data is null");
  HIPCHK(hipSetDevice(ctx->device));
  if ((rc = check_inputs(ctx, g, vel, geo, {}, st))) return rc;

  Common c;
  c.d = make_dims(g, ctx->tile_x);
  const Dims &d = c.d;
  const bool two = ctx->two_step;
  const int nf = two ? 4 : 2;                 // field buffers per shot
  const long per_shot = nf * d.field * 4 + (long)geo->nrec * 64;
  const int S = choose_batch(ctx, per_shot, (size_t)d.field * 8, geo->nshots);
  auto batches = split_batches(geo->nshots, S);
  choose_steps(ctx, c.d, S, false);
  TableSet ts = build_table_set(d, geo, batches, two);

  float *fields = nullptr;
  Carve cv;
  cv.add(&c.V, d.field);
  cv.add(&c.gz, d.LZ);
  cv.add(&c.gx, d.NX + kGxPad);
  cv.add(&c.tables, table_set_ints(ts) + 64 * batches.size() * 8);
  cv.add(&fields, nf * d.field * S);
  if ((rc = arena_get(ctx, cv)))
    return or_frugally(ctx, rc, d.T == 4, [&] { return fwime_model(ctx, g, vel, geo, data, stream); });
  if ((rc = upload_tables(ctx, ts, c.tables, st))) return rc;
  if ((rc = setup_common(ctx, c, g, vel, st))) return rc;

  HIPCHK(timing_begin(ctx, st));
  long launches = 0;
  for (size_t bi = 0; bi < batches.size(); ++bi) {
    const int s0 = batches[bi].first, Sb = batches[bi].second;
    const DevTables &t = ts.dev[bi];
    float *out_b = data + (long)s0 * geo->nrec * g->nt;
    if (!two) launches += g->nt - 1;
    if (two) {
      HIPCHK(zero_start(fields, d, Sb, st));
      Ring4 f(fields, d.field * Sb);
      rc = march2(ctx, c, f, Sb, 0, g->nt - 1, kModePlain, [&](Steps &p, int n, int) {
        with_src2(p, t, geo->wavelet + (long)s0 * g->nt, g, n);
        with_rec_extract(p, t, out_b, g->nt, n);
      }, st, nullptr, &launches);
      if (rc) return rc;
      HIPCHK(launch_gather(f.cur(), d.field, t.cells, Sb, geo->nrec, out_b, g->nt, g->nt - 1, st));
      continue;
    }
    float *A = fields, *B = fields + d.field * Sb;
    HIPCHK(launch_zero(fields, 2 * d.field * Sb, st));
    float *cur = A, *prev = B;
    for (int n = 0; n < g->nt - 1; ++n) {
      StepArgs a = batch_args(c, Sb, d.field);
      a.cur = cur;
      a.prev = prev;
      a.out = prev;
      with_src(a, t, geo, g, s0, n);
      with_rec_extract(a, t, out_b, g->nt, n);
      HIPCHK(launch_step(a, d.TX, kModePlain, st));
      std::swap(cur, prev);
    }
    HIPCHK(launch_gather(cur, d.field, t.cells, Sb, geo->nrec, out_b, g->nt, g->nt - 1, st));
  }
  HIPCHK(timing_end(ctx, st, launches));
  return FWIME_OK;
}

// ---------------------------------------------------------------------------
int fwime_model_static(fwime_ctx_t *ctx, const fwime_grid_t *g, const float *vel, const fwime_geom_t *geo,
                       float *data, void *stream) {
  if (!ctx) return FWIME_EINVAL;
  if (!ctx->static_scratch) return set_err(ctx, FWIME_EHIP, "the static scratch array has no device address");
  // every piece of scratch (validation partials, padded velocity, tapers,
  // geometry tables, wavefields) comes from the static array; shots run in as
  // many batches as it needs, and a call that cannot fit one shot fails
  // with FWIME_ENOMEM before anything is written
  ctx->fixed = ctx->static_scratch;
  ctx->fixed_bytes = FWIME_STATIC_SCRATCH_BYTES;
  const int rc = fwime_model(ctx, g, vel, geo, data, stream);
  ctx->fixed = nullptr;
  ctx->fixed_bytes = 0;
  return rc;
}

// ---------------------------------------------------------------------------
// bg: the background's T2 terms of every shot and step (shot s, step n at
// (s (nt - 1) + n) field; the variable-projection step keeps them), or null.
static int born_ext_fwd_run(fwime_ctx_t *ctx, const fwime_grid_t *g, const float *vel, const fwime_geom_t *geo,
                            int32_t nh, const float *ptilde, float *data, void *stream, const float *bg);

int fwime_born_ext_fwd(fwime_ctx_t *ctx, const fwime_grid_t *g, const float *vel, const fwime_geom_t *geo,
                       int32_t nh, const float *ptilde, float *data, void *stream) {
  return born_ext_fwd_run(ctx, g, vel, geo, nh, ptilde, data, stream, nullptr);
}

static int born_ext_fwd_run(fwime_ctx_t *ctx, const fwime_grid_t *g, const float *vel, const fwime_geom_t *geo,
                            int32_t nh, const float *ptilde, float *data, void *stream, const float *bg) {
  if (!ctx) return FWIME_EINVAL;
  ctx->err.clear();
  hipStream_t st = (hipStream_t)stream;
  int rc;
  if ((rc = check_grid(ctx, g)) || (rc = check_geom(ctx, g, geo)) || (rc = check_nh(ctx, g, nh))) return rc;
  if (!data || !ptilde) return set_err(ctx, FWIME_EINVAL, "data or ptilde is null");
  HIPCHK(hipSetDevice(ctx->device));
  if ((rc = check_inputs(ctx, g, vel, geo, {{ptilde, (long)nh * g->nx * g->nz}}, st))) return rc;

  Common c;
  c.d = make_dims(g, ctx->tile_x);
  const Dims &d = c.d;
  ExtGeom eg{d.nz, d.nx, d.nb, d.NZ, d.NX, d.LZ, nh, (nh - 1) / 2};
  const bool two = ctx->two_step;
  const int nf = two ? 8 : 4;                  // u and du~ field buffers per shot
  // two-step path: both fields also carry four BF16 low-part fields each; with
  // the background's T2 terms given, neither its fields nor their chunk
  auto per_shot = [&](int chunk) {
    return (nf + (bg ? 1L : 2L) * chunk + (two ? 4 : 0)) * d.field * 4 + (long)geo->nrec * 64;
  };
  const size_t fixed = (size_t)d.field * 8 + (size_t)nh * d.nx * d.nz * 4;
  // steps per scatter launch: 16, or long chunks where the memory is there.
  // Every workgroup of the scatter loads its offset weights once per launch:
  // at 300 x 1700, 8 shots and nh = 61 that was about half of a 16-step launch.
  const int Sh = !two ? 0 : hist_batch(ctx, geo->nshots, 0, [&](int S) {
    return fixed + (size_t)per_shot(hist_seg_len(g->nt, S)) * S;
  }, &ctx->arena);
  const int KC = Sh ? hist_seg_len(g->nt, Sh) : 16;
  const int S = Sh ? Sh : choose_batch(ctx, per_shot(KC), fixed, geo->nshots);
  auto batches = split_batches(geo->nshots, S);
  choose_steps(ctx, c.d, S, true);
  TableSet ts = build_table_set(d, geo, batches, two);

  float *coef = nullptr, *pairs = nullptr, *t2 = nullptr, *sc = nullptr;
  unsigned short *lows = nullptr;
  Carve cv;
  cv.add(&c.V, d.field);
  cv.add(&c.gz, d.LZ);
  cv.add(&c.gx, d.NX + kGxPad);
  cv.add(&c.tables, table_set_ints(ts) + 64 * batches.size() * 8);
  cv.add(&coef, (long)nh * d.nx * d.nz);
  cv.add(&pairs, nf * d.field * S);
  if (two) cv.add(&lows, 8 * d.field * S);
  if (!bg) cv.add(&t2, (long)KC * d.field * S);
  cv.add(&sc, (long)KC * d.field * S);
  if ((rc = arena_get(ctx, cv)))
    return or_frugally(ctx, rc, d.T == 4 || Sh > 0, [&] {
      return born_ext_fwd_run(ctx, g, vel, geo, nh, ptilde, data, stream, bg);
    });
  if ((rc = upload_tables(ctx, ts, c.tables, st))) return rc;
  if ((rc = setup_common(ctx, c, g, vel, st))) return rc;
  HIPCHK(launch_ext_coef(ptilde, vel, eg, (float)g->dt, coef, st));

  const long chunk_stride = (long)KC * d.field;   // per shot in t2 / sc
  for (size_t bi = 0; bi < batches.size(); ++bi) {
    const int s0 = batches[bi].first, Sb = batches[bi].second;
    const DevTables &t = ts.dev[bi];
    float *out_b = data + (long)s0 * geo->nrec * g->nt;
    if (two) {
      HIPCHK(zero_start(pairs, d, Sb, st));
      HIPCHK(zero_start(pairs + 4 * d.field * Sb, d, Sb, st));
      HIPCHK(zero_start(lows, d, Sb, st));
      HIPCHK(zero_start(lows + 4 * d.field * Sb, d, Sb, st));
      Ring4 fu(pairs, d.field * Sb), fw(pairs + 4 * d.field * Sb, d.field * Sb);
      Ring4L lu(lows, d.field * Sb), lw(lows + 4 * d.field * Sb, d.field * Sb);
      const float *wav_b = geo->wavelet + (long)s0 * g->nt;
      for (int c0 = 0; c0 < g->nt - 1; c0 += KC) {
        const int nk = std::min(KC, g->nt - 1 - c0);
        // background in extended precision: its T2 term is the scattering source
        const long bg_stride = (long)(g->nt - 1) * d.field;
        if (!bg) {
          rc = march2(ctx, c, fu, Sb, c0, c0 + nk, kModeT2, [&](Steps &p, int n, int k) {
            with_t2(p, t2 + (long)(n - c0) * d.field, d.field, k, chunk_stride);
            with_src2(p, t, wav_b, g, n);
          }, st, &lu);
          if (rc) return rc;
        }
        HIPCHK(launch_ext_scatter(coef, eg, +1, bg ? bg + s0 * bg_stride + (long)c0 * d.field : t2, d.field,
                                  bg ? bg_stride : chunk_stride, sc, d.field, chunk_stride, Sb, nk, st));
        // the scattered field in extended precision too: its FP32 rounding
        // would otherwise dominate the inconsistency of the B~ / B~^T pair
        rc = march2(ctx, c, fw, Sb, c0, c0 + nk, kModeDsrc, [&](Steps &p, int n, int k) {
          with_dsrc2(p, sc + (long)(n - c0) * d.field, d.field, k, chunk_stride);
          with_dense_range(p, eg, eg.H);
          with_rec_extract(p, t, out_b, g->nt, n);
        }, st, &lw);
        if (rc) return rc;
      }
      HIPCHK(launch_gather(fw.cur(), d.field, t.cells, Sb, geo->nrec, out_b, g->nt, g->nt - 1, st));
      continue;
    }
    float *u0 = pairs, *u1 = pairs + d.field * Sb;
    float *w0 = pairs + 2 * d.field * Sb, *w1 = pairs + 3 * d.field * Sb;
    HIPCHK(launch_zero(pairs, 4 * d.field * Sb, st));
    HIPCHK(launch_zero(sc, chunk_stride * Sb, st));
    float *ucur = u0, *uprev = u1, *wcur = w0, *wprev = w1;
    for (int c0 = 0; c0 < g->nt - 1; c0 += KC) {
      const int nk = std::min(KC, g->nt - 1 - c0);
      for (int m = 0; m < nk; ++m) {
        StepArgs a = batch_args(c, Sb, d.field);
        a.cur = ucur;
        a.prev = uprev;
        a.out = uprev;
        a.t2 = t2 + m * d.field;
        a.t2_sstride = chunk_stride;
        with_src(a, t, geo, g, s0, c0 + m);
        HIPCHK(launch_step(a, d.TX, kModeT2, st));
        std::swap(ucur, uprev);
      }
      HIPCHK(launch_ext_scatter(coef, eg, +1, t2, d.field, chunk_stride, sc, d.field, chunk_stride, Sb, nk, st));
      for (int m = 0; m < nk; ++m) {
        StepArgs a = batch_args(c, Sb, d.field);
        a.cur = wcur;
        a.prev = wprev;
        a.out = wprev;
        a.dsrc = sc + m * d.field;
        a.dsrc_sstride = chunk_stride;
        with_rec_extract(a, t, out_b, g->nt, c0 + m);
        HIPCHK(launch_step(a, d.TX, kModeDsrc, st));
        std::swap(wcur, wprev);
      }
    }
    HIPCHK(launch_gather(wcur, d.field, t.cells, Sb, geo->nrec, out_b, g->nt, g->nt - 1, st));
  }
  return FWIME_OK;
}

// ---------------------------------------------------------------------------
// Extended Born with time lags (lags tau_k = k L dt, k = -K .. K) and its
// adjoint.  The scattering source at step n takes the background's T2 term at
// steps n - 2kL, after n as well as before it, so the background's T2 history
// of a shot batch is kept whole (nt - 1 fields per shot); the batch size
// follows from that.  The background is carried in extended precision, as in
// the offset operators.
// ---------------------------------------------------------------------------
static int check_tau(fwime_ctx_t *ctx, const fwime_grid_t *g, int ntau, int lag) {
  if (ntau < 1 || ntau % 2 == 0 || ntau > 1023) return set_err(ctx, FWIME_EINVAL, "ntau must be odd, 1 <= ntau <= 1023");
  if (lag < 1 || (long)lag * (ntau - 1) > 4L * g->nt)
    return set_err(ctx, FWIME_EINVAL, "lag must be >= 1 with lag (ntau - 1) <= 4 nt");
  return FWIME_OK;
}

// Background T2 history of a shot batch: march all nt - 1 steps, T2 of step n
// into slot n of hist (per-shot stride hstride).
// Background of a shot batch in extended precision, keeping the T2 term of
// every step (slot n of shot s at hist + s hstride + n field); with rec_out
// (batch-local [Sb][nrec][nt]) it also records the receivers.
static int tau_background(fwime_ctx_t *ctx, const Common &c, const fwime_grid_t *g, const fwime_geom_t *geo,
                          int s0, int Sb, const DevTables &t, float *pairs, unsigned short *lows, float *hist,
                          long hstride, hipStream_t st, float *rec_out = nullptr) {
  const Dims &d = c.d;
  HIPCHK(zero_start(pairs, d, Sb, st));
  HIPCHK(zero_start(lows, d, Sb, st));
  Ring4 fu(pairs, d.field * Sb);
  Ring4L lu(lows, d.field * Sb);
  const float *wav_b = geo->wavelet + (long)s0 * g->nt;
  int rc = march2(ctx, c, fu, Sb, 0, g->nt - 1, kModeT2, [&](Steps &p, int n, int k) {
    with_t2(p, hist + (long)n * d.field, d.field, k, hstride);
    with_src2(p, t, wav_b, g, n);
    if (rec_out) with_rec_extract(p, t, rec_out, g->nt, n);
  }, st, &lu);
  if (rc || !rec_out) return rc;
  HIPCHK(launch_gather(fu.cur(), d.field, t.cells, Sb, geo->nrec, rec_out, g->nt, g->nt - 1, st));
  return FWIME_OK;
}

int fwime_born_ext_tau_fwd(fwime_ctx_t *ctx, const fwime_grid_t *g, const float *vel, const fwime_geom_t *geo,
                           int32_t ntau, int32_t lag, const float *ptau, float *data, void *stream) {
  if (!ctx) return FWIME_EINVAL;
  ctx->err.clear();
  hipStream_t st = (hipStream_t)stream;
  int rc;
  if ((rc = check_grid(ctx, g)) || (rc = check_geom(ctx, g, geo)) || (rc = check_tau(ctx, g, ntau, lag))) return rc;
  if (!data || !ptau) return set_err(ctx, FWIME_EINVAL, "data or ptau is null");
  HIPCHK(hipSetDevice(ctx->device));
  if ((rc = check_inputs(ctx, g, vel, geo, {{ptau, (long)ntau * g->nx * g->nz}}, st))) return rc;

  Common c;
  c.d = make_dims(g, ctx->tile_x);
  const Dims &d = c.d;
  ExtGeom eg{d.nz, d.nx, d.nb, d.NZ, d.NX, d.LZ, ntau, (ntau - 1) / 2};
  const int ns = g->nt - 1;                        // time steps (equations)
  // per shot: T2 history and source history (ns fields each), the two
  // wavefields' rings (8 fields) and the background's BF16 low parts (2)
  const long per_shot = (2L * ns + 10) * d.field * 4 + (long)geo->nrec * 64;
  const size_t fixed = (size_t)d.field * 8 + (size_t)ntau * d.nx * d.nz * 4;
  const int S = choose_batch(ctx, per_shot, fixed, geo->nshots);
  auto batches = split_batches(geo->nshots, S);
  choose_steps(ctx, c.d, S, true);
  TableSet ts = build_table_set(d, geo, batches, true);

  float *coef = nullptr, *pairs = nullptr, *hist = nullptr, *sc = nullptr;
  unsigned short *lows = nullptr;
  Carve cv;
  cv.add(&c.V, d.field);
  cv.add(&c.gz, d.LZ);
  cv.add(&c.gx, d.NX + kGxPad);
  cv.add(&c.tables, table_set_ints(ts) + 64 * batches.size() * 8);
  cv.add(&coef, (long)ntau * d.nx * d.nz);
  cv.add(&pairs, 8 * d.field * S);
  cv.add(&lows, 4 * d.field * S);
  cv.add(&hist, (long)ns * d.field * S);
  cv.add(&sc, (long)ns * d.field * S);
  if ((rc = arena_get(ctx, cv)))
    return or_frugally(ctx, rc, d.T == 4, [&] {
      return fwime_born_ext_tau_fwd(ctx, g, vel, geo, ntau, lag, ptau, data, stream);
    });
  if ((rc = upload_tables(ctx, ts, c.tables, st))) return rc;
  if ((rc = setup_common(ctx, c, g, vel, st))) return rc;
  HIPCHK(launch_ext_coef(ptau, vel, eg, (float)g->dt, coef, st));

  const long hstride = (long)ns * d.field;         // per shot in hist / sc
  for (size_t bi = 0; bi < batches.size(); ++bi) {
    const int s0 = batches[bi].first, Sb = batches[bi].second;
    const DevTables &t = ts.dev[bi];
    float *out_b = data + (long)s0 * geo->nrec * g->nt;
    if ((rc = tau_background(ctx, c, g, geo, s0, Sb, t, pairs, lows, hist, hstride, st))) return rc;
    HIPCHK(launch_tau_scatter(coef, eg, lag, hist, sc, d.field, hstride, ns, Sb, st));
    float *wp = pairs + 4 * d.field * Sb;
    HIPCHK(zero_start(wp, d, Sb, st));
    Ring4 fw(wp, d.field * Sb);
    rc = march2(ctx, c, fw, Sb, 0, ns, kModeDsrc, [&](Steps &p, int n, int k) {
      with_dsrc2(p, sc + (long)n * d.field, d.field, k, hstride);
      with_dense_range(p, eg, 0);
      with_rec_extract(p, t, out_b, g->nt, n);
    }, st);
    if (rc) return rc;
    HIPCHK(launch_gather(fw.cur(), d.field, t.cells, Sb, geo->nrec, out_b, g->nt, g->nt - 1, st));
  }
  return FWIME_OK;
}

int fwime_born_ext_tau_adj(fwime_ctx_t *ctx, const fwime_grid_t *g, const float *vel, const fwime_geom_t *geo,
                           int32_t ntau, int32_t lag, const float *data, float *ptau_out, void *stream) {
  if (!ctx) return FWIME_EINVAL;
  ctx->err.clear();
  hipStream_t st = (hipStream_t)stream;
  int rc;
  if ((rc = check_grid(ctx, g)) || (rc = check_geom(ctx, g, geo)) || (rc = check_tau(ctx, g, ntau, lag))) return rc;
  if (!data || !ptau_out) return set_err(ctx, FWIME_EINVAL, "data or ptau_out is null");
  HIPCHK(hipSetDevice(ctx->device));
  if ((rc = check_inputs(ctx, g, vel, geo, {{data, (long)geo->nshots * geo->nrec * g->nt}}, st))) return rc;

  Common c;
  c.d = make_dims(g, ctx->tile_x);
  const Dims &d = c.d;
  ExtGeom eg{d.nz, d.nx, d.nb, d.NZ, d.NX, d.LZ, ntau, (ntau - 1) / 2};
  const int ns = g->nt - 1;
  const int R = g->nt + 1;                         // adjoint field of every time 0 .. nt
  // per shot: T2 history (ns fields), adjoint history (R), background ring (4), low parts (2)
  const long per_shot = ((long)ns + R + 6) * d.field * 4 + (long)geo->nrec * 64;
  const size_t fixed = (size_t)d.field * 8;
  const int S = choose_batch(ctx, per_shot, fixed, geo->nshots);
  auto batches = split_batches(geo->nshots, S);
  choose_steps(ctx, c.d, S, true);
  TableSet ts = build_table_set(d, geo, batches, true);

  float *pairs = nullptr, *hist = nullptr, *lam = nullptr;
  unsigned short *lows = nullptr;
  Carve cv;
  cv.add(&c.V, d.field);
  cv.add(&c.gz, d.LZ);
  cv.add(&c.gx, d.NX + kGxPad);
  cv.add(&c.tables, table_set_ints(ts) + 64 * batches.size() * 8);
  cv.add(&pairs, 4 * d.field * S);
  cv.add(&lows, 4 * d.field * S);
  cv.add(&hist, (long)ns * d.field * S);
  cv.add(&lam, (long)R * d.field * S);
  if ((rc = arena_get(ctx, cv)))
    return or_frugally(ctx, rc, d.T == 4, [&] {
      return fwime_born_ext_tau_adj(ctx, g, vel, geo, ntau, lag, data, ptau_out, stream);
    });
  if ((rc = upload_tables(ctx, ts, c.tables, st))) return rc;
  if ((rc = setup_common(ctx, c, g, vel, st))) return rc;
  HIPCHK(launch_zero(ptau_out, (long)ntau * d.nx * d.nz, st));

  const long hstride = (long)ns * d.field, lstride = (long)R * d.field;
  for (size_t bi = 0; bi < batches.size(); ++bi) {
    const int s0 = batches[bi].first, Sb = batches[bi].second;
    const DevTables &t = ts.dev[bi];
    const float *data_b = data + (long)s0 * geo->nrec * g->nt;
    if ((rc = tau_background(ctx, c, g, geo, s0, Sb, t, pairs, lows, hist, hstride, st))) return rc;
    HIPCHK(zero_end(lam, lstride, R, d, Sb, st));
    if ((rc = march2_back_lambda(ctx, c, lam, lstride, R, Sb, 0, g->nt - 1, t, data_b, g->nt, st))) return rc;
    HIPCHK(launch_tau_image(hist, d.field, hstride, lam, d.field, lstride, ns, Sb, eg, lag, vel, (float)g->dt,
                            ptau_out, st));
  }
  return FWIME_OK;
}

// ---------------------------------------------------------------------------
// Background of the extended-precision adjoint kept across calls with the
// same model and shots (the variable-projection step): the T2 terms of every
// shot and step where they fit (hist, per shot nt - 1 fields), else the
// checkpoints (per shot 2 nseg fields, FP32 and BF16 low parts), in shot
// order.  `valid` once a call has filled them; later calls skip their forward
// pass.
struct AdjCache {
  float *hist = nullptr;
  float *ckpt = nullptr;
  unsigned short *ckpt_lo = nullptr;
  bool valid = false;
};

static int born_ext_adj_run(fwime_ctx_t *ctx, const fwime_grid_t *g, const float *vel, const fwime_geom_t *geo,
                            int32_t nh, const float *data, float *ptilde_out, void *stream, AdjCache *cache);

int fwime_born_ext_adj(fwime_ctx_t *ctx, const fwime_grid_t *g, const float *vel, const fwime_geom_t *geo,
                       int32_t nh, const float *data, float *ptilde_out, void *stream) {
  return born_ext_adj_run(ctx, g, vel, geo, nh, data, ptilde_out, stream, nullptr);
}

static int born_ext_adj_run(fwime_ctx_t *ctx, const fwime_grid_t *g, const float *vel, const fwime_geom_t *geo,
                            int32_t nh, const float *data, float *ptilde_out, void *stream, AdjCache *cache) {
  if (!ctx) return FWIME_EINVAL;
  ctx->err.clear();
  hipStream_t st = (hipStream_t)stream;
  int rc;
  if ((rc = check_grid(ctx, g)) || (rc = check_geom(ctx, g, geo)) || (rc = check_nh(ctx, g, nh))) return rc;
  if (!data || !ptilde_out) return set_err(ctx, FWIME_EINVAL, "data or ptilde_out is null");
  HIPCHK(hipSetDevice(ctx->device));
  if ((rc = check_inputs(ctx, g, vel, geo, {{data, (long)geo->nshots * geo->nrec * g->nt}}, st))) return rc;

  Common c;
  c.d = make_dims(g, ctx->tile_x);
  const Dims &d = c.d;
  ExtGeom eg{d.nz, d.nx, d.nb, d.NZ, d.NX, d.LZ, nh, (nh - 1) / 2};
  const bool two = ctx->two_step;
  const int nf = two ? 4 : 2;
  if (!two) cache = nullptr;                    // the one-step path recomputes inside its checkpoints
  float *hist = cache ? cache->hist : nullptr;  // whole T2 history: the cache's, or the arena's where it fits
  const bool own_hist = !cache;
  const long img = (long)nh * d.nx * d.nz;
  auto fixed = [&](long parts) { return (size_t)d.field * 8 + (size_t)img * (8 + 4 * parts); };   // FP64 image + partials
  auto hist_per_shot = [&](int S) {
    const long r = hist_seg_len(g->nt, S) + 2;
    return (nf + 2 + r + (r + 1) / 2 + (own_hist ? g->nt - 1L : 0L)) * d.field * 4 + (long)geo->nrec * 64;
  };
  const int Sh = !two || (cache && !hist) ? 0 : hist_batch(ctx, geo->nshots, (long)d.ntz2 * d.ntx, [&](int S) {
    return fixed(hist_parts(g->nt, hist_seg_len(g->nt, S), img)) + (size_t)hist_per_shot(S) * S;
  }, &ctx->arena);
  const bool keep = Sh > 0 || hist;
  const int seg = seg_len(g->nt);               // checkpointed segment
  const int K = Sh ? hist_seg_len(g->nt, Sh) : seg;
  const long nparts = hist_parts(g->nt, K, img);
  const int nseg = (g->nt - 1 + K - 1) / K;
  const int R = K + 2;
  // two-step path: BF16 low parts of the four work fields and the checkpoints
  // (cached checkpoints live outside the arena)
  const long ck_fields = cache || keep ? 0L : 2L * nseg + (two ? nseg : 0L);
  // (two-step path: the adjoint ring's BF16 low parts add R / 2 fields)
  const long per_shot = (nf + (keep ? 0 : K) + R + (two ? 2L + (R + 1) / 2 : 0L) + ck_fields) * d.field * 4 +
                        (long)geo->nrec * 64;
  const int S = Sh ? Sh : choose_batch(ctx, per_shot, fixed(nparts), geo->nshots);
  auto batches = split_batches(geo->nshots, S);
  choose_steps(ctx, c.d, S, true);
  TableSet ts = build_table_set(d, geo, batches, two);

  float *pairs = nullptr, *ckpt = nullptr, *t2 = nullptr, *ring = nullptr;
  double *acc = nullptr;
  Carve cv;
  cv.add(&c.V, d.field);
  cv.add(&c.gz, d.LZ);
  cv.add(&c.gx, d.NX + kGxPad);
  cv.add(&c.tables, table_set_ints(ts) + 64 * batches.size() * 8);
  unsigned short *lows = nullptr, *ckpt_lo = nullptr, *ring_lo = nullptr;
  float *parts = nullptr;
  cv.add(&acc, img);
  cv.add(&parts, nparts * img);
  cv.add(&pairs, nf * d.field * S);
  if (!cache && !keep) cv.add(&ckpt, 2L * nseg * d.field * S);
  if (two) {
    cv.add(&lows, 4 * d.field * S);
    cv.add(&ring_lo, (long)R * d.field * S);
    if (!cache && !keep) cv.add(&ckpt_lo, 2L * nseg * d.field * S);
  }
  const long hist_stride = (g->nt - 1L) * d.field;
  if (keep && own_hist) cv.add(&hist, hist_stride * S);
  if (!keep) cv.add(&t2, (long)K * d.field * S);
  cv.add(&ring, (long)R * d.field * S);
  if ((rc = arena_get(ctx, cv)))
    return or_frugally(ctx, rc, d.T == 4 || Sh > 0, [&] {
      return born_ext_adj_run(ctx, g, vel, geo, nh, data, ptilde_out, stream, cache);
    });
  if ((rc = upload_tables(ctx, ts, c.tables, st))) return rc;
  if ((rc = setup_common(ctx, c, g, vel, st))) return rc;
  HIPCHK(launch_zero_d(acc, img, st));

  const long ck_stride = 2L * nseg * d.field;   // per shot
  const long t2_stride = (long)K * d.field;
  const long ring_stride = (long)R * d.field;
  for (size_t bi = 0; bi < batches.size(); ++bi) {
    const int s0 = batches[bi].first, Sb = batches[bi].second;
    const DevTables &t = ts.dev[bi];
    const float *data_b = data + (long)s0 * geo->nrec * g->nt;
    if (two) {
      const float *wav_b = geo->wavelet + (long)s0 * g->nt;
      auto src = [&](Steps &p, int n, int) { with_src2(p, t, wav_b, g, n); };
      if (cache && !keep) {                     // this batch's shots in the cached checkpoints
        ckpt = cache->ckpt + (long)s0 * ck_stride;
        ckpt_lo = cache->ckpt_lo + (long)s0 * ck_stride;
      }
      // forward pass (extended precision) storing (u^{n0-1}, u^{n0}) at every
      // segment start, unless the cached checkpoints already hold them
      HIPCHK(zero_start(pairs, d, Sb, st));
      HIPCHK(zero_start(lows, d, Sb, st));
      Ring4 fu(pairs, d.field * Sb);
      Ring4L lu(lows, d.field * Sb);
      // with a whole history it stores T2 u_n of every step instead
      float *hist_b = keep ? hist + (own_hist ? 0L : s0 * hist_stride) : nullptr;
      if (keep && !(cache && cache->valid)) {
        rc = march2(ctx, c, fu, Sb, 0, g->nt - 1, kModeT2, [&](Steps &p, int n, int k) {
          with_t2(p, hist_b + (long)n * d.field, d.field, k, hist_stride);
          with_src2(p, t, wav_b, g, n);
        }, st, &lu);
        if (rc) return rc;
      }
      for (int j = 0; j < nseg && !keep && !(cache && cache->valid); ++j) {
        const int n0 = j * K, n1 = std::min(n0 + K, g->nt - 1);
        HIPCHK(launch_copy_fields(ckpt + (2L * j) * d.field, ck_stride, fu.prev(), d.field, Sb, d.field, st));
        HIPCHK(launch_copy_fields(ckpt + (2L * j + 1) * d.field, ck_stride, fu.cur(), d.field, Sb, d.field, st));
        HIPCHK(copy_lo(ckpt_lo + (2L * j) * d.field, ck_stride, lu.prev(), d.field, Sb, d.field, st));
        HIPCHK(copy_lo(ckpt_lo + (2L * j + 1) * d.field, ck_stride, lu.cur(), d.field, Sb, d.field, st));
        if (j == nseg - 1) break;   // the last segment is recomputed anyway
        if ((rc = march2(ctx, c, fu, Sb, n0, n1, kModePlain, src, st, &lu))) return rc;
      }
      // backward pass: recompute the segment from its checkpoint (keeping
      // T2 u_n), march lambda through the segment (in extended precision as
      // well), image
      HIPCHK(zero_end(ring, ring_stride, R, d, Sb, st));
      HIPCHK(zero_end(ring_lo, ring_stride, R, d, Sb, st));
      for (int j = nseg - 1; j >= 0; --j) {
        const int n0 = j * K, n1 = std::min(n0 + K, g->nt - 1), nk = n1 - n0;
        if (keep) {
          if ((rc = march2_back_lambda(ctx, c, ring, ring_stride, R, Sb, n0, n1, t, data_b, g->nt, st, ring_lo)))
            return rc;
          HIPCHK(launch_ext_image(hist_b + (long)n0 * d.field, d.field, hist_stride, ring, d.field, ring_stride, R, n0,
                                  Sb, nk, seg, eg, acc, parts, (int)nparts, st));
          continue;
        }
        Ring4 wu(pairs, d.field * Sb);
        Ring4L wl(lows, d.field * Sb);
        HIPCHK(launch_copy_fields(wu.prev(), d.field, ckpt + (2L * j) * d.field, ck_stride, Sb, d.field, st));
        HIPCHK(launch_copy_fields(wu.cur(), d.field, ckpt + (2L * j + 1) * d.field, ck_stride, Sb, d.field, st));
        HIPCHK(copy_lo(wl.prev(), d.field, ckpt_lo + (2L * j) * d.field, ck_stride, Sb, d.field, st));
        HIPCHK(copy_lo(wl.cur(), d.field, ckpt_lo + (2L * j + 1) * d.field, ck_stride, Sb, d.field, st));
        rc = march2(ctx, c, wu, Sb, n0, n1, kModeT2, [&](Steps &p, int n, int k) {
          with_t2(p, t2 + (long)(n - n0) * d.field, d.field, k, t2_stride);
          with_src2(p, t, wav_b, g, n);
        }, st, &wl);
        if (rc) return rc;
        if ((rc = march2_back_lambda(ctx, c, ring, ring_stride, R, Sb, n0, n1, t, data_b, g->nt, st, ring_lo)))
          return rc;
        HIPCHK(launch_ext_image(t2, d.field, t2_stride, ring, d.field, ring_stride, R, n0, Sb, nk, seg, eg, acc, parts,
                               (int)nparts, st));
      }
      continue;
    }
    // forward pass storing (u^{n0-1}, u^{n0}) at every segment start
    float *p0 = pairs, *p1 = pairs + d.field * Sb;
    HIPCHK(launch_zero(pairs, 2 * d.field * Sb, st));
    float *cur = p0, *prev = p1;
    for (int j = 0; j < nseg; ++j) {
      const int n0 = j * K, n1 = std::min(n0 + K, g->nt - 1);
      HIPCHK(launch_copy_fields(ckpt + (2L * j) * d.field, ck_stride, prev, d.field, Sb, d.field, st));
      HIPCHK(launch_copy_fields(ckpt + (2L * j + 1) * d.field, ck_stride, cur, d.field, Sb, d.field, st));
      if (j == nseg - 1) break;   // the last segment is recomputed anyway
      for (int n = n0; n < n1; ++n) {
        StepArgs a = batch_args(c, Sb, d.field);
        a.cur = cur;
        a.prev = prev;
        a.out = prev;
        with_src(a, t, geo, g, s0, n);
        HIPCHK(launch_step(a, d.TX, kModePlain, st));
        std::swap(cur, prev);
      }
    }
    // backward pass
    HIPCHK(launch_zero(ring, ring_stride * Sb, st));
    for (int j = nseg - 1; j >= 0; --j) {
      const int n0 = j * K, n1 = std::min(n0 + K, g->nt - 1), nk = n1 - n0;
      float *ccur = ckpt + (2L * j + 1) * d.field, *cprev = ckpt + (2L * j) * d.field;
      for (int n = n0; n < n1; ++n) {
        StepArgs a = batch_args(c, Sb, ck_stride);
        a.cur = ccur;
        a.prev = cprev;
        a.out = cprev;
        a.t2 = t2 + (long)(n - n0) * d.field;
        a.t2_sstride = t2_stride;
        with_src(a, t, geo, g, s0, n);
        HIPCHK(launch_step(a, d.TX, kModeT2, st));
        std::swap(ccur, cprev);
      }
      for (int k = n1; k >= n0 + 1; --k) {
        StepArgs a = batch_args(c, Sb, ring_stride);
        a.cur = ring + (long)(k % R) * d.field;
        a.prev = ring + (long)((k + 1) % R) * d.field;
        a.out = ring + (long)((k - 1) % R) * d.field;
        with_rec_inject(a, t, data_b, g->nt, k);
        HIPCHK(launch_step(a, d.TX, kModePlain, st));
      }
      HIPCHK(launch_ext_image(t2, d.field, t2_stride, ring, d.field, ring_stride, R, n0, Sb, nk, seg, eg, acc, parts,
                               (int)nparts, st));
    }
  }
  HIPCHK(launch_ext_finalize(acc, vel, eg, (float)g->dt, nullptr, nullptr, ptilde_out, st));
  if (cache) cache->valid = true;
  return FWIME_OK;
}

}  // extern "C"

namespace {

// ---------------------------------------------------------------------------
// FWIME gradient building blocks, shared by fwime_gradient and the tape API.
//
// Forward (one batch): u and du~ together, segment by segment; at each segment
// start the pairs (u^{n0-1}, u^{n0}) and (du~^{n0-1}, du~^{n0}) are stored, the
// segment's T2u_n feeds the extended scatter whose output drives du~, and the
// receivers of u and du~ are recorded separately.
// Backward (one batch, adjoint source r at the receivers): per segment, from
// last to first, recompute u (keeping T2u_n) and du~ (keeping T2du~_n), march
// lambda (source r), spread lambda into the e ring, march rho (source the
// transposed second time difference of e), then accumulate the extended image
// sum T2u(y-h) lambda(y+h) and the per-cell sum (T2u + T2du~) lambda + T2u rho.
// With whole histories (hist) the forward pass keeps T2u and T2du~ of every
// step, nothing is checkpointed and the backward pass recomputes nothing.
// The scattering source of du~ passes through the e ring: it is done with
// before the spread of the same steps is written.
// ---------------------------------------------------------------------------
struct GradPlan {
  int K, nseg, R;
  int seg;                  // checkpointed segment: K, or several to a segment with histories
  bool hist = false;
  long ck_stride, seg_stride, ring_stride;
  void set_segment(const Dims &d, int nt, int steps) {
    K = steps;
    nseg = (nt - 1 + K - 1) / K;
    R = K + 2;
    ring_stride = (long)R * d.field;
  }
  // first slot of segment start n0 in the T2 buffers
  long t2_off(const Dims &d, int n0) const { return hist ? (long)n0 * d.field : 0L; }
};

// hist_shots: shots per batch with whole histories, 0 to checkpoint
GradPlan grad_plan(const Dims &d, int nt, int hist_shots = 0) {
  GradPlan p;
  p.hist = hist_shots > 0;
  p.seg = seg_len(nt);
  p.set_segment(d, nt, p.hist ? hist_seg_len(nt, hist_shots) : p.seg);
  p.ck_stride = p.hist ? 0L : 2L * p.nseg * d.field;
  p.seg_stride = (p.hist ? (long)(nt - 1) : (long)p.K) * d.field;
  return p;
}

struct GradWork {       // per-batch working fields (+ partial images of the imaging kernel)
  float *pairs, *t2u, *t2d, *lam, *er, *rho;
  float *parts = nullptr;
  long nparts = 0;
};

int grad_forward_batch(fwime_ctx_t *ctx, const Common &c, const ExtGeom &eg, const GradPlan &pl,
                       const fwime_grid_t *g, int Sb, const DevTables &t, const float *wav_b, const float *coef,
                       float *uck, float *dck, const GradWork &wk, float *drec, float *ddrec, int nrec,
                       hipStream_t st) {
  const Dims &d = c.d;
  int rc;
  if (ctx->two_step) {
    HIPCHK(zero_start(wk.pairs, d, Sb, st));
    HIPCHK(zero_start(wk.pairs + 4 * d.field * Sb, d, Sb, st));
    Ring4 fu(wk.pairs, d.field * Sb), fw(wk.pairs + 4 * d.field * Sb, d.field * Sb);
    for (int j = 0; j < pl.nseg; ++j) {
      const int n0 = j * pl.K, n1 = std::min(n0 + pl.K, g->nt - 1), nk = n1 - n0;
      if (!pl.hist) {
        HIPCHK(launch_copy_fields(uck + (2L * j) * d.field, pl.ck_stride, fu.prev(), d.field, Sb, d.field, st));
        HIPCHK(launch_copy_fields(uck + (2L * j + 1) * d.field, pl.ck_stride, fu.cur(), d.field, Sb, d.field, st));
        HIPCHK(launch_copy_fields(dck + (2L * j) * d.field, pl.ck_stride, fw.prev(), d.field, Sb, d.field, st));
        HIPCHK(launch_copy_fields(dck + (2L * j + 1) * d.field, pl.ck_stride, fw.cur(), d.field, Sb, d.field, st));
      }
      float *t2u = wk.t2u + pl.t2_off(d, n0), *t2d = wk.t2d + pl.t2_off(d, n0);
      rc = march2(ctx, c, fu, Sb, n0, n1, kModeT2, [&](Steps &p, int n, int k) {
        with_t2(p, t2u + (long)(n - n0) * d.field, d.field, k, pl.seg_stride);
        with_src2(p, t, wav_b, g, n);
        with_rec_extract(p, t, drec, g->nt, n);
      }, st);
      if (rc) return rc;
      HIPCHK(launch_ext_scatter(coef, eg, +1, t2u, d.field, pl.seg_stride, wk.er, d.field, pl.ring_stride, Sb, nk,
                                st));
      rc = march2(ctx, c, fw, Sb, n0, n1, pl.hist ? kModeT2 | kModeDsrc : kModeDsrc, [&](Steps &p, int n, int k) {
        with_dsrc2(p, wk.er + (long)(n - n0) * d.field, d.field, k, pl.ring_stride);
        with_dense_range(p, eg, eg.H);
        if (pl.hist) with_t2(p, t2d + (long)(n - n0) * d.field, d.field, k, pl.seg_stride);
        with_rec_extract(p, t, ddrec, g->nt, n);
      }, st);
      if (rc) return rc;
    }
    HIPCHK(launch_gather(fu.cur(), d.field, t.cells, Sb, nrec, drec, g->nt, g->nt - 1, st));
    HIPCHK(launch_gather(fw.cur(), d.field, t.cells, Sb, nrec, ddrec, g->nt, g->nt - 1, st));
    return FWIME_OK;
  }
  float *u0 = wk.pairs, *u1 = wk.pairs + d.field * Sb, *w0 = wk.pairs + 2 * d.field * Sb,
        *w1 = wk.pairs + 3 * d.field * Sb;
  HIPCHK(launch_zero(wk.pairs, 4 * d.field * Sb, st));
  HIPCHK(launch_zero(wk.er, pl.ring_stride * Sb, st));   // the one-step kernel reads its source on the whole grid
  float *ucur = u0, *uprev = u1, *wcur = w0, *wprev = w1;
  for (int j = 0; j < pl.nseg; ++j) {
    const int n0 = j * pl.K, n1 = std::min(n0 + pl.K, g->nt - 1), nk = n1 - n0;
    if (!pl.hist) {
      HIPCHK(launch_copy_fields(uck + (2L * j) * d.field, pl.ck_stride, uprev, d.field, Sb, d.field, st));
      HIPCHK(launch_copy_fields(uck + (2L * j + 1) * d.field, pl.ck_stride, ucur, d.field, Sb, d.field, st));
      HIPCHK(launch_copy_fields(dck + (2L * j) * d.field, pl.ck_stride, wprev, d.field, Sb, d.field, st));
      HIPCHK(launch_copy_fields(dck + (2L * j + 1) * d.field, pl.ck_stride, wcur, d.field, Sb, d.field, st));
    }
    float *t2u = wk.t2u + pl.t2_off(d, n0), *t2d = wk.t2d + pl.t2_off(d, n0);
    for (int n = n0; n < n1; ++n) {
      StepArgs a = batch_args(c, Sb, d.field);
      a.cur = ucur;
      a.prev = uprev;
      a.out = uprev;
      a.t2 = t2u + (long)(n - n0) * d.field;
      a.t2_sstride = pl.seg_stride;
      with_src_w(a, t, wav_b, g, n);
      with_rec_extract(a, t, drec, g->nt, n);
      HIPCHK(launch_step(a, d.TX, kModeT2, st));
      std::swap(ucur, uprev);
    }
    HIPCHK(launch_ext_scatter(coef, eg, +1, t2u, d.field, pl.seg_stride, wk.er, d.field, pl.ring_stride, Sb, nk,
                              st));
    for (int n = n0; n < n1; ++n) {
      StepArgs a = batch_args(c, Sb, d.field);
      a.cur = wcur;
      a.prev = wprev;
      a.out = wprev;
      a.dsrc = wk.er + (long)(n - n0) * d.field;
      a.dsrc_sstride = pl.ring_stride;
      if (pl.hist) {
        a.t2 = t2d + (long)(n - n0) * d.field;
        a.t2_sstride = pl.seg_stride;
      }
      with_rec_extract(a, t, ddrec, g->nt, n);
      HIPCHK(launch_step(a, d.TX, pl.hist ? kModeT2 | kModeDsrc : kModeDsrc, st));
      std::swap(wcur, wprev);
    }
  }
  HIPCHK(launch_gather(ucur, d.field, t.cells, Sb, nrec, drec, g->nt, g->nt - 1, st));
  HIPCHK(launch_gather(wcur, d.field, t.cells, Sb, nrec, ddrec, g->nt, g->nt - 1, st));
  return FWIME_OK;
}

int grad_backward_batch(fwime_ctx_t *ctx, const Common &c, const ExtGeom &eg, const GradPlan &pl,
                        const fwime_grid_t *g, int Sb, const DevTables &t, const float *wav_b, const float *coef,
                        float *uck, float *dck, const GradWork &wk, const float *r, double *acc, float *gacc,
                        hipStream_t st) {
  const Dims &d = c.d;
  const int K = pl.K, R = pl.R;
  const bool two = ctx->two_step;
  for (float *ring : {wk.lam, wk.er, wk.rho}) {
    // (the one-step kernels read e on the whole grid)
    if (two) HIPCHK(zero_end(ring, pl.ring_stride, R, d, Sb, st));
    else HIPCHK(launch_zero(ring, pl.ring_stride * Sb, st));
  }
  int rc;
  for (int j = pl.nseg - 1; j >= 0; --j) {
    const int n0 = j * K, n1 = std::min(n0 + K, g->nt - 1), nk = n1 - n0;
    const float *t2u = wk.t2u + pl.t2_off(d, n0), *t2d = wk.t2d + pl.t2_off(d, n0);
    auto er_slot = [&](int k) { return wk.er + (long)(k % R) * d.field; };
    if (two && !pl.hist) {
      // u and du~ from their checkpoints, two steps per launch, keeping
      // T2 u_n and T2 du~_n; the scattering source of du~ takes the slots of
      // the e ring that this segment's spread fills afterwards
      Ring4 wu(wk.pairs, d.field * Sb), ww(wk.pairs + 4 * d.field * Sb, d.field * Sb);
      HIPCHK(launch_copy_fields(wu.prev(), d.field, uck + (2L * j) * d.field, pl.ck_stride, Sb, d.field, st));
      HIPCHK(launch_copy_fields(wu.cur(), d.field, uck + (2L * j + 1) * d.field, pl.ck_stride, Sb, d.field, st));
      HIPCHK(launch_copy_fields(ww.prev(), d.field, dck + (2L * j) * d.field, pl.ck_stride, Sb, d.field, st));
      HIPCHK(launch_copy_fields(ww.cur(), d.field, dck + (2L * j + 1) * d.field, pl.ck_stride, Sb, d.field, st));
      rc = march2(ctx, c, wu, Sb, n0, n1, kModeT2, [&](Steps &p, int n, int k) {
        with_t2(p, wk.t2u + (long)(n - n0) * d.field, d.field, k, pl.seg_stride);
        with_src2(p, t, wav_b, g, n);
      }, st);
      if (rc) return rc;
      HIPCHK(launch_ext_scatter(coef, eg, +1, wk.t2u, d.field, pl.seg_stride, wk.er, d.field, pl.ring_stride, Sb, nk,
                                st, 0, 0, R, n0));
      rc = march2(ctx, c, ww, Sb, n0, n1, kModeT2 | kModeDsrc, [&](Steps &p, int n, int k) {
        for (int i = 0; i < k; ++i) p.ds[i] = er_slot(n + i);
        p.ds_sstride = pl.ring_stride;
        with_dense_range(p, eg, eg.H);
        with_t2(p, wk.t2d + (long)(n - n0) * d.field, d.field, k, pl.seg_stride);
      }, st);
      if (rc) return rc;
    } else if (!pl.hist) {
      float *uc = uck + (2L * j + 1) * d.field, *up = uck + (2L * j) * d.field;
      for (int n = n0; n < n1; ++n) {
        StepArgs a = batch_args(c, Sb, pl.ck_stride);
        a.cur = uc;
        a.prev = up;
        a.out = up;
        a.t2 = wk.t2u + (long)(n - n0) * d.field;
        a.t2_sstride = pl.seg_stride;
        with_src_w(a, t, wav_b, g, n);
        HIPCHK(launch_step(a, d.TX, kModeT2, st));
        std::swap(uc, up);
      }
      // t2d holds T2 du~ of the later segment outside the scatter's range: clear it
      HIPCHK(launch_zero(wk.t2d, pl.seg_stride * Sb, st));
      HIPCHK(launch_ext_scatter(coef, eg, +1, wk.t2u, d.field, pl.seg_stride, wk.t2d, d.field, pl.seg_stride, Sb, nk,
                                st));
      float *wc = dck + (2L * j + 1) * d.field, *wp = dck + (2L * j) * d.field;
      for (int n = n0; n < n1; ++n) {
        StepArgs a = batch_args(c, Sb, pl.ck_stride);
        a.cur = wc;
        a.prev = wp;
        a.out = wp;
        a.dsrc = wk.t2d + (long)(n - n0) * d.field;   // read the source, then
        a.dsrc_sstride = pl.seg_stride;
        a.t2 = wk.t2d + (long)(n - n0) * d.field;     // overwrite it with T2 du~_n
        a.t2_sstride = pl.seg_stride;
        HIPCHK(launch_step(a, d.TX, kModeT2 | kModeDsrc, st));
        std::swap(wc, wp);
      }
    }
    if (two) {
      if ((rc = march2_back_lambda(ctx, c, wk.lam, pl.ring_stride, R, Sb, n0, n1, t, r, g->nt, st))) return rc;
    } else {
      for (int k = n1; k >= n0 + 1; --k) {
        StepArgs a = batch_args(c, Sb, pl.ring_stride);
        a.cur = wk.lam + (long)(k % R) * d.field;
        a.prev = wk.lam + (long)((k + 1) % R) * d.field;
        a.out = wk.lam + (long)((k - 1) % R) * d.field;
        with_rec_inject(a, t, r, g->nt, k);
        HIPCHK(launch_step(a, d.TX, kModePlain, st));
      }
    }
    HIPCHK(launch_ext_scatter(coef, eg, -1, wk.lam, d.field, pl.ring_stride, wk.er, d.field, pl.ring_stride, Sb, nk,
                              st, R, n0, R, n0));
    if (two) {
      rc = march2_back_ring(ctx, c, wk.rho, pl.ring_stride, R, Sb, n0, n1, kModeNu, [&](Steps &p, int k, int kk) {
        with_nu(p, er_slot, k, kk, pl.ring_stride);
        with_dense_range(p, eg, eg.H);
      }, st);
      if (rc) return rc;
    } else {
      for (int k = n1; k >= n0 + 1; --k) {
        StepArgs a = batch_args(c, Sb, pl.ring_stride);
        a.cur = wk.rho + (long)(k % R) * d.field;
        a.prev = wk.rho + (long)((k + 1) % R) * d.field;
        a.out = wk.rho + (long)((k - 1) % R) * d.field;
        a.nu = NuSource{er_slot(k - 1), er_slot(k), er_slot(k + 1), pl.ring_stride};
        HIPCHK(launch_step(a, d.TX, kModeNu, st));
      }
    }
    HIPCHK(launch_ext_image(t2u, d.field, pl.seg_stride, wk.lam, d.field, pl.ring_stride, R, n0, Sb, nk, pl.seg, eg,
                            acc, wk.parts, (int)wk.nparts, st));
    HIPCHK(launch_grad_accum(t2u, t2d, d.field, pl.seg_stride, wk.lam, wk.rho, d.field, pl.ring_stride, R, n0,
                             Sb, nk, pl.seg, d.NZ, d.NX, d.LZ, gacc, st));
  }
  return FWIME_OK;
}

// the two-step path keeps four field buffers per wavefield (u and du~)
long grad_work_per_shot(const Dims &d, const GradPlan &pl, bool two) {
  return (((two ? 8L : 4L) + 3L * pl.R) * d.field + 2L * pl.seg_stride) * 4;
}

// t2: with the T2 buffers (not those of a tape that holds whole histories)
void carve_work(Carve &cv, GradWork &wk, const Dims &d, const GradPlan &pl, int S, bool two, bool t2 = true) {
  cv.add(&wk.pairs, (two ? 8 : 4) * d.field * S);
  if (t2) {
    cv.add(&wk.t2u, pl.seg_stride * S);
    cv.add(&wk.t2d, pl.seg_stride * S);
  }
  cv.add(&wk.lam, (long)pl.R * d.field * S);
  cv.add(&wk.er, (long)pl.R * d.field * S);
  cv.add(&wk.rho, (long)pl.R * d.field * S);
}

}  // namespace

// ---------------------------------------------------------------------------
// Tape: device-resident state between a forward and a backward call.
// ---------------------------------------------------------------------------
struct fwime_tape {
  fwime_ctx_t *ctx = nullptr;             // null once the context is destroyed
  int device = 0;
  fwime_grid_t g{};
  int nh = 0, nshots = 0, nrec = 0;
  Dims d{};
  GradPlan pl{};
  std::vector<std::pair<int, int>> batches;
  TableSet ts;
  void *mem = nullptr;
  size_t bytes = 0, capacity = 0;         // used of `mem`, and held by it
  float *V = nullptr, *gz = nullptr, *gx = nullptr, *vel = nullptr, *pt = nullptr, *coef = nullptr, *wav = nullptr;
  float *uck = nullptr, *dck = nullptr;   // [nshots] x ck_stride each (whole T2 histories: x seg_stride)
  int *tables = nullptr;
  bool used = false;
};

static void detach_tapes(fwime_ctx_t *ctx) {
  std::lock_guard<std::mutex> lock(ctx->tape_mu);
  for (fwime_tape_t *t : ctx->tapes) t->ctx = nullptr;
  ctx->tapes.clear();
}

extern "C" {

// ---------------------------------------------------------------------------
// ---------------------------------------------------------------------------
// Variable-projection step (eqs. vp.obj, pert.opt, vp.pseudo.inv): linear
// conjugate gradient on (B~* B~ + eps^2 D* D) p~ = B~* (d_obs - f(m)) from
// p~ = 0.  Each iteration applies B~ and B~* once (four propagations per
// shot); the objective is tracked without further propagations as
// Phi_k = 1/2 ||d_obs - f(m)||^2 - 1/2 (b + r_k) . p~_k, which holds for any
// p~ with r = b - H p~ (b = B~* (d_obs - f(m)), H the normal matrix).
// The solver for either extension: subsurface offsets (tau false, nh
// offsets) or time lags (tau true, nh lags of `lag` steps).
static int vp_solve_run(fwime_ctx_t *ctx, const fwime_grid_t *g, const float *vel, const fwime_geom_t *geo,
                        int32_t nh, bool tau, int32_t lag, const float *dobs, double eps, const double *dso,
                        int32_t niter, float *ptilde_out, double *phi_out, void *stream) {
  if (!ctx) return FWIME_EINVAL;
  ctx->err.clear();
  hipStream_t st = (hipStream_t)stream;
  int rc;
  if ((rc = check_grid(ctx, g)) || (rc = check_geom(ctx, g, geo)) ||
      (rc = tau ? check_tau(ctx, g, nh, lag) : check_nh(ctx, g, nh)))
    return rc;
  if (!dobs || !dso || !ptilde_out || !phi_out) return set_err(ctx, FWIME_EINVAL, "null pointer argument");
  if (niter < 0) return set_err(ctx, FWIME_EINVAL, "niter must be >= 0");
  if (!std::isfinite(eps)) return set_err(ctx, FWIME_EINVAL, "eps must be finite");
  for (int h = 0; h < nh; ++h)
    if (!std::isfinite(dso[h])) return set_err(ctx, FWIME_EINVAL, "dso must be finite");
  HIPCHK(hipSetDevice(ctx->device));
  const long ndata = (long)geo->nshots * geo->nrec * g->nt;
  const long plane = (long)g->nx * g->nz;
  const long img = (long)nh * plane;
  if ((rc = check_inputs(ctx, g, vel, geo, {{dobs, ndata}}, st))) return rc;

  // the background does not change during the step: its T2 terms of every
  // shot and step are kept where they fit (hist), so that B~ and every B~*
  // after the first propagate only the scattered and the adjoint field; else
  // the extended-precision adjoint's checkpoints (2 nseg fields and their low
  // parts per shot), so that every B~* after the first skips its forward pass
  // (FWIME_VP_NOCACHE=1 turns both off)
  const Dims dd = make_dims(g, ctx->tile_x);
  const int K = seg_len(g->nt);
  const long nseg = (g->nt - 1 + K - 1) / K;
  const long ck_elems = 2L * nseg * dd.field * geo->nshots;
  bool use_cache = ctx->two_step && !tau;          // the time-lag adjoint keeps no checkpoints
  if (const char *e = std::getenv("FWIME_VP_NOCACHE")) use_cache = use_cache && std::atoi(e) == 0;
  if (use_cache) {
    size_t avail = 0, total = 0;
    if (hipMemGetInfo(&avail, &total) != hipSuccess) avail = 0;
    // the solver's own buffer (possibly already holding a cache) counts as free here
    const size_t need = (size_t)ck_elems * 6;
    use_cache = need < (size_t)((avail + ctx->vp_bytes + spare_bytes(ctx)) * 0.5) && (!ctx->budget || need < ctx->budget / 2);
  }
  const long hist_elems = (g->nt - 1L) * dd.field * geo->nshots;
  // beside it, at the same time: the rings and chunks of B~ and B~*
  auto beside = [&](int S) {
    const int K = hist_seg_len(g->nt, S);
    return ((16 + 2L * (K + 2)) * dd.field * 4 + geo->nrec * 64L) * S + img * (8 + 4 * hist_parts(g->nt, K, img));
  };
  const bool use_hist = use_cache && hist_batch(ctx, geo->nshots, 0, [&](int S) {
    return (size_t)(beside(S) + (g->nt - 1L) * dd.field * 4 * S + img * 16 + ndata * 8);
  }, &ctx->vp, (size_t)beside(geo->nshots)) > 0;
  // solver vectors, kept in the context between calls
  float *r = nullptr, *sdir = nullptr, *q = nullptr, *b = nullptr, *dres = nullptr, *dtmp = nullptr,
        *e2d2 = nullptr;
  double *part = nullptr, *res = nullptr;
  AdjCache cache;
  auto layout = [&](bool whole) {
    Carve cv;
    cache = AdjCache();
    if (whole) {
      cv.add(&cache.hist, hist_elems);
    } else if (use_cache) {
      cv.add(&cache.ckpt, ck_elems);
      cv.add(&cache.ckpt_lo, ck_elems);
    }
    cv.add(&r, img);
    cv.add(&sdir, img);
    cv.add(&q, img);
    cv.add(&b, img);
    cv.add(&dres, ndata);
    cv.add(&dtmp, ndata);
    cv.add(&e2d2, nh);
    cv.add(&part, dot_partials());
    cv.add(&res, 1);
    return cv;
  };
  Carve cv = layout(use_hist);
  if (cv.total > ctx->vp_bytes) {
    HIPCHK(hipStreamSynchronize(st));
    release_vp(ctx);
    hipError_t e = device_alloc(ctx, &ctx->vp, cv.total);
    if (e != hipSuccess && use_hist) {             // checkpoints, then
      (void)hipGetLastError();
      cv = layout(false);
      e = device_alloc(ctx, &ctx->vp, cv.total);
    }
    if (e != hipSuccess) {
      ctx->vp = nullptr;
      (void)hipGetLastError();
      return set_err(ctx, FWIME_ENOMEM, "cannot allocate the solver vectors");
    }
    ctx->vp_bytes = cv.total;
  }
  cv.assign(ctx->vp);
  if (cache.hist) {
    ctx->vp_hist = cv.total;
    ctx->vp_use = ctx->calls;
  }
  // the operators below size their shot batches from what is left of the budget
  struct Guard {
    fwime_ctx_t *c;
    size_t saved;
    ~Guard() {
      c->budget = saved;
      c->vp_busy = false;
    }
  } guard{ctx, ctx->budget};
  ctx->vp_busy = true;
  if (ctx->budget) ctx->budget = ctx->budget > ctx->vp_bytes ? ctx->budget - ctx->vp_bytes : 1;

  auto dot = [&](const float *x, const float *y, long n, double &out) -> int {
    HIPCHK(launch_dot(x, y, n, part, res, st));
    HIPCHK(hipMemcpyAsync(ctx->host_red, res, sizeof(double), hipMemcpyDeviceToHost, st));
    HIPCHK(hipStreamSynchronize(st));
    out = ctx->host_red[0];
    return FWIME_OK;
  };
  std::vector<float> e2(nh);
  for (int h = 0; h < nh; ++h) e2[h] = (float)(eps * eps * dso[h] * dso[h]);
  HIPCHK(hipMemcpyAsync(e2d2, e2.data(), nh * sizeof(float), hipMemcpyHostToDevice, st));

  // residual of the background model and the right-hand side
  if ((rc = fwime_model(ctx, g, vel, geo, dtmp, stream))) return rc;
  HIPCHK(launch_sub(dobs, dtmp, dres, ndata, st));
  double c0 = 0.0, rr = 0.0;
  if ((rc = dot(dres, dres, ndata, c0))) return rc;
  c0 *= 0.5;
  AdjCache *cp = use_cache ? &cache : nullptr;
  auto fwd = [&](const float *x, float *d) {
    return tau ? fwime_born_ext_tau_fwd(ctx, g, vel, geo, nh, lag, x, d, stream)
               : born_ext_fwd_run(ctx, g, vel, geo, nh, x, d, stream, cache.hist);
  };
  auto adj = [&](const float *d, float *x) {
    return tau ? fwime_born_ext_tau_adj(ctx, g, vel, geo, nh, lag, d, x, stream)
               : born_ext_adj_run(ctx, g, vel, geo, nh, d, x, stream, cp);
  };
  if ((rc = adj(dres, b))) return rc;
  HIPCHK(launch_zero(ptilde_out, img, st));
  HIPCHK(hipMemcpyAsync(r, b, img * sizeof(float), hipMemcpyDeviceToDevice, st));
  HIPCHK(hipMemcpyAsync(sdir, b, img * sizeof(float), hipMemcpyDeviceToDevice, st));
  if ((rc = dot(r, r, img, rr))) return rc;
  phi_out[0] = c0;
  int k = 0;
  for (; k < niter; ++k) {
    // q = (B~* B~ + eps^2 D* D) s
    if ((rc = fwd(sdir, dtmp))) return rc;
    if ((rc = adj(dtmp, q))) return rc;
    HIPCHK(launch_add_diag(q, sdir, e2d2, plane, nh, st));
    double curv = 0.0;
    if ((rc = dot(sdir, q, img, curv))) return rc;
    if (!(curv > 0.0) || !std::isfinite(curv)) break;    // no curvature left along s: p~ is final
    const double alpha = rr / curv;
    HIPCHK(launch_cg_step(ptilde_out, r, sdir, q, (float)alpha, img, st));
    double rr_new = 0.0, bp = 0.0, rp = 0.0;
    if ((rc = dot(r, r, img, rr_new)) || (rc = dot(b, ptilde_out, img, bp)) || (rc = dot(r, ptilde_out, img, rp)))
      return rc;
    phi_out[k + 1] = c0 - 0.5 * (bp + rp);
    HIPCHK(launch_cg_dir(sdir, r, (float)(rr_new / rr), img, st));
    rr = rr_new;
  }
  for (int j = k + 1; j <= niter; ++j) phi_out[j] = phi_out[k];
  return FWIME_OK;
}

int fwime_vp_solve(fwime_ctx_t *ctx, const fwime_grid_t *g, const float *vel, const fwime_geom_t *geo,
                   int32_t nh, const float *dobs, double eps, const double *dso, int32_t niter,
                   float *ptilde_out, double *phi_out, void *stream) {
  return vp_solve_run(ctx, g, vel, geo, nh, false, 0, dobs, eps, dso, niter, ptilde_out, phi_out, stream);
}

int fwime_vp_solve_tau(fwime_ctx_t *ctx, const fwime_grid_t *g, const float *vel, const fwime_geom_t *geo,
                       int32_t ntau, int32_t lag, const float *dobs, double eps, const double *dso, int32_t niter,
                       float *ptau_out, double *phi_out, void *stream) {
  return vp_solve_run(ctx, g, vel, geo, ntau, true, lag, dobs, eps, dso, niter, ptau_out, phi_out, stream);
}

int fwime_gradient(fwime_ctx_t *ctx, const fwime_grid_t *g, const float *vel, const fwime_geom_t *geo, int32_t nh,
                   const float *ptilde, const float *dobs, double eps, const double *dso, double *obj,
                   float *grad_vel, float *grad_ptilde, void *stream) {
  if (!ctx) return FWIME_EINVAL;
  ctx->err.clear();
  hipStream_t st = (hipStream_t)stream;
  int rc;
  if ((rc = check_grid(ctx, g)) || (rc = check_geom(ctx, g, geo)) || (rc = check_nh(ctx, g, nh))) return rc;
  if (!ptilde || !dobs || !dso || !obj || !grad_vel || !grad_ptilde)
    return set_err(ctx, FWIME_EINVAL, "null pointer argument");
  if (!std::isfinite(eps)) return set_err(ctx, FWIME_EINVAL, "eps must be finite");
  for (int h = 0; h < nh; ++h)
    if (!std::isfinite(dso[h])) return set_err(ctx, FWIME_EINVAL, "dso must be finite");
  HIPCHK(hipSetDevice(ctx->device));
  const long ndata = (long)geo->nshots * geo->nrec * g->nt;
  if ((rc = check_inputs(ctx, g, vel, geo, {{ptilde, (long)nh * g->nx * g->nz}, {dobs, ndata}}, st))) return rc;

  Common c;
  c.d = make_dims(g, ctx->tile_x);
  const Dims &d = c.d;
  ExtGeom eg{d.nz, d.nx, d.nb, d.NZ, d.NX, d.LZ, nh, (nh - 1) / 2};
  const long img = (long)nh * d.nx * d.nz;
  const long nrt = (long)geo->nrec * g->nt;
  auto fixed = [&](const GradPlan &p) {
    return (size_t)d.field * 12 + (size_t)img * 4 * (5 + hist_parts(g->nt, p.K, img));
  };
  auto per_shot = [&](const GradPlan &p) {
    return grad_work_per_shot(d, p, ctx->two_step) + 2 * p.ck_stride * 4 + 2 * nrt * 4 + (long)geo->nrec * 64;
  };
  const int Sh = hist_batch(ctx, geo->nshots, (long)d.ntz2 * d.ntx, [&](int S) {
    const GradPlan p = grad_plan(d, g->nt, S);
    return fixed(p) + (size_t)per_shot(p) * S;
  }, &ctx->arena);
  const GradPlan pl = grad_plan(d, g->nt, Sh);
  const int S = Sh ? Sh : choose_batch(ctx, per_shot(pl), fixed(pl), geo->nshots);
  auto batches = split_batches(geo->nshots, S);
  choose_steps(ctx, c.d, S, false);
  TableSet ts = build_table_set(d, geo, batches, ctx->two_step);

  double *acc = nullptr;
  float *coef = nullptr, *imgs = nullptr, *gacc = nullptr, *uck = nullptr, *dck = nullptr,
        *drec = nullptr, *ddrec = nullptr, *e2d2 = nullptr;
  double *sumsq = nullptr, *rpart = nullptr;
  GradWork wk;
  Carve cv;
  cv.add(&c.V, d.field);
  cv.add(&c.gz, d.LZ);
  cv.add(&c.gx, d.NX + kGxPad);
  cv.add(&c.tables, table_set_ints(ts) + 64 * batches.size() * 8);
  cv.add(&sumsq, 2);
  cv.add(&rpart, red_partials());
  cv.add(&e2d2, nh);
  cv.add(&coef, img);
  cv.add(&acc, img);
  cv.add(&imgs, img);
  cv.add(&gacc, d.field);
  cv.add(&uck, pl.ck_stride * S);
  cv.add(&dck, pl.ck_stride * S);
  carve_work(cv, wk, d, pl, S, ctx->two_step);
  wk.nparts = hist_parts(g->nt, pl.K, img);
  cv.add(&wk.parts, wk.nparts * img);
  cv.add(&drec, nrt * S);
  cv.add(&ddrec, nrt * S);
  if ((rc = arena_get(ctx, cv)))
    return or_frugally(ctx, rc, d.T == 4 || Sh > 0, [&] {
      return fwime_gradient(ctx, g, vel, geo, nh, ptilde, dobs, eps, dso, obj, grad_vel, grad_ptilde, stream);
    });
  if ((rc = upload_tables(ctx, ts, c.tables, st))) return rc;
  if ((rc = setup_common(ctx, c, g, vel, st))) return rc;
  std::vector<float> e2(nh);
  for (int h = 0; h < nh; ++h) e2[h] = (float)(eps * eps * dso[h] * dso[h]);
  HIPCHK(hipMemcpyAsync(e2d2, e2.data(), nh * sizeof(float), hipMemcpyHostToDevice, st));
  HIPCHK(launch_ext_coef(ptilde, vel, eg, (float)g->dt, coef, st));
  HIPCHK(launch_zero_d(acc, img, st));
  HIPCHK(launch_zero(gacc, d.field, st));
  HIPCHK(launch_zero_d(sumsq, 2, st));

  for (size_t bi = 0; bi < batches.size(); ++bi) {
    const int s0 = batches[bi].first, Sb = batches[bi].second;
    const DevTables &t = ts.dev[bi];
    const float *wav_b = geo->wavelet + (long)s0 * g->nt;
    if ((rc = grad_forward_batch(ctx, c, eg, pl, g, Sb, t, wav_b, coef, uck, dck, wk, drec, ddrec, geo->nrec, st)))
      return rc;
    HIPCHK(launch_residual(drec, ddrec, dobs + (long)s0 * nrt, nrt * Sb, rpart, sumsq, st));
    if ((rc = grad_backward_batch(ctx, c, eg, pl, g, Sb, t, wav_b, coef, uck, dck, wk, drec, acc, gacc, st)))
      return rc;
  }
  HIPCHK(launch_ext_finalize(acc, vel, eg, (float)g->dt, nullptr, nullptr, imgs, st));
  HIPCHK(launch_grad_finalize(gacc, c.V, vel, eg, (float)g->dt, ptilde, imgs, grad_vel, st));
  HIPCHK(launch_ext_finalize(acc, vel, eg, (float)g->dt, ptilde, e2d2, grad_ptilde, st));
  HIPCHK(launch_objective(sumsq, ptilde, e2d2, eg, rpart, obj, st));
  return FWIME_OK;
}

// ---------------------------------------------------------------------------
// FWIME objective and gradients with the time-lag extension.  Every history
// of a shot batch is kept whole (slot n of shot s at base + s hs + n field,
// hs = (nt + 1) fields): T2u and T2du~ of every step, the adjoint field of
// every time, and the scattering source, whose buffer then holds the spread
// e; rho runs in a ring of chunks of kTauChunk steps, each followed by its
// share of the gradient sums.
// ---------------------------------------------------------------------------
int fwime_gradient_tau(fwime_ctx_t *ctx, const fwime_grid_t *g, const float *vel, const fwime_geom_t *geo,
                       int32_t ntau, int32_t lag, const float *ptau, const float *dobs, double eps,
                       const double *dso, double *obj, float *grad_vel, float *grad_ptau, void *stream) {
  if (!ctx) return FWIME_EINVAL;
  ctx->err.clear();
  hipStream_t st = (hipStream_t)stream;
  int rc;
  if ((rc = check_grid(ctx, g)) || (rc = check_geom(ctx, g, geo)) || (rc = check_tau(ctx, g, ntau, lag))) return rc;
  if (!ptau || !dobs || !dso || !obj || !grad_vel || !grad_ptau)
    return set_err(ctx, FWIME_EINVAL, "null pointer argument");
  if (!(eps >= 0.0) || !std::isfinite(eps)) return set_err(ctx, FWIME_EINVAL, "eps must be finite and >= 0");
  for (int h = 0; h < ntau; ++h)
    if (!std::isfinite(dso[h])) return set_err(ctx, FWIME_EINVAL, "dso weights must be finite");
  HIPCHK(hipSetDevice(ctx->device));
  const long plane = (long)g->nx * g->nz, img = (long)ntau * plane;
  const long nrt = (long)geo->nrec * g->nt;
  if ((rc = check_inputs(ctx, g, vel, geo, {{ptau, img}, {dobs, nrt * geo->nshots}}, st))) return rc;

  constexpr int kTauChunk = 64;
  Common c;
  c.d = make_dims(g, ctx->tile_x);
  const Dims &d = c.d;
  ExtGeom eg{d.nz, d.nx, d.nb, d.NZ, d.NX, d.LZ, ntau, (ntau - 1) / 2};
  const int ns = g->nt - 1, R = g->nt + 1, RR = kTauChunk + 2;
  const long hs = (long)R * d.field, rs = (long)RR * d.field;
  // per shot: four histories of R fields, the rho ring, the wavefield rings
  // (8 fields) and the background's BF16 low parts (2), receiver data of u
  // and du~, tables
  const long per_shot = (4L * R + RR + 10) * d.field * 4 + 2 * nrt * 4 + (long)geo->nrec * 64;
  const size_t fixed = (size_t)d.field * 8 + (size_t)img * 4 * 3;
  const int S = choose_batch(ctx, per_shot, fixed, geo->nshots);
  auto batches = split_batches(geo->nshots, S);
  choose_steps(ctx, c.d, S, true);
  TableSet ts = build_table_set(d, geo, batches, true);

  float *coef = nullptr, *coefr = nullptr, *acc = nullptr, *gacc = nullptr, *e2d2 = nullptr, *pairs = nullptr,
        *hu = nullptr, *hdu = nullptr, *lam = nullptr, *sc = nullptr, *rho = nullptr, *drec = nullptr,
        *ddrec = nullptr;
  unsigned short *lows = nullptr;
  double *sumsq = nullptr, *rpart = nullptr;
  Carve cv;
  cv.add(&c.V, d.field);
  cv.add(&c.gz, d.LZ);
  cv.add(&c.gx, d.NX + kGxPad);
  cv.add(&c.tables, table_set_ints(ts) + 64 * batches.size() * 8);
  cv.add(&sumsq, 2);
  cv.add(&rpart, red_partials());
  cv.add(&e2d2, ntau);
  cv.add(&coef, img);
  cv.add(&coefr, img);
  cv.add(&acc, img);
  cv.add(&gacc, d.field);
  cv.add(&pairs, 8 * d.field * S);
  cv.add(&lows, 4 * d.field * S);
  cv.add(&hu, hs * S);
  cv.add(&hdu, hs * S);
  cv.add(&lam, hs * S);
  cv.add(&sc, hs * S);
  cv.add(&rho, rs * S);
  cv.add(&drec, nrt * S);
  cv.add(&ddrec, nrt * S);
  if ((rc = arena_get(ctx, cv)))
    return or_frugally(ctx, rc, d.T == 4, [&] {
      return fwime_gradient_tau(ctx, g, vel, geo, ntau, lag, ptau, dobs, eps, dso, obj, grad_vel, grad_ptau, stream);
    });
  if ((rc = upload_tables(ctx, ts, c.tables, st))) return rc;
  if ((rc = setup_common(ctx, c, g, vel, st))) return rc;
  std::vector<float> e2(ntau);
  for (int h = 0; h < ntau; ++h) e2[h] = (float)(eps * eps * dso[h] * dso[h]);
  HIPCHK(hipMemcpyAsync(e2d2, e2.data(), ntau * sizeof(float), hipMemcpyHostToDevice, st));
  HIPCHK(launch_ext_coef(ptau, vel, eg, (float)g->dt, coef, st));
  // the spread e_m = sum_k c_k lam_{m + 2kL} is the lag scatter with the
  // coefficient planes in reverse order: c'_k = c_{-k}
  for (int k = 0; k < ntau; ++k)
    HIPCHK(hipMemcpyAsync(coefr + (long)k * plane, coef + (long)(ntau - 1 - k) * plane, plane * sizeof(float),
                          hipMemcpyDeviceToDevice, st));
  HIPCHK(launch_zero(acc, img, st));
  HIPCHK(launch_zero(gacc, d.field, st));
  HIPCHK(launch_zero_d(sumsq, 2, st));

  for (size_t bi = 0; bi < batches.size(); ++bi) {
    const int s0 = batches[bi].first, Sb = batches[bi].second;
    const DevTables &t = ts.dev[bi];
    // background: T2u of every step, and its receiver data
    if ((rc = tau_background(ctx, c, g, geo, s0, Sb, t, pairs, lows, hu, hs, st, drec))) return rc;
    // scattering source history, then du~ with its T2 history and receivers
    HIPCHK(launch_tau_scatter(coef, eg, lag, hu, sc, d.field, hs, ns, Sb, st));
    float *wp = pairs + 4 * d.field * Sb;
    HIPCHK(zero_start(wp, d, Sb, st));
    Ring4 fw(wp, d.field * Sb);
    rc = march2(ctx, c, fw, Sb, 0, ns, kModeT2 | kModeDsrc, [&](Steps &p, int n, int k) {
      with_dsrc2(p, sc + (long)n * d.field, d.field, k, hs);
      with_dense_range(p, eg, 0);
      with_t2(p, hdu + (long)n * d.field, d.field, k, hs);
      with_rec_extract(p, t, ddrec, g->nt, n);
    }, st);
    if (rc) return rc;
    HIPCHK(launch_gather(fw.cur(), d.field, t.cells, Sb, geo->nrec, ddrec, g->nt, g->nt - 1, st));
    // residual r = R(u + du~) - d_obs (into drec) and its sum of squares
    HIPCHK(launch_residual(drec, ddrec, dobs + (long)s0 * nrt, nrt * Sb, rpart, sumsq, st));
    // adjoint field of every time
    HIPCHK(zero_end(lam, hs, R, d, Sb, st));
    if ((rc = march2_back_lambda(ctx, c, lam, hs, R, Sb, 0, g->nt - 1, t, drec, g->nt, st))) return rc;
    // spread e over the adjoint history (slots 0 .. ns-1; zero from ns on)
    HIPCHK(launch_zero_fields(sc + (long)ns * d.field, hs, Sb, 2 * d.field, st));
    HIPCHK(launch_tau_scatter(coefr, eg, lag, lam, sc, d.field, hs, ns, Sb, st));
    // rho = M^-T nu, nu^k = e_{k-1}/g - 2 e_k + g e_{k+1}, chunk by chunk
    // backwards, each chunk followed by its gradient sums
    auto e_slot = [&](int k) { return sc + (long)k * d.field; };
    HIPCHK(zero_end(rho, rs, RR, d, Sb, st));
    const int nchunk = (ns + kTauChunk - 1) / kTauChunk;
    for (int j = nchunk - 1; j >= 0; --j) {
      const int n0 = j * kTauChunk, n1 = std::min(n0 + kTauChunk, ns);
      rc = march2_back_ring(ctx, c, rho, rs, RR, Sb, n0, n1, kModeNu, [&](Steps &p, int k, int kk) {
        with_nu(p, e_slot, k, kk, hs);
        with_dense_range(p, eg, 0);
      }, st);
      if (rc) return rc;
      HIPCHK(launch_grad_accum2(hu + (long)n0 * d.field, hdu + (long)n0 * d.field, d.field, hs, lam, d.field, hs, R,
                                n0, rho, d.field, rs, RR, n0, Sb, n1 - n0, kTauChunk, d.NZ, d.NX, d.LZ, gacc, st));
    }
    // B~_tau^T r (scaled by 2 / (v^3 dt^2) in the kernel)
    HIPCHK(launch_tau_image(hu, d.field, hs, lam, d.field, hs, ns, Sb, eg, lag, vel, (float)g->dt, acc, st));
  }
  HIPCHK(launch_grad_finalize(gacc, c.V, vel, eg, (float)g->dt, ptau, acc, grad_vel, st));
  HIPCHK(hipMemcpyAsync(grad_ptau, acc, img * sizeof(float), hipMemcpyDeviceToDevice, st));
  HIPCHK(launch_add_diag(grad_ptau, ptau, e2d2, plane, ntau, st));
  HIPCHK(launch_objective(sumsq, ptau, e2d2, eg, rpart, obj, st));
  return FWIME_OK;
}

// ---------------------------------------------------------------------------
void fwime_tape_free(fwime_tape_t *tape) {
  if (!tape) return;
  if (tape->mem) {
    (void)hipSetDevice(tape->device);
    (void)hipDeviceSynchronize();
    void *drop = tape->mem;
    if (fwime_ctx_t *ctx = tape->ctx) {
      std::lock_guard<std::mutex> lock(ctx->tape_mu);
      ctx->tape_bytes -= tape->bytes;
      if (tape->pl.hist) ctx->tape_hist -= tape->bytes;
      ctx->tapes.erase(std::find(ctx->tapes.begin(), ctx->tapes.end(), tape));
      if (!ctx->budget && tape->capacity > ctx->spare_bytes) {   // idle on every stream: kept
        drop = ctx->spare;
        ctx->spare = tape->mem;
        ctx->spare_bytes = tape->capacity;
        ctx->spare_use = ctx->calls.load();
      }
    }
    if (drop) (void)hipFree(drop);
  }
  delete tape;
}

int fwime_forward_tape(fwime_ctx_t *ctx, const fwime_grid_t *g, const float *vel, const fwime_geom_t *geo,
                       int32_t nh, const float *ptilde, float *data, fwime_tape_t **tape_out, void *stream) {
  if (!ctx) return FWIME_EINVAL;
  ctx->err.clear();
  hipStream_t st = (hipStream_t)stream;
  int rc;
  if (!tape_out) return set_err(ctx, FWIME_EINVAL, "tape_out is null");
  *tape_out = nullptr;
  if ((rc = check_grid(ctx, g)) || (rc = check_geom(ctx, g, geo)) || (rc = check_nh(ctx, g, nh))) return rc;
  if (!ptilde || !data) return set_err(ctx, FWIME_EINVAL, "null pointer argument");
  HIPCHK(hipSetDevice(ctx->device));
  if ((rc = check_inputs(ctx, g, vel, geo, {{ptilde, (long)nh * g->nx * g->nz}}, st))) return rc;

  fwime_tape_t *tp = new fwime_tape_t();
  tp->ctx = ctx;
  tp->device = ctx->device;
  tp->g = *g;
  tp->nh = nh;
  tp->nshots = geo->nshots;
  tp->nrec = geo->nrec;
  tp->d = make_dims(g, ctx->tile_x);
  const Dims &d = tp->d;
  ExtGeom eg{d.nz, d.nx, d.nb, d.NZ, d.NX, d.LZ, nh, (nh - 1) / 2};
  const long img = (long)nh * d.nx * d.nz;
  const long nrt = (long)geo->nrec * g->nt;
  // checkpoints (or whole histories) of every shot live in the tape; working
  // fields in the arena
  const size_t rest = 2 * nrt * 4 + (size_t)geo->nrec * 64;
  // whole histories only if every shot's fit (the tape holds them all)
  auto beside = [&](int S) {                       // in the arena
    const GradPlan p = grad_plan(d, g->nt, S);
    return (grad_work_per_shot(d, p, ctx->two_step) - 2L * p.seg_stride * 4 + rest) * S +
           (size_t)img * 4 * (5 + hist_parts(g->nt, p.K, img));
  };
  const int Sh = hist_batch(ctx, geo->nshots, 0, [&](int S) {
    return beside(S) + (size_t)(2L * (g->nt - 1) * S + 2) * d.field * 4;
  }, nullptr, beside(geo->nshots));
  tp->pl = grad_plan(d, g->nt, Sh);
  const GradPlan &pl = tp->pl;
  const size_t per_shot = grad_work_per_shot(d, pl, ctx->two_step) + rest;
  const size_t tape_fixed = (size_t)(2 * pl.ck_stride * 4) * geo->nshots;
  const int S = Sh ? Sh : choose_batch(ctx, per_shot, tape_fixed + (size_t)d.field * 8, geo->nshots);
  tp->batches = split_batches(geo->nshots, S);
  choose_steps(ctx, tp->d, S, false);
  tp->ts = build_table_set(d, geo, tp->batches, ctx->two_step);

  Carve tc;   // tape memory
  tc.add(&tp->V, d.field);
  tc.add(&tp->gz, d.LZ);
  tc.add(&tp->gx, d.NX + kGxPad);
  tc.add(&tp->tables, table_set_ints(tp->ts) + 64 * tp->batches.size() * 8);
  tc.add(&tp->vel, (long)d.nx * d.nz);
  tc.add(&tp->pt, img);
  tc.add(&tp->coef, img);
  tc.add(&tp->wav, (long)geo->nshots * g->nt);
  tc.add(&tp->uck, pl.hist ? pl.seg_stride * geo->nshots : pl.ck_stride * geo->nshots);
  tc.add(&tp->dck, pl.hist ? pl.seg_stride * geo->nshots : pl.ck_stride * geo->nshots);
  const bool less = d.T == 4 || Sh > 0;
  auto again = [&] { return fwime_forward_tape(ctx, g, vel, geo, nh, ptilde, data, tape_out, stream); };
  if (ctx->budget && live_tape_bytes(ctx) + tc.total + ctx->arena_bytes > ctx->budget) {
    delete tp;
    return or_frugally(ctx, set_err(ctx, FWIME_ENOMEM, "tape does not fit the HBM budget"), less, again);
  }
  bool small = false;                      // a fraction of the spare, which waits for a large tape
  {
    std::lock_guard<std::mutex> lock(ctx->tape_mu);
    small = tc.total < ctx->spare_bytes / 4;
    if (!small && tc.total <= ctx->spare_bytes) {
      tp->mem = ctx->spare;
      tp->capacity = ctx->spare_bytes;
      ctx->spare = nullptr;
      ctx->spare_bytes = 0;
    }
  }
  if (!tp->mem) {
    if (!small) release_spare(ctx);        // too small: room for the larger one
    if (device_alloc(ctx, &tp->mem, tc.total) != hipSuccess) {
      (void)hipGetLastError();
      delete tp;
      return or_frugally(ctx, set_err(ctx, FWIME_ENOMEM, "hipMalloc of the tape failed"), less, again);
    }
    tp->capacity = tc.total;
  }
  tp->bytes = tc.total;
  {
    std::lock_guard<std::mutex> lock(ctx->tape_mu);
    ctx->tape_bytes += tc.total;
    if (pl.hist) ctx->tape_hist += tc.total;
    ctx->tapes.push_back(tp);
  }
  {
    char *p = (char *)tp->mem;
    for (auto &it : tc.items) {
      *it.first = p;
      p += it.second;
    }
  }
  auto fail = [&](int code) {
    fwime_tape_free(tp);
    return code;
  };
  if ((rc = upload_tables(ctx, tp->ts, tp->tables, st))) return fail(rc);
  Common c;
  c.d = d;
  c.V = tp->V;
  c.gz = tp->gz;
  c.gx = tp->gx;
  c.tables = tp->tables;
  if ((rc = setup_common(ctx, c, g, vel, st))) return fail(rc);
  if (hipMemcpyAsync(tp->vel, vel, sizeof(float) * d.nx * d.nz, hipMemcpyDeviceToDevice, st) != hipSuccess ||
      hipMemcpyAsync(tp->pt, ptilde, sizeof(float) * img, hipMemcpyDeviceToDevice, st) != hipSuccess ||
      hipMemcpyAsync(tp->wav, geo->wavelet, sizeof(float) * geo->nshots * g->nt, hipMemcpyDeviceToDevice, st) !=
          hipSuccess)
    return fail(set_err(ctx, FWIME_EHIP, "tape copy failed"));
  if (launch_ext_coef(tp->pt, tp->vel, eg, (float)g->dt, tp->coef, st) != hipSuccess)
    return fail(set_err(ctx, FWIME_EHIP, "coefficient launch failed"));

  float *drec = nullptr, *ddrec = nullptr;
  GradWork wk;
  Carve cv;
  carve_work(cv, wk, d, pl, S, ctx->two_step, !pl.hist);
  cv.add(&drec, nrt * S);
  cv.add(&ddrec, nrt * S);
  if ((rc = arena_get(ctx, cv))) return or_frugally(ctx, fail(rc), less, again);
  if (pl.hist) {
    wk.t2u = tp->uck;
    wk.t2d = tp->dck;
  }
  for (size_t bi = 0; bi < tp->batches.size(); ++bi) {
    const int s0 = tp->batches[bi].first, Sb = tp->batches[bi].second;
    if ((rc = grad_forward_batch(ctx, c, eg, pl, g, Sb, tp->ts.dev[bi], tp->wav + (long)s0 * g->nt, tp->coef,
                                 tp->uck + s0 * pl.ck_stride, tp->dck + s0 * pl.ck_stride, wk, drec, ddrec,
                                 geo->nrec, st)))
      return fail(rc);
    // data = f(m) + B~ p~ for the batch
    if (launch_residual_sum(data + (long)s0 * nrt, drec, ddrec, nrt * Sb, st) != hipSuccess)
      return fail(set_err(ctx, FWIME_EHIP, "data sum failed"));
  }
  *tape_out = tp;
  return FWIME_OK;
}

int fwime_backward_tape(fwime_ctx_t *ctx, fwime_tape_t *tp, const float *adjsrc, float *grad_vel,
                        float *grad_ptilde, void *stream) {
  if (!ctx) return FWIME_EINVAL;
  ctx->err.clear();
  hipStream_t st = (hipStream_t)stream;
  int rc;
  if (!tp || tp->ctx != ctx) return set_err(ctx, FWIME_EINVAL, "tape is null or belongs to another context");
  if (tp->used) return set_err(ctx, FWIME_EINVAL, "the tape's checkpoints were consumed by a previous backward");
  if (!adjsrc || !grad_vel || !grad_ptilde) return set_err(ctx, FWIME_EINVAL, "null pointer argument");
  HIPCHK(hipSetDevice(ctx->device));
  const fwime_grid_t *g = &tp->g;
  const Dims &d = tp->d;
  GradPlan pl = tp->pl;
  ExtGeom eg{d.nz, d.nx, d.nb, d.NZ, d.NX, d.LZ, tp->nh, (tp->nh - 1) / 2};
  const long img = (long)tp->nh * d.nx * d.nz;
  const long nrt = (long)tp->nrec * g->nt;
  {
    // finiteness of the adjoint source, checked before anything is written
    std::vector<double> r3;
    if ((rc = device_ranges(ctx, {{adjsrc, nrt * tp->nshots}}, st, r3))) return rc;
    if (r3[2] > 0) return set_err(ctx, FWIME_ENONFINITE, "adjoint source has non-finite values");
  }
  int S = 0;
  for (auto &b : tp->batches) S = std::max(S, b.second);
  double *acc = nullptr;
  float *imgs = nullptr, *gacc = nullptr;
  GradWork wk;
  auto scratch = [&]() {
    Carve cv;
    cv.add(&acc, img);
    cv.add(&imgs, img);
    cv.add(&gacc, d.field);
    carve_work(cv, wk, d, pl, S, ctx->two_step, !pl.hist);
    wk.nparts = hist_parts(g->nt, pl.K, img);
    cv.add(&wk.parts, wk.nparts * img);
    return arena_get(ctx, cv);
  };
  rc = scratch();
  if (rc == FWIME_ENOMEM && pl.hist && pl.K > pl.seg) {
    pl.set_segment(d, g->nt, pl.seg);              // rings of checkpointed segments, then
    rc = scratch();
  }
  if (rc) return rc;
  if (pl.hist) {
    wk.t2u = tp->uck;
    wk.t2d = tp->dck;
  }
  Common c;
  c.d = d;
  c.V = tp->V;
  c.gz = tp->gz;
  c.gx = tp->gx;
  c.tables = tp->tables;
  if ((rc = setup_common(ctx, c, g, tp->vel, st))) return rc;
  HIPCHK(launch_zero_d(acc, img, st));
  HIPCHK(launch_zero(gacc, d.field, st));
  tp->used = true;   // backward recomputes the segments in place over the checkpoints
  for (size_t bi = 0; bi < tp->batches.size(); ++bi) {
    const int s0 = tp->batches[bi].first, Sb = tp->batches[bi].second;
    if ((rc = grad_backward_batch(ctx, c, eg, pl, g, Sb, tp->ts.dev[bi], tp->wav + (long)s0 * g->nt, tp->coef,
                                  tp->uck + s0 * pl.ck_stride, tp->dck + s0 * pl.ck_stride, wk,
                                  adjsrc + (long)s0 * nrt, acc, gacc, st)))
      return rc;
  }
  HIPCHK(launch_ext_finalize(acc, tp->vel, eg, (float)g->dt, nullptr, nullptr, imgs, st));
  HIPCHK(launch_grad_finalize(gacc, c.V, tp->vel, eg, (float)g->dt, tp->pt, imgs, grad_vel, st));
  HIPCHK(hipMemcpyAsync(grad_ptilde, imgs, sizeof(float) * img, hipMemcpyDeviceToDevice, st));
  return FWIME_OK;
}

}  // extern "C"

namespace {

// ---------------------------------------------------------------------------
// Many modeling jobs of different grids in one launch per time step (two
// time steps per launch by default).
//
// Every job keeps its own padded velocity, taper, receiver tables and four
// (two with one step per launch) field buffers per shot; a device array of
// job descriptors lets one k_step2_multi (k_step_multi) launch advance all of
// them.  The time loop is recorded once as a graph of G (stencil, step-counter
// bump) node pairs on a private capture stream and replayed on the caller's
// stream until the longest job is done.
// The tile width comes from an autotuner: for a batch signature not seen
// before, each candidate width is timed on scratch fields (zero initial
// state, real velocity and sources) and the fastest is cached in the context.
// ---------------------------------------------------------------------------
struct BatchPlan {
  bool two = false;              // two time steps per launch (k_step2_multi)
  std::vector<int> order;        // position k in the launch -> caller's job index
  std::vector<Common> com;       // per position
  std::vector<TableSet> ts;
  std::vector<BatchJob> jobs;    // one-step descriptors
  std::vector<BatchJob2> jobs2;  // two-step descriptors
  std::vector<int> prefix;       // tiles before position k
  int total = 0;
  int nt_max = 0;
  bool fs = false;               // some job has a free surface
  int *dtile_job = nullptr;      // device: position k of every tile (two-step plans)
  int stride() const { return two ? 2 : 1; }
  // launches until the longest job has sampled its last time
  long launches() const { return two ? (nt_max - 1) / 2 + 1 : nt_max; }
  int nt_at(int k) const { return two ? jobs2[k].nt : jobs[k].nt; }
};

// Jobs are laid out in order of decreasing time-axis length, so the jobs still
// running at step n are a prefix of the list and a launch can stop at that
// prefix's last tile.
int batch_plan(fwime_ctx_t *ctx, int njobs, const fwime_job_t *jobs, int tx, BatchPlan &bp,
               std::vector<std::pair<void **, size_t>> *) {
  bp.two = ctx->two_step;
  bp.order.resize(njobs);
  for (int j = 0; j < njobs; ++j) bp.order[j] = j;
  std::stable_sort(bp.order.begin(), bp.order.end(),
                   [&](int a, int b) { return jobs[a].grid.nt > jobs[b].grid.nt; });
  bp.com.assign(njobs, Common());
  bp.ts.clear();
  bp.jobs.assign(bp.two ? 0 : njobs, BatchJob());
  bp.jobs2.assign(bp.two ? njobs : 0, BatchJob2());
  bp.prefix.assign(njobs + 1, 0);
  bp.total = 0;
  bp.nt_max = 0;
  bp.fs = false;
  for (int k = 0; k < njobs; ++k) {
    const int j = bp.order[k];
    bp.fs = bp.fs || jobs[j].grid.free_surface != 0;
    bp.com[k].d = make_dims(&jobs[j].grid, tx);
    const Dims &d = bp.com[k].d;
    bp.ts.push_back(build_table_set(d, &jobs[j].geom, {{0, jobs[j].geom.nshots}}, bp.two));
    if (bp.two) {
      bp.jobs2[k].tile_begin = bp.total;
      bp.jobs2[k].t0 = 0;
      bp.jobs2[k].nt = jobs[j].grid.nt;
      bp.total += d.ntz2 * d.ntx * jobs[j].geom.nshots;
    } else {
      bp.jobs[k].tile_begin = bp.total;
      bp.jobs[k].t0 = 0;
      bp.jobs[k].nt = jobs[j].grid.nt;
      bp.total += d.ntz * d.ntx * jobs[j].geom.nshots;
    }
    bp.prefix[k + 1] = bp.total;
    bp.nt_max = std::max(bp.nt_max, jobs[j].grid.nt);
  }
  return FWIME_OK;
}

// tiles of the jobs whose time index n is still within [0, nt - 1]
int batch_active_tiles(const BatchPlan &bp, long n) {
  int k = 0;
  const int nj = (int)bp.order.size();
  while (k < nj && n <= bp.nt_at(k) - 1) ++k;
  return bp.prefix[k];
}

// one multi-job launch (one or two time steps).  With a device step counter
// (graph replay) the launch is followed by the counter's bump; without one
// the global step is passed by value and nothing else is launched.
hipError_t batch_launch(const BatchPlan &bp, const void *djobs, int tiles, int *dstep, int step_val, int tx,
                        hipStream_t st) {
  const int nj = (int)bp.order.size();
  hipError_t e = bp.two ? launch_step2_multi((const BatchJob2 *)djobs, bp.dtile_job, nj, tiles, dstep, step_val, tx,
                                             bp.fs, st)
                        : launch_step_multi((const BatchJob *)djobs, nj, tiles, dstep, step_val, tx, bp.fs, st);
  if (e != hipSuccess || !dstep) return e;
  return launch_bump(dstep, bp.stride(), st);
}

// Scratch of a batch and what its launches read: the tables, tapers and
// descriptors of all jobs go to the device as one blob, and one launch
// prepares every job's velocity and zero start.  (A copy each for a job's
// tables and two tapers and a launch each for its velocity and fields were 240
// commands for 48 jobs, 2 ms of a 49 ms call.)
int batch_carve_and_setup(fwime_ctx_t *ctx, int njobs, const fwime_job_t *jobs, BatchPlan &bp, void **djobs,
                          int **dstep, hipStream_t st) {
  Carve cv;
  std::vector<float *> fields(njobs);
  const int nf = bp.two ? 4 : 2;
  const size_t jb_bytes = bp.two ? sizeof(BatchJob2) : sizeof(BatchJob);
  static_assert(sizeof(BatchJob2) % 8 == 0 && sizeof(BatchJob) % 8 == 0 && sizeof(PrepJob) % 8 == 0, "blob pieces");
  size_t blob_ints = 64 * 4 + (jb_bytes + sizeof(PrepJob)) / 4 * njobs + (bp.two ? bp.total : 0);
  for (int k = 0; k < njobs; ++k) {
    const int j = bp.order[k];
    const Dims &d = bp.com[k].d;
    cv.add(&bp.com[k].V, d.field);
    cv.add(&fields[k], nf * d.field * jobs[j].geom.nshots);
    blob_ints += table_set_ints(bp.ts[k]) + 64 * 8 + d.LZ + d.NX + kGxPad + 2 * 64;
  }
  int *dblob = nullptr;
  cv.add(&dblob, blob_ints);
  cv.add(dstep, 1);
  int rc = arena_get(ctx, cv);
  if (rc) return rc;
  std::vector<int> blob;
  blob.reserve(blob_ints);
  // piece of `nint` ints on a 64-int boundary: its place in the blob
  auto piece = [&](size_t nint) {
    const size_t off = (blob.size() + 63) / 64 * 64;
    blob.resize(off + nint);
    return off;
  };
  std::vector<PrepJob> prep(njobs);
  int blocks = 0;
  for (int k = 0; k < njobs; ++k) {
    const int j = bp.order[k];
    Common &c = bp.com[k];
    const Dims &d = c.d;
    const fwime_grid_t *g = &jobs[j].grid;
    const int S = jobs[j].geom.nshots;
    layout_tables(bp.ts[k], blob, dblob);
    for (int axis = 0; axis < 2; ++axis) {
      std::vector<float> t;
      if (axis == 0) taper_host(d.nz, d.nb, g->sponge_alpha, d.LZ, t);
      else taper_host(d.nx, d.nb, g->sponge_alpha, d.NX + kGxPad, t);
      const size_t off = piece(t.size());
      std::memcpy(blob.data() + off, t.data(), t.size() * sizeof(float));
      (axis == 0 ? c.gz : c.gx) = reinterpret_cast<float *>(dblob + off);
    }
    common_args(c, g);
    // u^{-1} = u^0 = 0
    const long nzero = 2 * d.field * S;
    const int nb = (int)std::min<long>(512, (std::max(nzero, d.field) + 4095) / 4096);
    prep[k] = PrepJob{jobs[j].vel, c.V, fields[k], nzero, d.nz, d.nx, d.nb, d.NZ, d.NX, d.LZ, (float)g->dt, blocks, nb};
    blocks += nb;
    const DevTables &t = bp.ts[k].dev[0];
    if (bp.two) {
      BatchJob2 &bj = bp.jobs2[k];
      bj.p.a = batch_args(c, S, d.field);
      bj.p.a.ntz = d.ntz2;
      with_src2(bj.p, t, jobs[j].geom.wavelet, g, 0);
      with_rec_extract(bj.p.a, t, jobs[j].data, g->nt, 0);
      for (int q = 0; q < 4; ++q) bj.buf[q] = fields[k] + q * d.field * S;
    } else {
      BatchJob &bj = bp.jobs[k];
      bj.a = batch_args(c, S, d.field);
      with_src(bj.a, t, &jobs[j].geom, g, 0, 0);
      with_rec_extract(bj.a, t, jobs[j].data, g->nt, 0);
      bj.bufA = fields[k];
      bj.bufB = fields[k] + d.field * S;
    }
  }
  const void *host = bp.two ? (const void *)bp.jobs2.data() : (const void *)bp.jobs.data();
  const size_t dj = piece(jb_bytes / 4 * njobs);
  std::memcpy(blob.data() + dj, host, jb_bytes * njobs);
  const size_t dp = piece(sizeof(PrepJob) / 4 * njobs);
  std::memcpy(blob.data() + dp, prep.data(), sizeof(PrepJob) * njobs);
  // the job of every tile, so that a workgroup finds its job with one load
  if (bp.two) {
    const size_t tj = piece(bp.total);
    for (int k = 0; k < njobs; ++k)
      std::fill(blob.begin() + tj + bp.prefix[k], blob.begin() + tj + bp.prefix[k + 1], k);
    bp.dtile_job = dblob + tj;
  }
  if (blob.size() > blob_ints) return set_err(ctx, FWIME_EHIP, "batch tables exceed their scratch");
  HIPCHK(hipMemcpyAsync(dblob, blob.data(), blob.size() * sizeof(int), hipMemcpyHostToDevice, st));
  HIPCHK(launch_prep_multi(reinterpret_cast<PrepJob *>(dblob + dp), njobs, blocks, st));
  HIPCHK(hipStreamSynchronize(st));
  *djobs = dblob + dj;
  return FWIME_OK;
}

std::string batch_signature(int njobs, const fwime_job_t *jobs) {
  std::string sig;
  char buf[96];
  for (int j = 0; j < njobs; ++j) {
    std::snprintf(buf, sizeof buf, "%d,%d,%d,%d;", jobs[j].grid.nz + 2 * jobs[j].grid.nb,
                  jobs[j].grid.nx + 2 * jobs[j].grid.nb, jobs[j].geom.nshots, jobs[j].grid.nt > 1);
    sig += buf;
  }
  return sig;
}

// Times every tile width on the batch's first steps (receivers off) and
// keeps the context's width unless another is at least 2 % faster: the
// widths next to the best one are within a few per cent of it, and a choice
// made on noise would move the launch time from call to call.  Each width
// gets three timed windows of 8 launches; its time is the fastest window.
int batch_autotune(fwime_ctx_t *ctx, int njobs, const fwime_job_t *jobs, hipStream_t st, int *best_tx) {
  const int cand[5] = {16, 24, 32, 48, 64};
  float t_cand[5];
  *best_tx = ctx->tile_x;
  hipEvent_t e0, e1;
  HIPCHK(hipEventCreate(&e0));
  HIPCHK(hipEventCreate(&e1));
  int rc = FWIME_OK;
  for (int ci = 0; ci < 5; ++ci) {
    const int tx = cand[ci];
    t_cand[ci] = 1e30f;
    BatchPlan bp;
    void *dj = nullptr;
    int *dstep = nullptr;
    if ((rc = batch_plan(ctx, njobs, jobs, tx, bp, nullptr))) break;
    if ((rc = batch_carve_and_setup(ctx, njobs, jobs, bp, &dj, &dstep, st))) break;
    // scratch run: receivers off, time kept below every job's last step
    for (auto &jb : bp.jobs) jb.a.ext.ptr = nullptr;
    for (auto &jb : bp.jobs2) jb.p.a.ext.ptr = nullptr;
    const void *host = bp.two ? (const void *)bp.jobs2.data() : (const void *)bp.jobs.data();
    const size_t jb_bytes = bp.two ? sizeof(BatchJob2) : sizeof(BatchJob);
    if (hipMemcpyAsync(dj, host, jb_bytes * njobs, hipMemcpyHostToDevice, st) != hipSuccess ||
        launch_zero(reinterpret_cast<float *>(dstep), 1, st) != hipSuccess) {   // all-zero bits: int 0
      rc = set_err(ctx, FWIME_EHIP, "autotune setup failed");
      break;
    }
    const int warm = 2, timed = 8, windows = 3;
    for (int i = 0; i < warm && rc == FWIME_OK; ++i)
      if (batch_launch(bp, dj, bp.total, dstep, 0, tx, st) != hipSuccess)
        rc = set_err(ctx, FWIME_EHIP, "autotune launch failed");
    for (int wdw = 0; wdw < windows && rc == FWIME_OK; ++wdw) {
      (void)hipEventRecord(e0, st);
      for (int i = 0; i < timed && rc == FWIME_OK; ++i)
        if (batch_launch(bp, dj, bp.total, dstep, 0, tx, st) != hipSuccess)
          rc = set_err(ctx, FWIME_EHIP, "autotune launch failed");
      if (rc) break;
      (void)hipEventRecord(e1, st);
      if (hipEventSynchronize(e1) != hipSuccess) {
        rc = set_err(ctx, FWIME_EHIP, "autotune sync failed");
        break;
      }
      float ms = 0.f;
      (void)hipEventElapsedTime(&ms, e0, e1);
      t_cand[ci] = std::min(t_cand[ci], ms);
    }
    if (rc) break;
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (rc) return rc;
  float t_def = 1e30f, t_best = 1e30f;
  int tx_best = ctx->tile_x;
  for (int ci = 0; ci < 5; ++ci) {
    if (cand[ci] == ctx->tile_x) t_def = t_cand[ci];
    if (t_cand[ci] < t_best) {
      t_best = t_cand[ci];
      tx_best = cand[ci];
    }
  }
  *best_tx = t_best < 0.98f * t_def ? tx_best : ctx->tile_x;
  return FWIME_OK;
}

}  // namespace

extern "C" {

int fwime_model_batch(fwime_ctx_t *ctx, int32_t njobs, const fwime_job_t *jobs, void *stream) {
  if (!ctx) return FWIME_EINVAL;
  ctx->err.clear();
  hipStream_t st = (hipStream_t)stream;
  int rc;
  if (njobs < 1 || !jobs) return set_err(ctx, FWIME_EINVAL, "need njobs >= 1 and a job array");
  long nt_steps = 0;
  for (int j = 0; j < njobs; ++j) {
    if ((rc = check_grid(ctx, &jobs[j].grid)) || (rc = check_geom(ctx, &jobs[j].grid, &jobs[j].geom))) return rc;
    if (!jobs[j].data) return set_err(ctx, FWIME_EINVAL, "job data is null");
    nt_steps = std::max<long>(nt_steps, jobs[j].grid.nt);
  }
  HIPCHK(hipSetDevice(ctx->device));
  {
    // every job's velocity and wavelets in one device pass and one synchronization
    std::vector<std::pair<const float *, long>> arrays;
    for (int j = 0; j < njobs; ++j) {
      if (!jobs[j].vel) return set_err(ctx, FWIME_EINVAL, "job velocity is null");
      arrays.push_back({jobs[j].vel, (long)jobs[j].grid.nx * jobs[j].grid.nz});
      arrays.push_back({jobs[j].geom.wavelet, (long)jobs[j].geom.nshots * jobs[j].grid.nt});
    }
    std::vector<double> r;
    if ((rc = device_ranges(ctx, arrays, st, r))) return rc;
    for (int j = 0; j < njobs; ++j) {
      if ((rc = check_velocity_range(ctx, &jobs[j].grid, &r[6 * j]))) return rc;
      if (r[6 * j + 5] > 0) return set_err(ctx, FWIME_ENONFINITE, "input array has non-finite values");
    }
  }
  release_graph(ctx);   // the input checks synchronized the stream: earlier replays are done

  const std::string sig = batch_signature(njobs, jobs);
  int tx = ctx->tile_x;
  if (!std::getenv("FWIME_TILE_X")) {
    auto it = ctx->tuned.find(sig);
    if (it != ctx->tuned.end()) {
      tx = it->second;
    } else {
      if ((rc = batch_autotune(ctx, njobs, jobs, st, &tx))) return rc;
      ctx->tuned[sig] = tx;
    }
  }
  ctx->last_batch_tile = tx;

  BatchPlan bp;
  void *dj = nullptr;
  int *dstep = nullptr;
  if ((rc = batch_plan(ctx, njobs, jobs, tx, bp, nullptr))) return rc;
  if ((rc = batch_carve_and_setup(ctx, njobs, jobs, bp, &dj, &dstep, st))) return rc;
  HIPCHK(launch_zero(reinterpret_cast<float *>(dstep), 1, st));   // all-zero bits: int 0

  const int G = ctx->graph_steps;
  // Large batches: one direct launch per step over the still-running jobs
  // only (launch latency is negligible next to the step).  Small batches:
  // replay a captured graph of G full-width steps (idle jobs exit at once).
  const bool use_graph = !std::getenv("FWIME_NO_GRAPH") && bp.total <= kGraphMaxTiles;
  const long L = bp.launches();
  if (!use_graph) {
    HIPCHK(timing_begin(ctx, st));
    for (long i = 0; i < L; ++i)
      HIPCHK(batch_launch(bp, dj, batch_active_tiles(bp, i * bp.stride()), nullptr, (int)(i * bp.stride()), tx, st));
    HIPCHK(timing_end(ctx, st, L));
    return FWIME_OK;
  }
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
  // the capture stream is made on first use: contexts that never capture
  // (one per serving slot, say) do not take a hardware queue for it
  if (!ctx->capture) HIPCHK(hipStreamCreateWithFlags(&ctx->capture, hipStreamNonBlocking));
  HIPCHK(hipStreamBeginCapture(ctx->capture, hipStreamCaptureModeRelaxed));
  hipError_t cap = hipSuccess;
  for (int i = 0; i < G && cap == hipSuccess; ++i) cap = batch_launch(bp, dj, bp.total, dstep, 0, tx, ctx->capture);
  hipError_t endc = hipStreamEndCapture(ctx->capture, &graph);
  if (cap != hipSuccess || endc != hipSuccess) {
    if (graph) (void)hipGraphDestroy(graph);
    return set_err(ctx, FWIME_EHIP, "graph capture failed");
  }
  if (hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0) != hipSuccess) {
    (void)hipGraphDestroy(graph);
    return set_err(ctx, FWIME_EHIP, "graph instantiation failed");
  }
  const long replays = (L + G - 1) / G;
  HIPCHK(timing_begin(ctx, st));
  hipError_t le = hipSuccess;
  for (long r = 0; r < replays && le == hipSuccess; ++r) le = hipGraphLaunch(exec, st);
  if (le == hipSuccess) HIPCHK(timing_end(ctx, st, replays * G));
  ctx->graph = graph;          // kept until the replays have certainly finished
  ctx->graph_exec = exec;
  if (le != hipSuccess) return set_err(ctx, FWIME_EHIP, "graph launch failed");
  return FWIME_OK;
}

int fwime_footprint(const fwime_grid_t *g, int32_t nshots, int32_t nrec, int32_t nh, int32_t op, size_t *bytes) {
  if (!g || !bytes || nshots < 1 || nrec < 1 || nh < 1 || g->nt < 2) return FWIME_EINVAL;
  const Dims d = make_dims(g, 32);
  const long fb = d.field * 4;
  const long img = (long)nh * d.nx * d.nz * 4;
  const long nrt = (long)nrec * g->nt * 4;
  const GradPlan pl = grad_plan(d, g->nt);
  long per_shot = 0, fixed = fb + (long)(d.NX + d.LZ) * 4;
  // field buffers of the two-step path (the larger of the two paths)
  switch (op) {
    case FWIME_OP_MODEL: per_shot = 4 * fb; break;
    case FWIME_OP_BORN_FWD: per_shot = (8 + 2 * 16 + 4) * fb; fixed += img; break;
    case FWIME_OP_BORN_ADJ:
      per_shot = (4 + 2L * pl.nseg + pl.K + pl.R + 2 + (pl.R + 1) / 2 + pl.nseg) * fb;
      fixed += (2 + kImageGroups) * img;          // FP64 accumulator and partial images
      break;
    case FWIME_OP_GRADIENT:
      per_shot = grad_work_per_shot(d, pl, true) + 2 * pl.ck_stride * 4 + 2 * nrt;
      fixed += (5 + kImageGroups) * img;
      break;
    default: return FWIME_EINVAL;
  }
  *bytes = (size_t)(fixed + per_shot * nshots + (long)nrec * nshots * 64);
  return FWIME_OK;
}

}  // extern "C"

// ---------------------------------------------------------------------------
// Continuous batching of modeling jobs (the request loop's engine).
//
// Jobs join a running multi-job time loop at the next round boundary and
// leave it when their last sample is recorded.  A round advances every
// active job by the same number of time steps in shared two-step launches
// (k_step2_multi, one launch per two steps over the tiles of all active
// jobs); a job's time index is the global step minus the step at which it
// joined, so jobs of different lengths and arrival times share launches.
// Per-job device memory (padded velocity, tapers, geometry tables, four
// wavefield buffers per shot) is allocated stream-ordered on the engine's
// stream when the job is submitted and freed the same way once its last
// round has completed; the job descriptors of a round go to one slot of a
// small device ring, reused only after that round's event has completed.
// ---------------------------------------------------------------------------
namespace {

struct EngineJob {
  int64_t ticket = 0;
  fwime_grid_t grid{};
  fwime_geom_t geom{};
  std::vector<int32_t> src_iz, src_ix, rec_iz, rec_ix;   // host copies of the geometry
  Common com;
  TableSet ts;
  void *mem = nullptr;
  BatchJob2 desc;
  int tiles = 0;
  long t0 = -1;            // global step at which the job's time index is 0
};

constexpr int kEngineRing = 4;

}  // namespace

struct fwime_engine {
  fwime_ctx_t *ctx = nullptr;
  hipStream_t st = nullptr;              // the engine's stream (all of its work)
  int steps = 64;                        // time steps per round (even)
  int max_jobs = 0;
  long step = 0;                         // global step counter
  int64_t next_ticket = 1;
  std::vector<EngineJob *> pending, active;
  std::vector<std::pair<EngineJob *, hipEvent_t>> finishing;
  std::vector<hipEvent_t> free_events;
  BatchJob2 *host_desc[kEngineRing] = {};
  BatchJob2 *dev_desc[kEngineRing] = {};
  hipEvent_t ring_ev[kEngineRing] = {};
  bool ring_used[kEngineRing] = {};
  int ring_i = 0;
  long rounds = 0;
  long launches = 0;
};

namespace {

void engine_release_job(fwime_engine_t *e, EngineJob *j) {
  if (j->mem) (void)hipFreeAsync(j->mem, e->st);
  delete j;
}

hipError_t engine_event(fwime_engine_t *e, hipEvent_t *ev) {
  if (!e->free_events.empty()) {
    *ev = e->free_events.back();
    e->free_events.pop_back();
    return hipSuccess;
  }
  return hipEventCreateWithFlags(ev, hipEventDisableTiming);
}

}  // namespace

extern "C" {

int fwime_engine_create(fwime_ctx_t *ctx, int32_t steps_per_round, int32_t max_jobs, void *stream,
                        fwime_engine_t **out) {
  if (!ctx || !out) return FWIME_EINVAL;
  *out = nullptr;
  if (steps_per_round < 2 || steps_per_round % 2 || max_jobs < 1)
    return set_err(ctx, FWIME_EINVAL, "steps_per_round must be even and >= 2, max_jobs >= 1");
  HIPCHK(hipSetDevice(ctx->device));
  fwime_engine_t *e = new fwime_engine_t();
  e->ctx = ctx;
  e->st = (hipStream_t)stream;
  e->steps = steps_per_round;
  e->max_jobs = max_jobs;
  const size_t bytes = sizeof(BatchJob2) * (size_t)max_jobs;
  for (int i = 0; i < kEngineRing; ++i) {
    if (hipHostMalloc((void **)&e->host_desc[i], bytes, hipHostMallocDefault) != hipSuccess ||
        device_alloc(ctx, (void **)&e->dev_desc[i], bytes) != hipSuccess ||
        hipEventCreateWithFlags(&e->ring_ev[i], hipEventDisableTiming) != hipSuccess) {
      (void)hipGetLastError();
      fwime_engine_destroy(e);
      return set_err(ctx, FWIME_ENOMEM, "engine descriptor ring allocation failed");
    }
  }
  *out = e;
  return FWIME_OK;
}

int fwime_engine_submit(fwime_engine_t *e, const fwime_job_t *job, void *check_stream, int64_t *ticket) {
  if (!e || !job || !ticket) return FWIME_EINVAL;
  fwime_ctx_t *ctx = e->ctx;
  ctx->err.clear();
  int rc;
  if ((rc = check_grid(ctx, &job->grid)) || (rc = check_geom(ctx, &job->grid, &job->geom))) return rc;
  if (!job->data || !job->vel) return set_err(ctx, FWIME_EINVAL, "job data or velocity is null");
  if ((long)e->pending.size() + (long)e->active.size() >= e->max_jobs)
    return set_err(ctx, FWIME_ENOMEM, "the engine holds max_jobs jobs already");
  HIPCHK(hipSetDevice(ctx->device));
  {
    // velocity range and finite wavelets, on the stream that produced them
    std::vector<double> r;
    hipStream_t cs = (hipStream_t)check_stream;
    if ((rc = device_ranges(ctx, {{job->vel, (long)job->grid.nx * job->grid.nz},
                                  {job->geom.wavelet, (long)job->geom.nshots * job->grid.nt}}, cs, r)))
      return rc;
    if ((rc = check_velocity_range(ctx, &job->grid, r.data()))) return rc;
    if (r[5] > 0) return set_err(ctx, FWIME_ENONFINITE, "input array has non-finite values");
  }
  EngineJob *j = new EngineJob();
  j->grid = job->grid;
  j->geom = job->geom;
  const long ns = job->geom.nshots, nr = (long)job->geom.nshots * job->geom.nrec;
  j->src_iz.assign(job->geom.src_iz, job->geom.src_iz + ns);
  j->src_ix.assign(job->geom.src_ix, job->geom.src_ix + ns);
  j->rec_iz.assign(job->geom.rec_iz, job->geom.rec_iz + nr);
  j->rec_ix.assign(job->geom.rec_ix, job->geom.rec_ix + nr);
  j->geom.src_iz = j->src_iz.data();
  j->geom.src_ix = j->src_ix.data();
  j->geom.rec_iz = j->rec_iz.data();
  j->geom.rec_ix = j->rec_ix.data();
  Common &c = j->com;
  c.d = make_dims(&j->grid, ctx->tile_x);
  const Dims &d = c.d;
  const int S = (int)ns;
  j->ts = build_table_set(d, &j->geom, {{0, S}}, true);
  float *fields = nullptr;
  Carve cv;
  cv.add(&c.V, d.field);
  cv.add(&c.gz, d.LZ);
  cv.add(&c.gx, d.NX + kGxPad);
  cv.add(&c.tables, table_set_ints(j->ts) + 64 * 8);
  cv.add(&fields, 4 * d.field * S);
  if (ctx->budget && cv.total > ctx->budget) {
    delete j;
    return set_err(ctx, FWIME_ENOMEM, "the job exceeds the HBM budget");
  }
  hipError_t alloc = hipMallocAsync(&j->mem, cv.total, e->st);
  if (alloc != hipSuccess) {               // as device_alloc
    (void)hipGetLastError();
    release_idle(ctx, nullptr);
    alloc = hipMallocAsync(&j->mem, cv.total, e->st);
  }
  if (alloc != hipSuccess) {
    (void)hipGetLastError();
    delete j;
    return set_err(ctx, FWIME_ENOMEM, "hipMallocAsync of " + std::to_string(cv.total) + " bytes failed");
  }
  cv.assign(j->mem);
  // the blob stays alive in the job until it is released, after the copy
  if ((rc = upload_tables(ctx, j->ts, c.tables, e->st, false)) || (rc = setup_common(ctx, c, &j->grid, job->vel, e->st)) ||
      (launch_zero(fields, 4 * d.field * S, e->st) != hipSuccess ? (rc = FWIME_EHIP) : 0)) {
    engine_release_job(e, j);
    return rc ? rc : set_err(ctx, FWIME_EHIP, "engine job setup failed");
  }
  const DevTables &t = j->ts.dev[0];
  BatchJob2 &bj = j->desc;
  bj.p.a = batch_args(c, S, d.field);
  bj.p.a.ntz = d.ntz2;
  with_src2(bj.p, t, job->geom.wavelet, &j->grid, 0);
  with_rec_extract(bj.p.a, t, job->data, j->grid.nt, 0);
  for (int q = 0; q < 4; ++q) bj.buf[q] = fields + q * d.field * S;
  bj.nt = j->grid.nt;
  j->tiles = d.ntz2 * d.ntx * S;
  j->ticket = e->next_ticket++;
  e->pending.push_back(j);
  *ticket = j->ticket;
  return FWIME_OK;
}

int fwime_engine_run(fwime_engine_t *e) {
  if (!e) return FWIME_EINVAL;
  fwime_ctx_t *ctx = e->ctx;
  ctx->err.clear();
  HIPCHK(hipSetDevice(ctx->device));
  // jobs join at this round's boundary
  for (EngineJob *j : e->pending) {
    j->t0 = e->step;
    j->desc.t0 = (int)e->step;
    e->active.push_back(j);
  }
  e->pending.clear();
  if (e->active.empty()) return FWIME_OK;
  // descriptor slot of this round: free once the round that used it last is done
  const int i = e->ring_i;
  if (e->ring_used[i]) HIPCHK(hipEventSynchronize(e->ring_ev[i]));
  int total = 0;
  bool fs = false;
  const int nj = (int)e->active.size();
  for (int k = 0; k < nj; ++k) {
    EngineJob *j = e->active[k];
    j->desc.tile_begin = total;
    total += j->tiles;
    fs = fs || j->grid.free_surface != 0;
    e->host_desc[i][k] = j->desc;
  }
  HIPCHK(hipMemcpyAsync(e->dev_desc[i], e->host_desc[i], sizeof(BatchJob2) * nj, hipMemcpyHostToDevice, e->st));
  const int L = e->steps / 2;
  for (int l = 0; l < L; ++l)
    HIPCHK(launch_step2_multi(e->dev_desc[i], nullptr, nj, total, nullptr, (int)(e->step + 2L * l), ctx->tile_x, fs,
                              e->st));
  HIPCHK(hipEventRecord(e->ring_ev[i], e->st));
  e->ring_used[i] = true;
  e->ring_i = (i + 1) % kEngineRing;
  e->step += e->steps;
  e->rounds += 1;
  e->launches += L;
  // jobs whose last sample (time index nt - 1) was recorded in this round leave
  std::vector<EngineJob *> keep;
  for (EngineJob *j : e->active) {
    // the last launch of the round ran time index e->step - 2 - t0; the job
    // recorded its last sample once that index reached nt - 2 (two-step
    // launch) or nt - 1 (sample only): e->step - t0 >= nt, both being even
    if (e->step - j->t0 >= (long)j->grid.nt) {
      hipEvent_t ev;
      HIPCHK(engine_event(e, &ev));
      HIPCHK(hipEventRecord(ev, e->st));
      e->finishing.push_back({j, ev});
    } else {
      keep.push_back(j);
    }
  }
  e->active.swap(keep);
  return FWIME_OK;
}

int fwime_engine_poll(fwime_engine_t *e, int64_t *tickets, int32_t cap, int32_t *ndone) {
  if (!e || !ndone || (cap > 0 && !tickets)) return FWIME_EINVAL;
  fwime_ctx_t *ctx = e->ctx;
  HIPCHK(hipSetDevice(ctx->device));
  int n = 0;
  std::vector<std::pair<EngineJob *, hipEvent_t>> keep;
  for (auto &f : e->finishing) {
    if (n < cap && hipEventQuery(f.second) == hipSuccess) {
      tickets[n++] = f.first->ticket;
      e->free_events.push_back(f.second);
      engine_release_job(e, f.first);
    } else {
      (void)hipGetLastError();
      keep.push_back(f);
    }
  }
  e->finishing.swap(keep);
  *ndone = n;
  return FWIME_OK;
}

int fwime_engine_info(const fwime_engine_t *e, fwime_engine_info_t *out) {
  if (!e || !out) return FWIME_EINVAL;
  out->pending = (int32_t)e->pending.size();
  out->active = (int32_t)e->active.size();
  out->finishing = (int32_t)e->finishing.size();
  out->step = e->step;
  out->rounds = e->rounds;
  out->launches = e->launches;
  return FWIME_OK;
}

void fwime_engine_destroy(fwime_engine_t *e) {
  if (!e) return;
  (void)hipSetDevice(e->ctx->device);
  if (e->st) (void)hipStreamSynchronize(e->st);
  for (EngineJob *j : e->pending) engine_release_job(e, j);
  for (EngineJob *j : e->active) engine_release_job(e, j);
  for (auto &f : e->finishing) {
    engine_release_job(e, f.first);
    (void)hipEventDestroy(f.second);
  }
  if (e->st) (void)hipStreamSynchronize(e->st);
  for (hipEvent_t ev : e->free_events) (void)hipEventDestroy(ev);
  for (int i = 0; i < kEngineRing; ++i) {
    if (e->host_desc[i]) (void)hipHostFree(e->host_desc[i]);
    if (e->dev_desc[i]) (void)hipFree(e->dev_desc[i]);
    if (e->ring_ev[i]) (void)hipEventDestroy(e->ring_ev[i]);
  }
  delete e;
}

}  // extern "C"

// ---------------------------------------------------------------------------
// Linear spline operator S and its adjoint (Section 2's spline grid)
// ---------------------------------------------------------------------------
namespace fw {
hipError_t launch_spline_tables(const double *nodes, int nn, const double *pts, int nf, double h, int *cell,
                                float *wt, int *start, hipStream_t st);
hipError_t launch_spline_apply(const float *mc, int nzn, const int *cz, const float *tz, const int *cx,
                               const float *tx, int nz, int nx, float *out, hipStream_t st);
hipError_t launch_spline_adjoint(const float *f, int nz, int nx, const float *tz, const int *sz, int nzn,
                                 const float *tx, const int *sx, int nxn, float *tmp, float *out, hipStream_t st);
}  // namespace fw

namespace {

struct SplineAxes {
  double *zn = nullptr, *xn = nullptr;
  int *cz = nullptr, *cx = nullptr, *sz = nullptr, *sx = nullptr;
  float *tz = nullptr, *tx = nullptr;
};

int check_spline_axis(fwime_ctx_t *ctx, const double *n, int32_t nn, int32_t nf, double h, const char *name) {
  const std::string nm(name);
  if (nn < 2) return set_err(ctx, FWIME_EINVAL, nm + ": at least two spline nodes are needed");
  if (nn > kSplineMaxNodes) return set_err(ctx, FWIME_EINVAL, nm + ": more than 2^24 spline nodes");
  if (nf < 1 || nf > (1 << 30)) return set_err(ctx, FWIME_EINVAL, nm + ": the grid needs 1 to 2^30 points");
  if (!(h > 0.0) || !std::isfinite(h)) return set_err(ctx, FWIME_EINVAL, nm + ": grid spacing must be positive");
  if (!n) return set_err(ctx, FWIME_EINVAL, nm + " node coordinates are null");
  for (int j = 0; j < nn; ++j)
    if (!std::isfinite(n[j])) return set_err(ctx, FWIME_EINVAL, nm + " node coordinates must be finite");
  for (int j = 1; j < nn; ++j)
    if (!(n[j] > n[j - 1])) return set_err(ctx, FWIME_EINVAL, nm + " node coordinates must be strictly increasing");
  const double tol = 1e-9 * std::max(1.0, std::fabs(n[nn - 1] - n[0]));
  if (n[0] > tol || (nf - 1) * h > n[nn - 1] + tol)
    return set_err(ctx, FWIME_EINVAL, nm + " nodes must cover every grid point");
  return FWIME_OK;
}

int check_spline(fwime_ctx_t *ctx, int32_t nz, int32_t nx, double dz, double dx, int32_t nzn, const double *zn,
                 int32_t nxn, const double *xn, const void *in, void *out) {
  int rc;
  if ((rc = check_spline_axis(ctx, zn, nzn, nz, dz, "z")) || (rc = check_spline_axis(ctx, xn, nxn, nx, dx, "x")))
    return rc;
  if (!in || !out) return set_err(ctx, FWIME_EINVAL, "input or output is null");
  HIPCHK(hipSetDevice(ctx->device));
  return FWIME_OK;
}

// Most fine points (of n, at multiples of h) in the two cells of any node.
double spline_span(const double *nodes, int32_t nn, int32_t n, double h) {
  double span = 0.0;
  for (int j = 0; j < nn; ++j)
    span = std::max(span, nodes[std::min(j + 1, nn - 1)] - nodes[std::max(j - 1, 0)]);
  return std::min((double)n, std::floor(span / h) + 1.0);
}

// Whether S and S* run as one launch: few enough nodes and rows for it, and
// for S* few enough fine points to a workgroup, which gathers the two cells of
// its node column: kSplineSerial values read by a thread one after the other.
// Measured, us, two passes against one launch, by that number: 60 (300 x 1700,
// 31 x 171 nodes) 53.5 / 13.8; 320 (31 x 28) 77 / 43; 384 (2000 x 2500, 33 x 251)
// 105 / 62; 640 (500 x 2500, 9 x 41) 83 / 79; 1080 (300 x 1700, 11 x 10) 123 / 122;
// 1200 (2000 x 2500, 11 x 85) 116 / 155; 2176 (33 x 41) 134 / 300; the largest
// (9 x 11) 209 / 1420.
constexpr double kSplineSerial = 512;
bool spline_one_launch(int32_t nz, int32_t nx, double dz, double dx, int32_t nzn, const double *zn, int32_t nxn,
                       const double *xn, bool adjoint, SplineNodes &s) {
  if ((long)nzn + nxn > kSplineNodes || nz > kSplineRows) return false;
  if (adjoint) {
    const double rounds = std::ceil(spline_span(xn, nxn, nx, dx) * nzn / 256);   // of 256 threads
    if (rounds * spline_span(zn, nzn, nz, dz) > kSplineSerial) return false;
  }
  s.nzn = nzn;
  s.nxn = nxn;
  std::copy(zn, zn + nzn, s.n);
  std::copy(xn, xn + nxn, s.n + nzn);
  return true;
}

// carves the tables (plus `extra` floats) from the arena, uploads the node
// coordinates and builds the per-axis tables on `st`
int spline_setup(fwime_ctx_t *ctx, int32_t nz, int32_t nx, double dz, double dx, int32_t nzn, const double *zn,
                 int32_t nxn, const double *xn, long extra, float **extra_ptr, SplineAxes &a, hipStream_t st) {
  int rc;
  HIPCHK(hipStreamSynchronize(st));      // earlier work on the stream may still use the arena
  Carve cv;
  cv.add(&a.zn, nzn);
  cv.add(&a.xn, nxn);
  cv.add(&a.cz, nz);
  cv.add(&a.cx, nx);
  cv.add(&a.tz, nz);
  cv.add(&a.tx, nx);
  cv.add(&a.sz, (long)nzn + 1);
  cv.add(&a.sx, (long)nxn + 1);
  if (extra > 0) cv.add(extra_ptr, extra);
  if ((rc = arena_get(ctx, cv))) return rc;
  // pageable sources are copied synchronously: nothing of the caller's is read later
  HIPCHK(hipMemcpyAsync(a.zn, zn, nzn * sizeof(double), hipMemcpyHostToDevice, st));
  HIPCHK(hipMemcpyAsync(a.xn, xn, nxn * sizeof(double), hipMemcpyHostToDevice, st));
  HIPCHK(hipStreamSynchronize(st));
  HIPCHK(launch_spline_tables(a.zn, nzn, nullptr, nz, dz, a.cz, a.tz, a.sz, st));
  HIPCHK(launch_spline_tables(a.xn, nxn, nullptr, nx, dx, a.cx, a.tx, a.sx, st));
  return FWIME_OK;
}

}  // namespace

extern "C" {

int fwime_spline_apply(fwime_ctx_t *ctx, int32_t nz, int32_t nx, double dz, double dx, int32_t nzn, const double *zn,
                       int32_t nxn, const double *xn, const float *mc, float *out, void *stream) {
  if (!ctx) return FWIME_EINVAL;
  ctx->err.clear();
  hipStream_t st = (hipStream_t)stream;
  int rc = check_spline(ctx, nz, nx, dz, dx, nzn, zn, nxn, xn, mc, out);
  if (rc) return rc;
  SplineNodes nodes;
  if (spline_one_launch(nz, nx, dz, dx, nzn, zn, nxn, xn, false, nodes)) {
    HIPCHK(launch_spline_apply1(nodes, nz, nx, dz, dx, mc, out, st));
    return FWIME_OK;
  }
  SplineAxes a;
  if ((rc = spline_setup(ctx, nz, nx, dz, dx, nzn, zn, nxn, xn, 0, nullptr, a, st))) return rc;
  HIPCHK(launch_spline_apply(mc, nzn, a.cz, a.tz, a.cx, a.tx, nz, nx, out, st));
  return FWIME_OK;
}

int fwime_spline_adjoint(fwime_ctx_t *ctx, int32_t nz, int32_t nx, double dz, double dx, int32_t nzn,
                         const double *zn, int32_t nxn, const double *xn, const float *f, float *mc_out,
                         void *stream) {
  if (!ctx) return FWIME_EINVAL;
  ctx->err.clear();
  hipStream_t st = (hipStream_t)stream;
  int rc = check_spline(ctx, nz, nx, dz, dx, nzn, zn, nxn, xn, f, mc_out);
  if (rc) return rc;
  SplineNodes nodes;
  if (spline_one_launch(nz, nx, dz, dx, nzn, zn, nxn, xn, true, nodes)) {
    HIPCHK(launch_spline_adjoint1(nodes, nz, nx, dz, dx, f, mc_out, st));
    return FWIME_OK;
  }
  SplineAxes a;
  float *tmp = nullptr;
  if ((rc = spline_setup(ctx, nz, nx, dz, dx, nzn, zn, nxn, xn, (long)nx * nzn, &tmp, a, st))) return rc;
  HIPCHK(launch_spline_adjoint(f, nz, nx, a.tz, a.sz, nzn, a.tx, a.sx, nxn, tmp, mc_out, st));
  return FWIME_OK;
}

int fwime_spline_refine(fwime_ctx_t *ctx, int32_t nzn, const double *zn, int32_t nxn, const double *xn,
                        const float *mc, int32_t nzf, const double *zf, int32_t nxf, const double *xf,
                        float *mf_out, void *stream) {
  if (!ctx) return FWIME_EINVAL;
  ctx->err.clear();
  hipStream_t st = (hipStream_t)stream;
  // the new nodes: strictly increasing, inside the old nodes' span
  auto targets = [&](const double *t, int32_t nt_, const double *n, int32_t nn, const char *name) -> int {
    const std::string nm(name);
    if (nt_ < 1 || nt_ > kSplineMaxNodes) return set_err(ctx, FWIME_EINVAL, nm + ": 1 to 2^24 new nodes");
    if (!t) return set_err(ctx, FWIME_EINVAL, nm + " new node coordinates are null");
    for (int j = 0; j < nt_; ++j)
      if (!std::isfinite(t[j]) || (j > 0 && !(t[j] > t[j - 1])))
        return set_err(ctx, FWIME_EINVAL, nm + " new node coordinates must be finite and strictly increasing");
    if (nn >= 2 && n) {
      const double tol = 1e-9 * std::max(1.0, std::fabs(n[nn - 1] - n[0]));
      if (t[0] < n[0] - tol || t[nt_ - 1] > n[nn - 1] + tol)
        return set_err(ctx, FWIME_EINVAL, nm + " new nodes must lie within the old nodes");
    }
    return FWIME_OK;
  };
  int rc;
  if ((rc = check_spline_axis(ctx, zn, nzn, 1, 1.0, "z")) || (rc = check_spline_axis(ctx, xn, nxn, 1, 1.0, "x")) ||
      (rc = targets(zf, nzf, zn, nzn, "z")) || (rc = targets(xf, nxf, xn, nxn, "x")))
    return rc;
  if (!mc || !mf_out) return set_err(ctx, FWIME_EINVAL, "input or output is null");
  HIPCHK(hipSetDevice(ctx->device));
  HIPCHK(hipStreamSynchronize(st));      // earlier work on the stream may still use the arena
  SplineAxes a;
  double *zt = nullptr, *xt = nullptr;
  Carve cv;
  cv.add(&a.zn, nzn);
  cv.add(&a.xn, nxn);
  cv.add(&zt, nzf);
  cv.add(&xt, nxf);
  cv.add(&a.cz, nzf);
  cv.add(&a.cx, nxf);
  cv.add(&a.tz, nzf);
  cv.add(&a.tx, nxf);
  cv.add(&a.sz, (long)nzn + 1);
  cv.add(&a.sx, (long)nxn + 1);
  if ((rc = arena_get(ctx, cv))) return rc;
  HIPCHK(hipMemcpyAsync(a.zn, zn, nzn * sizeof(double), hipMemcpyHostToDevice, st));
  HIPCHK(hipMemcpyAsync(a.xn, xn, nxn * sizeof(double), hipMemcpyHostToDevice, st));
  HIPCHK(hipMemcpyAsync(zt, zf, nzf * sizeof(double), hipMemcpyHostToDevice, st));
  HIPCHK(hipMemcpyAsync(xt, xf, nxf * sizeof(double), hipMemcpyHostToDevice, st));
  HIPCHK(hipStreamSynchronize(st));
  HIPCHK(launch_spline_tables(a.zn, nzn, zt, nzf, 0.0, a.cz, a.tz, a.sz, st));
  HIPCHK(launch_spline_tables(a.xn, nxn, xt, nxf, 0.0, a.cx, a.tx, a.sx, st));
  HIPCHK(launch_spline_apply(mc, nzn, a.cz, a.tz, a.cx, a.tx, nzf, nxf, mf_out, st));
  return FWIME_OK;
}

}  // extern "C"

// ---------------------------------------------------------------------------
// L-BFGS search direction (Section 3: the outer minimization uses L-BFGS)
// ---------------------------------------------------------------------------
namespace fw {
hipError_t launch_axpby(const float *x, float a, float *y, float b, long n, hipStream_t st);
}  // namespace fw

namespace {

constexpr int kLbfgsMaxEvals = 100;      // trial steps per line search
constexpr long kLbfgsWorkHead = 4096;    // floats of the workspace before the vectors (dot partials)

// Whether k pairs of n elements go by inner products (gram_direction) rather
// than by the recursion on the vectors (two_loop).  Inner products save its
// 3 k + 1 round trips of about 20 us, but read the vectors from few workgroups
// (their partial sums go to the host) and their number grows with k squared.
// Measured, us, recursion against inner products: n = 1e6, k = 1 106 / 65, 5 356 /
// 116, 15 992 / 269; n = 3e6, k = 1 119 / 119; n = 4e6, k = 1 130 / 148, 2 213 / 152;
// n = 5e6, k = 5 510 / 452, 15 1592 / 1433; n = 3.1e7, k = 5 1936 / 2773, 15 5460 /
// 8750: the lines cross at 3e6 for one pair and between 6e6 and 1.1e7 for more.
bool by_inner_products(long k, long n) {
  return k <= kLbfgsGramPairs && n <= (k == 0 ? LONG_MAX : k == 1 ? 3000000L : 6000000L);
}

// d = -H g from the inner products of the pairs (oldest first) and g, at most
// kLbfgsGramPairs of them: the same recursion as two_loop below, on numbers.
// With q = g - sum_j alpha_j y_j and r = gamma q + sum_j (alpha_j - beta_j) s_j
// written out, alpha_i = rho_i s_i.q and beta_i = rho_i y_i.r need s_i.y_j,
// y_i.y_j, s_i.g and y_i.g only.  One synchronization; every pair's curvature
// is checked before d is written.
int gram_direction(fwime_ctx_t *ctx, long n, const std::vector<const float *> &S, const std::vector<const float *> &Y,
                   const float *g, float *d, hipStream_t st) {
  const int k = (int)S.size();
  LbfgsVectors v;
  std::copy(S.begin(), S.end(), v.s);
  std::copy(Y.begin(), Y.end(), v.y);
  v.g = g;
  v.k = k;
  LbfgsCoefs c;
  c.g = -1.0;
  if (k > 0) {
    const int nb = lbfgs_gram_blocks(k, n), groups = (2 * k + 3) / 4;
    int rc = host_red_reserve(ctx, (size_t)nb * groups * 64);
    if (rc) return rc;
    HIPCHK(launch_lbfgs_gram(v, n, ctx->host_red, st));
    HIPCHK(hipStreamSynchronize(st));
    std::vector<double> dot((size_t)groups * 64, 0.0);     // [row][16]
    for (int gr = 0; gr < groups; ++gr)
      for (int b = 0; b < nb; ++b)
        for (int q = 0; q < 64; ++q) dot[gr * 64 + q] += ctx->host_red[((size_t)gr * nb + b) * 64 + q];
    auto sy = [&](int i, int j) { return dot[i * 16 + j]; };         // s_i . y_j, j = k: s_i . g
    auto yy = [&](int i, int j) { return dot[(k + i) * 16 + j]; };   // y_i . y_j, j = k: y_i . g
    for (int i = 0; i < k; ++i)
      if (!(sy(i, i) > 0.0) || !std::isfinite(sy(i, i)))
        return set_err(ctx, FWIME_EINVAL, "pair " + std::to_string(i) + " has s.y <= 0 or non-finite");
    const double gamma = sy(k - 1, k - 1) / yy(k - 1, k - 1);
    std::vector<double> alpha(k), diff(k);
    for (int i = k - 1; i >= 0; --i) {
      double sq = sy(i, k);
      for (int j = k - 1; j > i; --j) sq -= alpha[j] * sy(i, j);
      alpha[i] = sq / sy(i, i);
    }
    for (int i = 0; i < k; ++i) {
      double yr = yy(i, k);
      for (int j = 0; j < k; ++j) yr -= alpha[j] * yy(i, j);
      yr *= gamma;
      for (int j = 0; j < i; ++j) yr += diff[j] * sy(j, i);
      diff[i] = alpha[i] - yr / sy(i, i);
    }
    c.g = -gamma;
    for (int i = 0; i < k; ++i) {
      c.s[i] = -diff[i];
      c.y[i] = gamma * alpha[i];
    }
  }
  HIPCHK(launch_lbfgs_combine(v, c, n, d, st));
  return FWIME_OK;
}

// d = -H g by the two-loop recursion over the pairs S[i], Y[i] (oldest first),
// H_0 = (s.y / y.y of the newest pair) I; FP64 inner products, FP32 updates.
// Every pair's curvature is checked before d is written.
int two_loop(fwime_ctx_t *ctx, long n, const std::vector<const float *> &S, const std::vector<const float *> &Y,
             const float *g, float *d, double *part, double *res, hipStream_t st) {
  const int k = (int)S.size();
  int rc;
  auto dot = [&](const float *a, const float *b, double &out) -> int {
    HIPCHK(launch_dot(a, b, n, part, res, st));
    HIPCHK(hipMemcpyAsync(ctx->host_red, res, sizeof(double), hipMemcpyDeviceToHost, st));
    HIPCHK(hipStreamSynchronize(st));
    out = ctx->host_red[0];
    return FWIME_OK;
  };
  std::vector<double> rho(k), alpha(k);
  double sy = 0.0, yy = 1.0;
  for (int i = 0; i < k; ++i) {
    if ((rc = dot(S[i], Y[i], sy))) return rc;
    if (!(sy > 0.0) || !std::isfinite(sy))
      return set_err(ctx, FWIME_EINVAL, "pair " + std::to_string(i) + " has s.y <= 0 or non-finite");
    rho[i] = 1.0 / sy;
  }
  double gamma = 1.0;
  if (k > 0) {
    if ((rc = dot(Y[k - 1], Y[k - 1], yy))) return rc;
    gamma = (1.0 / rho[k - 1]) / yy;
  }
  if (d != g) HIPCHK(hipMemcpyAsync(d, g, (size_t)n * sizeof(float), hipMemcpyDeviceToDevice, st));
  for (int i = k - 1; i >= 0; --i) {
    double sq;
    if ((rc = dot(S[i], d, sq))) return rc;
    alpha[i] = rho[i] * sq;
    HIPCHK(launch_axpby(Y[i], (float)-alpha[i], d, 1.0f, n, st));
  }
  HIPCHK(launch_axpby(d, 0.0f, d, (float)gamma, n, st));
  for (int i = 0; i < k; ++i) {
    double yr;
    if ((rc = dot(Y[i], d, yr))) return rc;
    HIPCHK(launch_axpby(S[i], (float)(alpha[i] - rho[i] * yr), d, 1.0f, n, st));
  }
  HIPCHK(launch_axpby(d, 0.0f, d, -1.0f, n, st));
  return FWIME_OK;
}

}  // namespace

extern "C" {

int fwime_lbfgs_direction(fwime_ctx_t *ctx, int64_t n, int32_t npairs, const float *s, const float *y,
                          const float *g, float *d_out, void *stream) {
  if (!ctx) return FWIME_EINVAL;
  ctx->err.clear();
  hipStream_t st = (hipStream_t)stream;
  if (n < 1) return set_err(ctx, FWIME_EINVAL, "n must be >= 1");
  if (npairs < 0 || npairs > kLbfgsMaxPairs)
    return set_err(ctx, FWIME_EINVAL, "npairs must be in [0, " + std::to_string(kLbfgsMaxPairs) + "]");
  if (!g || !d_out || (npairs > 0 && (!s || !y))) return set_err(ctx, FWIME_EINVAL, "null vector");
  HIPCHK(hipSetDevice(ctx->device));
  std::vector<const float *> S(npairs), Y(npairs);
  for (int i = 0; i < npairs; ++i) {
    S[i] = s + (long)i * n;
    Y[i] = y + (long)i * n;
  }
  if (by_inner_products(npairs, (long)n)) return gram_direction(ctx, (long)n, S, Y, g, d_out, st);
  HIPCHK(hipStreamSynchronize(st));      // earlier work on the stream may still use the arena
  double *part = nullptr, *res = nullptr;
  Carve cv;
  cv.add(&part, dot_partials());
  cv.add(&res, 1);
  int rc;
  if ((rc = arena_get(ctx, cv))) return rc;
  return two_loop(ctx, (long)n, S, Y, g, d_out, part, res, st);
}

int fwime_lbfgs_minimize(fwime_ctx_t *ctx, int64_t n, int32_t memory, int32_t maxiter, double gtol,
                         fwime_objective_fn fg, void *user, float *x, float *work, int64_t work_floats,
                         double *f_hist, int32_t *iters, void *stream) {
  if (!ctx) return FWIME_EINVAL;
  ctx->err.clear();
  hipStream_t st = (hipStream_t)stream;
  if (n < 1) return set_err(ctx, FWIME_EINVAL, "n must be >= 1");
  if (memory < 1 || memory > kLbfgsMaxPairs)
    return set_err(ctx, FWIME_EINVAL, "memory must be in [1, " + std::to_string(kLbfgsMaxPairs) + "]");
  if (maxiter < 0) return set_err(ctx, FWIME_EINVAL, "maxiter must be >= 0");
  if (!(gtol >= 0.0) || !std::isfinite(gtol)) return set_err(ctx, FWIME_EINVAL, "gtol must be finite and >= 0");
  if (!fg || !x || !work || !f_hist || !iters) return set_err(ctx, FWIME_EINVAL, "null argument");
  if ((reinterpret_cast<uintptr_t>(work) & 7) != 0) return set_err(ctx, FWIME_EINVAL, "work must be 8-byte aligned");
  if (n > (int64_t(1) << 40) || work_floats < kLbfgsWorkHead + (2 * (int64_t)memory + 6) * n)
    return set_err(ctx, FWIME_EINVAL, "work needs 4096 + (2 memory + 6) n floats");
  HIPCHK(hipSetDevice(ctx->device));
  // work: dot partials, then g, d, trial x, trial g and memory + 1 slots each of s and y
  double *part = (double *)work, *res = part + dot_partials();
  float *vec = work + kLbfgsWorkHead;
  auto V = [&](long j) { return vec + j * (long)n; };
  float *g = V(0), *d = V(1), *xt = V(2), *gt = V(3);
  std::vector<float *> sslot(memory + 1), yslot(memory + 1);
  for (int j = 0; j <= memory; ++j) {
    sslot[j] = V(4 + j);
    yslot[j] = V(5 + memory + j);
  }
  int rc;
  auto dot = [&](const float *a, const float *b, double &out) -> int {
    HIPCHK(launch_dot(a, b, (long)n, part, res, st));
    HIPCHK(hipMemcpyAsync(ctx->host_red, res, sizeof(double), hipMemcpyDeviceToHost, st));
    HIPCHK(hipStreamSynchronize(st));
    out = ctx->host_red[0];
    return FWIME_OK;
  };
  auto eval = [&](const float *at, float *grad, double &f) -> int {
    const int cb = fg(user, at, grad, &f);
    if (cb != 0) return set_err(ctx, FWIME_EINVAL, "objective callback returned " + std::to_string(cb));
    if (!std::isfinite(f)) return set_err(ctx, FWIME_ENONFINITE, "objective is not finite");
    return FWIME_OK;
  };
  double f = 0.0, gg = 0.0;
  if ((rc = eval(x, g, f)) || (rc = dot(g, g, gg))) return rc;
  const double g0 = std::sqrt(gg);
  f_hist[0] = f;
  // pairs kept oldest first, as slot indices; one slot is always free
  std::vector<int> pairs, free_slots;
  for (int j = memory; j >= 0; --j) free_slots.push_back(j);
  int it = 0;
  for (; it < maxiter; ++it) {
    if (std::sqrt(gg) <= gtol * g0) break;
    std::vector<const float *> S, Y;
    for (int j : pairs) {
      S.push_back(sslot[j]);
      Y.push_back(yslot[j]);
    }
    // descent direction -H g
    if ((rc = by_inner_products((long)S.size(), (long)n) ? gram_direction(ctx, (long)n, S, Y, g, d, st)
                                               : two_loop(ctx, (long)n, S, Y, g, d, part, res, st)))
      return rc;
    double dphi0;
    if ((rc = dot(g, d, dphi0))) return rc;
    if (!(dphi0 < 0.0)) break;
    MoreThuente ls;
    ls.stpmin = 0.0;
    ls.stpmax = 1e10;
    auto status = ls.start(1.0, f, dphi0);
    double ft = 0.0;
    for (int nfev = 0; status == MoreThuente::kEvaluate && nfev < kLbfgsMaxEvals; ++nfev) {
      HIPCHK(hipMemcpyAsync(xt, x, (size_t)n * sizeof(float), hipMemcpyDeviceToDevice, st));
      HIPCHK(launch_axpby(d, (float)ls.stp, xt, 1.0f, (long)n, st));
      double dphi;
      if ((rc = eval(xt, gt, ft)) || (rc = dot(gt, d, dphi))) return rc;
      status = ls.next(ft, dphi);
    }
    if (status != MoreThuente::kConverged) break;
    // new pair: s = x_t - x, y = g_t - g, kept if its curvature is positive
    const int slot = free_slots.back();
    float *sn = sslot[slot], *yn = yslot[slot];
    HIPCHK(hipMemcpyAsync(sn, xt, (size_t)n * sizeof(float), hipMemcpyDeviceToDevice, st));
    HIPCHK(launch_axpby(x, -1.0f, sn, 1.0f, (long)n, st));
    HIPCHK(hipMemcpyAsync(yn, gt, (size_t)n * sizeof(float), hipMemcpyDeviceToDevice, st));
    HIPCHK(launch_axpby(g, -1.0f, yn, 1.0f, (long)n, st));
    double sy, ss, yy;
    if ((rc = dot(sn, yn, sy)) || (rc = dot(sn, sn, ss)) || (rc = dot(yn, yn, yy))) return rc;
    if (sy > 1e-12 * std::sqrt(ss) * std::sqrt(yy)) {
      free_slots.pop_back();
      pairs.push_back(slot);
      if ((int)pairs.size() > memory) {
        free_slots.push_back(pairs.front());
        pairs.erase(pairs.begin());
      }
    }
    HIPCHK(hipMemcpyAsync(x, xt, (size_t)n * sizeof(float), hipMemcpyDeviceToDevice, st));
    HIPCHK(hipMemcpyAsync(g, gt, (size_t)n * sizeof(float), hipMemcpyDeviceToDevice, st));
    f = ft;
    if ((rc = dot(g, g, gg))) return rc;
    f_hist[it + 1] = f;
  }
  for (int j = it + 1; j <= maxiter; ++j) f_hist[j] = f;
  *iters = it;
  HIPCHK(hipStreamSynchronize(st));
  return FWIME_OK;
}

}  // extern "C"
