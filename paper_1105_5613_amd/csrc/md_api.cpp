// md_api.cpp -- the C ABI declared in include/md.h: validation, derived
// constants, device buffers, the per-step launch sequence and error latch.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <functional>
#include <mutex>
#include <string>
#include <type_traits>
#include <vector>

#include "brick.h"
#include "md_internal.h"
#include "stage.h"

using namespace mdk;

// Pair-distance histogram of md_rdf_static: a fixed device array, so that
// call allocates nothing.  Every GPU the library runs on holds its own copy
// (64 KiB) until the process ends; host code addresses it only through the
// per-device pointer hipGetSymbolAddress returns (scratch_dev).
constexpr int32_t kStaticBins = 8192;
static __device__ __align__(256) unsigned long long scratch[kStaticBins];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
unsigned long long* g_scratch_dev[kMaxDevices] = {};

// Look up this device's copy of scratch once (the device must be current).
hipError_t scratch_setup(int dev) {
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_dev[dev]) return hipSuccess;
  void* ptr = nullptr;
  const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
  if (e != hipSuccess) return e;
  g_scratch_dev[dev] = (unsigned long long*)ptr;
  return hipSuccess;
}

unsigned long long* scratch_dev(int dev) {
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  return dev >= 0 && dev < kMaxDevices ? g_scratch_dev[dev] : nullptr;
}
}  // namespace

struct md_ctx_s {
  md_params p{};
  int32_t device = 0;  // the device current at md_init
  int32_t nrep = 0, ntot = 0, stride = 0, ncells = 0, ntiles = 0, cap = 0, tpp = 1, unroll = 4;
  int32_t mixed = 0;
  // staged path (row tiles with LDS-staged neighbourhoods)
  int32_t staged = 0, nrt = 0, lcap_f = 0;
  int32_t cells = 0;  // list-free cell path (row tiles, no neighbour list)
  // brick path (brick.h): what MD_PATH_AUTO runs where it can (plan_bricks)
  bool brick = false;
  // list-free path on the same tiles (force_search.hip)
  bool search = false;
  int32_t search_threads = 0;
  std::vector<BrickTile> btiles_h;
  std::vector<Brick> bricks_h;
  BrickArgs ba{};
  BrickPair bp_h{};
  BrickPair* bp = nullptr;
  int32_t brick_parts = 0;   // partials of the force kernel
  double brick_homes = 0.0;  // expected home particles of the fullest tile
  int32_t brick_extra = 0;   // list chunks beyond the capacity's (one per pass but the first)
  int64_t brick_layer = 0;   // most particles of a layer of tiles (list_span_fits)
  int32_t last_thermo = 0;  // the last md_step call ran the thermostat (md_autotune)
  int32_t brick_tpp = 0, brick_unroll = 0;  // variant to return to the tiles with (enter_tiles)
  int32_t any_multi = 0;  // some replica has >= 3 cells per side
  int32_t ntiles1 = 0;    // tiles of the replicas with one cell
  Tile* tiles1 = nullptr;
  bool small_chain = false;  // one small replica: the one-block rebuild chain
  bool small_list = false;   // ... and the 32-lanes-per-particle list build
  std::vector<RowTile> rtiles_h;
  RowTile* rtiles = nullptr;
  uint16_t* nbr16 = nullptr;
  int32_t* cell_tile = nullptr;  // staged path: row tile of each cell
  hipStream_t stream = nullptr;
  std::vector<RepDesc> reps_h;
  std::vector<Tile> tiles_h;
  // device buffers
  RepDesc* reps = nullptr;
  Tile* tiles = nullptr;
  PairTab* tab = nullptr;
  int32_t thr_form = 4;  // form of the list thresholds in the neighbour search (fma_pair_form)
  int32_t rc2_form = 4;  // form of the force cutoffs on the list-free path
  int32_t nmax_rep = 0;  // particles of the largest replica
  DevState* st = nullptr;
  int32_t *cell_rep = nullptr, *counts = nullptr, *cell_start = nullptr, *bsum = nullptr;
  int32_t *cell_of = nullptr, *slot = nullptr, *tmp_src = nullptr;
  double4 *pos = nullptr, *pos_tmp = nullptr;
  int4* pos16 = nullptr;  // mixed form, gather path: cell-relative FP32 records
  double *vel = nullptr, *vel_tmp = nullptr, *xref = nullptr;
  void* frc = nullptr;
  int32_t *id = nullptr, *id_tmp = nullptr, *img = nullptr;
  uint32_t* nbr = nullptr;
  int32_t* ncount = nullptr;
  double* part = nullptr;
  int32_t* rebuild = nullptr;
  double* dmax = nullptr;   // [ntiles] per-tile max of the last drift
  // fused NVE steps (force mode 2): the drifted positions go to the other
  // buffer of a pair, pos <-> pos_tmp (pos_tmp is scratch of the rebuild
  // chain otherwise) and pos16 <-> pos16_alt; dpend [nrep] holds the drift
  // maximum measured for the next step
  int4* pos16_alt = nullptr;
  double* dpend = nullptr;
  // two-level reduction of the force partials (large replicas only)
  std::vector<RedChunk> chunks_h;
  RedChunk* chunks = nullptr;
  int32_t nchunks = 0, max_chunks = 0;
  double* part2 = nullptr;
  md_obs* obs = nullptr;
  int64_t* kcall = nullptr;
  double* lam = nullptr;
  double* therm = nullptr;  // T0 [nrep], T1 [nrep]
  double* u0 = nullptr;     // MSD reference, original id order [N][3]
  double* msd_part = nullptr;
  double* msd_out = nullptr;
  unsigned long long* rdf_hist = nullptr;  // pair counts of md_rdf
  md_obs* log_dev = nullptr;
  int64_t log_cap = 0;
  std::vector<void*> owned;
  md_allocator alloc{};  // alloc.alloc == nullptr: hipMalloc / hipFree
  // captured K-step graphs (md_params.graph_steps)
  hipStream_t cap_stream = nullptr;
  hipGraphExec_t gexec = nullptr;
  int64_t gkey[16] = {0};
  int32_t prof_epoch = 0;
  // force-kernel timing
  int32_t prof_every = 0;
  std::vector<hipEvent_t> ev_pool;
  size_t ev_used = 0;
  bool has_state = false, built = false, forces_valid = false;
  std::string err;
  int32_t err_bits = 0;  // device error bits behind the last failure of sync_and_check
};

namespace {

std::string g_init_error;

md_status fail(md_ctx c, md_status code, const std::string& msg) {
  if (c)
    c->err = msg;
  else
    g_init_error = msg;
  return code;
}

#define HIPCHECK(c, call)                                                                  \
  do {                                                                                     \
    hipError_t e_ = (call);                                                                \
    if (e_ != hipSuccess)                                                                  \
      return fail(c, MD_EHIP, std::string(#call " failed: ") + hipGetErrorString(e_));     \
  } while (0)

template <typename T>
md_status dalloc(md_ctx c, T** ptr, size_t count) {
  void* p = nullptr;
  size_t bytes = std::max<size_t>(count, 1) * sizeof(T);
  if (c->alloc.alloc) {
    p = c->alloc.alloc(c->alloc.u, bytes, (void*)c->stream);
    if (!p) return fail(c, MD_ENOMEM, "allocator returned NULL for " + std::to_string(bytes) + " bytes");
  } else if (hipMalloc(&p, bytes) != hipSuccess) {
    (void)hipGetLastError();
    return fail(c, MD_ENOMEM, "hipMalloc of " + std::to_string(bytes) + " bytes failed");
  }
  c->owned.push_back(p);
  *ptr = (T*)p;
  return MD_OK;
}

void dfree(md_ctx c, void* p) {
  if (!p) return;
  auto it = std::find(c->owned.begin(), c->owned.end(), p);
  if (it != c->owned.end()) c->owned.erase(it);
  if (c->alloc.alloc) {
    (void)hipStreamSynchronize(c->stream);  // nothing queued may still use p
    c->alloc.free(c->alloc.u, p, (void*)c->stream);
  } else {
    (void)hipFree(p);
  }
}

double max_rc(const md_params& p) {
  double m = 0.0;
  for (int a = 0; a < p.ntypes; ++a)
    for (int b = 0; b < p.ntypes; ++b) m = std::max(m, p.rc[a * MD_MAXT + b]);
  return m;
}

// Untruncated pair potential (Eq. (1) / Eq. (2)) and dV/dr at r, for the
// host-side shift constants of Eq. (3).
void plain_v(const md_params& p, int ab, double r, double* v, double* dv) {
  double s = p.sig[ab] / r;
  double s6 = s * s * s * s * s * s, s12 = s6 * s6;
  double e = p.eps[ab];
  if (p.potential == MD_POT_SOFT) {
    *v = 4.0 * e * s12;
    *dv = -48.0 * e * s12 / r;
  } else {
    *v = 4.0 * e * (s12 - s6);
    *dv = -4.0 * e * (12.0 * s12 - 6.0 * s6) / r;
  }
}

md_status validate(const md_params* p, std::string* why) {
  if (!p) return *why = "params is NULL", MD_EINVAL;
  if (p->ntypes < 1 || p->ntypes > MD_MAXT) return *why = "ntypes must be 1..4", MD_EINVAL;
  if (p->potential != MD_POT_LJ && p->potential != MD_POT_SOFT)
    return *why = "unknown potential", MD_EINVAL;
  if (p->trunc != MD_TRUNC_SHIFTED_FORCE && p->trunc != MD_TRUNC_SHIFT)
    return *why = "unknown truncation", MD_EINVAL;
  if (p->precision != MD_FP64 && p->precision != MD_MIXED)
    return *why = "unknown precision", MD_EINVAL;
  for (int a = 0; a < p->ntypes; ++a) {
    if (!(p->mass[a] > 0.0) || !std::isfinite(p->mass[a])) return *why = "mass must be > 0", MD_EINVAL;
    for (int b = 0; b < p->ntypes; ++b) {
      int ab = a * MD_MAXT + b, ba = b * MD_MAXT + a;
      if (!(p->sig[ab] > 0.0) || !(p->rc[ab] > 0.0) || !std::isfinite(p->eps[ab]) ||
          !std::isfinite(p->sig[ab]) || !std::isfinite(p->rc[ab]))
        return *why = "sigma and rc must be finite and > 0", MD_EINVAL;
      if (p->eps[ab] != p->eps[ba] || p->sig[ab] != p->sig[ba] || p->rc[ab] != p->rc[ba])
        return *why = "species tables must be symmetric", MD_EINVAL;
    }
  }
  if (!(p->skin >= 0.0) || !std::isfinite(p->skin)) return *why = "skin must be >= 0", MD_EINVAL;
  if (!(p->dt > 0.0) || !std::isfinite(p->dt)) return *why = "dt must be > 0", MD_EINVAL;
  if (p->max_neighbors < 0) return *why = "max_neighbors must be >= 0", MD_EINVAL;
  if (p->tpp != 0 && p->tpp != 1 && p->tpp != 2 && p->tpp != 4 && p->tpp != 8)
    return *why = "tpp must be 0, 1, 2, 4 or 8", MD_EINVAL;
  if (p->graph_steps < 0) return *why = "graph_steps must be >= 0", MD_EINVAL;
  if (p->unroll != 0 && p->unroll != 1 && p->unroll != 2 && p->unroll != 4 && p->unroll != 8)
    return *why = "unroll must be 0, 1, 2, 4 or 8", MD_EINVAL;
  if (p->path < MD_PATH_AUTO || p->path > MD_PATH_CELLS) return *why = "unknown path", MD_EINVAL;
  if (p->tile_cells < 0 || p->tile_cells > kMaxRowCells)
    return *why = "tile_cells must be 0..64", MD_EINVAL;
  if (p->stage_slots != 0 && p->stage_slots < 64) return *why = "stage_slots must be 0 or >= 64", MD_EINVAL;
  if (p->split_kick != 0 && p->split_kick != 1) return *why = "split_kick must be 0 or 1", MD_EINVAL;
  if (p->small_box != 0 && p->small_box != 1) return *why = "small_box must be 0 or 1", MD_EINVAL;
  return MD_OK;
}

md_status sync_and_check(md_ctx c) {
  HIPCHECK(c, hipStreamSynchronize(c->stream));
  DevState st{};
  HIPCHECK(c, hipMemcpy(&st, c->st, sizeof(DevState), hipMemcpyDeviceToHost));
  c->err_bits = st.err;
  if (st.err) {
    DevState z{};
    HIPCHECK(c, hipMemcpy(c->st, &z, sizeof(DevState), hipMemcpyHostToDevice));
    if (st.err & kErrSlots)
      return fail(c, MD_EOVERFLOW,
                  c->staged ? "a staged row tile's neighbourhood exceeds 16383 LDS slots (use "
                              "smaller tile_cells)"
                            : "a tile's neighbourhood exceeds its LDS slots");
    if (st.err & kErrOverflow)
      return fail(c, MD_EOVERFLOW, "neighbour list capacity exceeded");
    if (st.err & kErrType) return fail(c, MD_EINVAL, "species index out of range");
    if (st.err & kErrStray)
      return fail(c, MD_ENONFINITE, "a position left the box by more than one box length");
    return fail(c, MD_ENONFINITE, "non-finite position, velocity or force");
  }
  return MD_OK;
}

// zeroed: the kick of this step (or the fused force launch of the previous
// step) already cleared the cell histogram (one replica, see
// launch_kick_drift's nzero and FuseOut)
void run_chain(md_ctx c, hipStream_t s, bool zeroed = false) {
  // several replicas rebuild at different steps: spread each one's blocks
  // (bin/scatter: groups of 4 tiles; list build: groups of 32 cells)
  const int32_t spread_t = c->nrep > 1 ? 4 : 0, spread_c = c->nrep > 1 ? 32 : 0;
  if (c->small_chain) {
    // its histogram lives in LDS: nothing to clear
    launch_chain_small(s, c->ntot, c->reps, c->rebuild, c->pos, c->id, c->img, c->cell_start, c->stride,
                       c->vel, c->id_tmp, c->pos_tmp, c->vel_tmp, c->st, c->ba);
  } else {
    if (!zeroed) launch_zero_counts(s, c->ncells, c->cell_rep, c->rebuild, c->st, c->counts);
    launch_bin(s, c->ntiles, c->tiles, c->reps, c->rebuild, c->pos, c->id, c->img, c->counts,
               c->cell_of, c->slot, c->st, spread_t);
    launch_scan(s, c->ncells, c->counts, c->cell_start, c->bsum, c->st);
    launch_scatter(s, c->ntiles, c->tiles, c->rebuild, c->cell_of, c->slot, c->cell_start,
                   c->tmp_src, c->st, spread_t);
    launch_cell_gather(s, c->ncells, c->cell_rep, c->rebuild, c->cell_start, c->tmp_src,
                       c->stride, c->id, c->pos, c->vel, c->id_tmp, c->pos_tmp, c->vel_tmp,
                       c->st, c->reps, c->ba, c->nrep > 1);
  }
  if (c->brick)
    launch_nlist_brick(s, c->ba, c->p.ntypes, c->reps, c->rebuild, c->tab, c->cell_start,
                       c->stride, c->cap, c->bp_h, c->pos_tmp, c->vel_tmp, c->id_tmp, c->pos,
                       c->vel, c->id, c->xref, c->ncount, c->st, spread_c);
  else if (c->cells)
    launch_commit_order(s, c->ntiles, c->tiles, c->rebuild, c->stride, c->pos_tmp, c->vel_tmp,
                        c->id_tmp, c->pos, c->vel, c->id, c->xref, c->st);
  else if (c->staged)
    launch_nlist_tiles(s, c->ncells, c->cell_rep, c->reps, c->rebuild, c->tab, c->thr_form,
                       c->cell_start,
                       c->stride, c->cap, c->pos_tmp, c->vel_tmp, c->id_tmp, c->pos, c->vel, c->id,
                       c->xref, c->nbr16, c->ncount, c->st, c->cell_tile, c->rtiles, spread_c);
  else if (c->small_list && c->any_multi)
    launch_nlist_small(s, c->ntot, c->reps, c->rebuild, c->tab, c->cell_start, c->stride, c->cap,
                       c->pos_tmp, c->vel_tmp, c->id_tmp, c->pos, c->vel, c->id, c->xref, c->nbr,
                       c->ncount, c->st, c->pos16);
  else
    launch_nlist(s, c->ntiles1, c->tiles1, c->reps, c->rebuild, c->tab, c->thr_form, c->cell_start,
                 c->stride, c->cap, c->pos_tmp, c->vel_tmp, c->id_tmp, c->pos, c->vel, c->id,
                 c->xref, c->nbr, c->ncount, c->st, c->ncells, c->cell_rep, c->any_multi, c->pos16,
                 spread_c);
}

// Threads of a brick force block: the expected homes of the fullest tile with
// some room, at least four waves (which share the copy to LDS) and at most
// eight, of which three blocks run per CU; with no more blocks than CUs each
// has its CU to itself and takes sixteen for the copy.
int32_t brick_threads(md_ctx c) {
  const int32_t want = (int32_t)std::ceil(1.1 * c->brick_homes * c->tpp / 64.0) * 64;
  return c->ba.ntiles * c->ba.split <= 256 ? kBrickThreads : std::max(256, std::min(want, 512));
}

// energy: form PE and W (the row-tile kernels always do).
// mode 2 (gather lists, tiles of cells): the fused NVE step, see FuseOut; the caller
// swaps the position buffers after the launch.
void launch_forces(md_ctx c, int32_t mode, hipStream_t s, int32_t energy = 1,
                   int32_t nzero = 0) {
  if (c->brick)
    launch_force_brick(s, c->mixed, mode, energy, c->tpp, brick_threads(c), c->bp_h.four, c->ba,
                       c->reps, c->tab, c->bp, c->pos, c->vel, c->frc, c->stride, c->p.dt,
                       c->part, c->st, FuseOut{c->pos_tmp, nullptr, c->xref, c->counts, nzero});
  else if (c->search)
    launch_force_search(s, c->mixed, mode, energy, c->search_threads, c->bp_h.four, c->ba, c->reps,
                        c->tab, c->bp, c->cell_start, c->pos, c->vel, c->frc, c->stride, c->p.dt,
                        c->part, c->st, FuseOut{c->pos_tmp, nullptr, c->xref, c->counts, nzero});
  else if (c->cells)
    launch_force_cells(s, c->mixed, mode, c->rc2_form, c->nrt, c->rtiles, c->reps, c->tab,
                       c->cell_start, c->pos, c->vel, c->frc, c->stride, c->p.dt, c->part,
                       c->st);
  else if (c->staged)
    launch_force_staged(s, c->mixed, mode, c->tpp, c->unroll, c->nrt, c->rtiles, c->reps,
                        c->tab, c->cell_start, c->pos, c->vel, c->frc, c->nbr16, c->ncount,
                        c->stride, c->cap, c->lcap_f, c->p.dt, c->part, c->st);
  else
    launch_force(s, c->mixed, mode, energy,
                 (size_t)c->nmax_rep * c->cap * sizeof(uint32_t) > kStreamListBytes, c->tpp,
                 c->unroll, c->ntiles, c->tiles, c->reps, c->tab, c->pos, c->pos16, c->vel,
                 c->frc, c->nbr, c->ncount, c->stride, c->cap, c->p.dt, c->part, c->st,
                 FuseOut{c->pos_tmp, c->pos16_alt, c->xref, c->counts, nzero});
}

// Constants of the brick force kernel from the pair table.  The two-species
// form needs base + 2 d = value bit for bit for every constant, with the base
// taken for one species throughout; that holds for one of the two choices
// unless the constants are very uneven, and then (as with more species) the
// kernel reads a table.
BrickPair brick_pair(const md_params& p, const PairTab& t) {
  BrickPair b{};
  b.mk = p.potential == MD_POT_SOFT ? 0.0f : 0.5f;
  double smin = p.sig[0];
  for (int a = 0; a < p.ntypes; ++a)
    for (int q = 0; q < p.ntypes; ++q) smin = std::min(smin, p.sig[a * MD_MAXT + q]);
  b.tiny = 1e-30 * smin * smin;  // (smin^2 / tiny)^7 is an ordinary double
  b.four = 1;
  if (p.ntypes > 2) return b;
  for (int32_t flip = p.ntypes == 1 ? 1 : 0; flip < 2; ++flip) {
    bool exact = true;
    auto split = [&](auto (&out)[2], double base, double value) {
      using V = std::remove_reference_t<decltype(out[0])>;
      const V lo = (V)base, v = (V)value;
      const V d = (v - lo) * (V)0.5;
      out[0] = lo;
      out[1] = d;
      exact = exact && std::fma(d, (V)2.0, lo) == v;
    };
    for (int a = 0; a < p.ntypes; ++a) {
      // species 1 - flip: bit clear; species flip: bit set (absent with one species)
      const int k0 = a * MD_MAXT + (1 - flip), k1 = p.ntypes == 1 ? k0 : a * MD_MAXT + flip;
      auto s6 = [&](int k) { return t.sig2[k] * t.sig2[k] * t.sig2[k]; };
      split(b.rc2[a], t.rc2[k0], t.rc2[k1]);
      split(b.a[a], t.f12[k0] * (s6(k0) * s6(k0)), t.f12[k1] * (s6(k1) * s6(k1)));
      split(b.b[a], t.f6[k0] * s6(k0), t.f6[k1] * s6(k1));
      split(b.fs[a], t.fs[k0], t.fs[k1]);
      split(b.msig2[a], t.sig2[k0], t.sig2[k1]);
      split(b.mf12[a], t.f12[k0], t.f12[k1]);
      split(b.mfs[a], t.fs[k0], t.fs[k1]);
      // energies only, where the last bit of a constant does not matter
      auto v12 = [&](int k) { return 12.0 * (t.vc[k] - t.rc[k] * t.fs[k]); };
      b.v12[a][0] = v12(k0);
      b.v12[a][1] = (v12(k1) - v12(k0)) * 0.5;
      b.mrc[a][0] = (float)t.rc[k0];
      b.mrc[a][1] = (float)t.rc[k1];
      b.mv12[a][0] = (float)(12.0 * t.vc[k0]);
      b.mv12[a][1] = (float)(12.0 * t.vc[k1]);
    }
    if (exact) {
      b.flip = flip;
      b.four = 0;
      return b;
    }
  }
  b.flip = 0;
  return b;
}

// List chunks per particle on the brick path for a capacity in entries.
int32_t chunk_capacity(md_ctx c, int32_t cap) {
  const int64_t chunks = ((int64_t)cap + kChunkEntries - 1) / kChunkEntries;
  return (int32_t)std::min<int64_t>(chunks + c->brick_extra, kMostChunks);
}

// Whether the context takes the brick path, or on MD_PATH_CELLS the search on
// tiles of cells, and its tiles and bricks.  Conditions: MD_PATH_AUTO with no
// force variant asked for by tpp or unroll (those name gather variants), or
// MD_PATH_CELLS with no row tile asked for by tile_cells; at least three cells
// per side in every replica, parameters whose r^-12 coefficient is an ordinary
// double, and in every replica 27 cells that fit the LDS slots.  (The search
// keeps to the smaller LDS layout, two blocks of which leave room for its
// words, and spares 6 %: a tile that outgrows it costs one rebuild.  20 steps
// without lists at 1,372 / 20,000 / 1,048,576 particles FP64: 74 / 65 / 441 us
// a step, by row tiles 278 / 269 / 1,397.)
//
// Tiles: the most home cells (up to 4 per axis) whose expected neighbourhood
// fits the slots with 12 % to spare and whose homes fit one or two rounds of
// a block (240), as the copy to LDS is paid per neighbourhood cell.  (Cells
// between 2.8 and 3 wide hold 26 to 32 particles: 2 x 2 x 2 of them need up to
// 2,350 slots, hence the larger LDS layout.)  The smaller layout, of which
// three blocks fit a CU, is taken where it holds eight home cells: nine in the
// larger one (16,777,216 particles, 26.4 per cell) took 2,855 us per mixed
// launch, eight here 2,545; with six or seven the larger one is the faster (262,144
// particles, 28.3 per cell: 103 us a step, six cells in the smaller 120).  A
// replica's tiles follow from its own density only, so that its sums on them are
// the same alone and in a batch.  Whether the context takes them is decided by
// all its replicas together.
bool plan_bricks(md_ctx c) {
  const md_params& p = c->p;
  const bool cells = c->cells;  // for the list-free search
  if (cells ? p.tile_cells != 0 : p.path != MD_PATH_AUTO || p.tpp != 0 || p.unroll != 0)
    return false;
  for (int a = 0; a < p.ntypes; ++a)
    for (int b = 0; b < p.ntypes; ++b) {
      const double s = p.sig[a * MD_MAXT + b], e = std::fabs(p.eps[a * MD_MAXT + b]);
      if (s < 1e-15 || s > 1e15 || (e != 0.0 && (e < 1e-60 || e > 1e60))) return false;
    }
  const double spare = cells ? 1.06 : 1.12;
  const int32_t most = cells ? kBrickSlots : kBrickSlotsBig;
  auto slots = [&](double ppc, int x, int y, int z) {
    return spare * ppc * (x + 2) * (y + 2) * (z + 2) + 48.0;
  };
  // cells per axis of a replica's tiles, and whether they take the larger layout
  struct Shape {
    int32_t x, y, z;
    bool big;
  };
  auto shape = [&](const RepDesc& d) {
    const double ppc = (double)d.n / ((double)d.nc * d.nc * d.nc);
    Shape b{};
    auto fits = [&](int32_t room) {
      b.x = b.y = b.z = 1;
      for (int x = 1; x <= std::min(4, d.nc); ++x)
        for (int y = 1; y <= x; ++y)
          for (int z = 1; z <= y; ++z) {
            const double homes = ppc * x * y * z;
            if (homes > 240.0 || slots(ppc, x, y, z) >= room) continue;
            const int v = x * y * z, bv = b.x * b.y * b.z;
            const int h = (x + 2) * (y + 2) * (z + 2), bh = (b.x + 2) * (b.y + 2) * (b.z + 2);
            if (v > bv || (v == bv && h < bh)) b.x = x, b.y = y, b.z = z;
          }
      return b.x * b.y * b.z;
    };
    if (fits(std::min(most, kBrickSlots)) < 8) fits(most);
    // three cells a side: nine even tiles of one row of cells in the smaller
    // layout instead of six to eight uneven ones in the larger (replicas of 1,000
    // particles, per step, tiles of 3 x 2 x 1 -> so: 64 of them 93.0 -> 86.5 us,
    // mixed 89.5 -> 84.0, 256: 148 -> 135 and 140 -> 130; by gathers 82, 81, 151
    // and 131; 8: 40.9 -> 42.4, by gathers 73)
    if (!cells && d.nc == 3 && slots(ppc, 3, 1, 1) < kBrickSlots)
      b.x = 3, b.y = b.z = 1;
    b.big = slots(ppc, b.x, b.y, b.z) >= kBrickSlots;
    return b;
  };
  int64_t tiles = 0;
  c->brick_layer = 0;
  for (const RepDesc& d : c->reps_h) {
    if (d.nc < 3) return false;
    // short lists: the copy of the neighbourhood is not earned back (the
    // soft-sphere box, 15 entries: 57 us by gathers, 96 by bricks; without
    // lists the search is the faster form there too, 20 steps of 1,048,576
    // particles in 6,360 us against 10,510)
    const double side = max_rc(p) + p.skin;
    if (!cells && (double)d.n / d.volume * 4.0 / 3.0 * M_PI * side * side * side < 48.0)
      return false;
    if (slots((double)d.n / ((double)d.nc * d.nc * d.nc), 1, 1, 1) >= most) return false;
    const Shape b = shape(d);
    auto along = [&](int32_t t) { return (int64_t)((d.nc + t - 1) / t); };
    tiles += along(b.x) * along(b.y) * along(b.z);
    // a layer of tiles: each holds its cells and those around them in the
    // slots, and in tiles up to two cells wide every cell is counted twice
    const int64_t twice = (b.x <= 2 ? 2 : 1) * (b.y <= 2 ? 2 : 1);
    const int64_t layer = (along(b.x) * along(b.y) * (kBrickSlotsBig - 1) + twice - 1) / twice;
    c->brick_layer = std::max(c->brick_layer, std::min<int64_t>(d.n, layer));
  }
  // (with the default capacity: up to 2^26 particles, the most of the path)
  if (!cells &&
      !list_span_fits(c->brick_layer, std::min(kMostChunks, c->cap / kChunkEntries + 5)))
    return false;
  // a launch holds fewer than 2^32 threads, and a force launch one block of at
  // most 512 per tile (of 1,024 where there are at most 256 blocks): 8.4
  // million tiles, which only list-free boxes of some 10^9 particles reach when
  // they are dilute; row tiles take them
  if (tiles > 0xffffffffll / (64 * search_waves())) return false;
  c->btiles_h.clear();
  c->bricks_h.clear();
  c->brick_parts = 0;
  c->ba = BrickArgs{};
  bool big = false;
  int32_t waves = 1;  // of the search, most of a tile
  for (int32_t r = 0; r < c->nrep; ++r) {
    RepDesc& d = c->reps_h[r];
    const int32_t nc = d.nc;
    const double ppc = (double)d.n / ((double)nc * nc * nc);
    const Shape sh = shape(d);
    const int32_t bx = sh.x, by = sh.y, bz = sh.z;
    const bool rbig = sh.big;
    const int32_t pass = nlist_brick_pass(rbig);
    big |= rbig;
    // bricks of a tile: the matrix product takes 32 homes at a time against
    // 64 candidates; three chunks' worth of time per brick go elsewhere
    int hx = 1, hy = 1, hz = 1;
    double best = 1e300;
    for (int x = 1; x <= bx; ++x)
      for (int y = 1; y <= by; ++y)
        for (int z = 1; z <= bz; ++z) {
          const double homes = ppc * x * y * z, cand = ppc * (x + 2) * (y + 2) * (z + 2);
          // (the search has one wave per brick: as many as a tile has cells, up to eight)
          const int32_t of_tile = ((bx + x - 1) / x) * ((by + y - 1) / y) * ((bz + z - 1) / z);
          if (cells && of_tile < std::min(bx * by * bz, search_waves())) continue;
          const double cost = (std::ceil(cand * 1.02 / 64.0) + 3.0) *
                              std::ceil(1.08 * homes / 32.0) / homes;
          if (cost < best) best = cost, hx = x, hy = y, hz = z;
        }
    const double cand = ppc * (hx + 2) * (hy + 2) * (hz + 2);
    // search in tiles of few, crowded bricks: several waves take a brick's
    // groups of homes (a step of 1,048,576 particles mixed: 32 per cell, four
    // bricks a tile, one wave each 1,307 us, two waves each 716; 43 per cell,
    // one brick and one wave of two cells 2,925, two bricks of two waves 1,113;
    // by row tiles 1,262 and 1,728)
    const int32_t full = ((bx + hx - 1) / hx) * ((by + hy - 1) / hy) * ((bz + hz - 1) / hz);
    const int32_t share = std::max(1, std::min((int32_t)std::ceil(1.08 * ppc * hx * hy * hz / 32.0),
                                               search_waves() / full));
    c->ba.groups = std::max(c->ba.groups,
                            (int32_t)std::ceil(1.15 * ppc * hx * hy * hz / 32.0));
    c->brick_extra = std::max(c->brick_extra, (int32_t)(1.15 * cand / (64 * pass)));
    d.fb0 = c->brick_parts;
    // the tiles along each axis, as even as they come, and their bricks
    struct Piece {
      int32_t first, cells;
    };
    auto cut = [](int32_t n, int32_t most_cells) {
      const int32_t parts = (n + most_cells - 1) / most_cells;
      std::vector<Piece> v(parts);
      for (int32_t k = 0; k < parts; ++k) {
        v[k].first = (int32_t)((int64_t)n * k / parts);
        v[k].cells = (int32_t)((int64_t)n * (k + 1) / parts) - v[k].first;
      }
      return v;
    };
    const std::vector<Piece> tx = cut(nc, bx), ty = cut(nc, by), tz = cut(nc, bz);
    std::vector<Piece> cx[5], cy[5], cz[5];  // bricks of a tile of that many cells
    for (int32_t t = 1; t <= 4; ++t) cx[t] = cut(t, hx), cy[t] = cut(t, hy), cz[t] = cut(t, hz);
    const int32_t units =
        !cells && (int64_t)tx.size() * ty.size() * tz.size() <= 256 ? kTileUnits : 1;
    c->btiles_h.reserve(c->btiles_h.size() + tx.size() * ty.size() * tz.size());
    c->bricks_h.reserve(c->bricks_h.size() +
                        (size_t)(1.3 * nc * nc * nc / (hx * hy * hz)) + 64);
    for (const Piece& z : tz)
      for (const Piece& y : ty)
        for (const Piece& x : tx) {
          BrickTile t{};
          t.rep = r;
          t.cx = x.first;
          t.cy = y.first;
          t.cz = z.first;
          t.tx = x.cells;
          t.ty = y.cells;
          t.tz = z.cells;
          t.units = units;
          t.part = c->brick_parts;
          c->brick_parts += units;
          const int32_t id = (int32_t)c->btiles_h.size();
          t.b0 = (int32_t)c->bricks_h.size();
          for (const Piece& w : cz[t.tz])
            for (const Piece& v : cy[t.ty])
              for (const Piece& u : cx[t.tx]) {
                Brick b{};
                b.tile = id;
                b.pass = (int8_t)pass;
                b.lx = (int8_t)u.first;
                b.ly = (int8_t)v.first;
                b.lz = (int8_t)w.first;
                b.hx = (int8_t)u.cells;
                b.hy = (int8_t)v.cells;
                b.hz = (int8_t)w.cells;
                c->bricks_h.push_back(b);
              }
          t.nb = (int32_t)c->bricks_h.size() - t.b0;
          t.groups = share;
          t.waves = std::min(t.nb * share, search_waves());
          waves = std::max(waves, t.waves);
          c->btiles_h.push_back(t);
          c->ba.rows = std::max(c->ba.rows, (t.ty + 2) * (t.tz + 2));
          c->ba.hrows = std::max(c->ba.hrows, t.ty * t.tz);
          c->brick_homes = std::max(c->brick_homes, ppc * t.tx * t.ty * t.tz);
        }
    d.fb1 = c->brick_parts;
  }
  c->ba.ntiles = (int32_t)c->btiles_h.size();
  c->ba.nbricks = (int32_t)c->bricks_h.size();
  c->ba.slots = big ? kBrickSlotsBig : kBrickSlots;
  c->ba.shift = big ? 2 : 3;
  // few tiles: a tile's homes go to several blocks, each with a copy of the
  // neighbourhood (4,000 particles, 27 tiles: a launch 16.4 us
  // with one block per tile, 12.2 us with four; the gather kernel 17.2 us)
  c->ba.split = c->ba.ntiles <= 64 ? 4 : (c->ba.ntiles <= 128 ? 2 : 1);
  for (const BrickTile& t : c->btiles_h)
    if (t.units == 1) c->ba.split = 1;
  c->brick = !cells;
  c->search = cells;
  c->search_threads = 64 * waves;
  return true;
}

void drop_graph(md_ctx c);
md_status leave_brick(md_ctx c);
void free_gather(md_ctx c);
void free_chunks(md_ctx c);

// Grow the neighbour capacity after an overflowed build to the longest row it
// found plus 16 (never below the old capacity).  The rows already built move
// to the new layout (a replica that did not rebuild keeps its list bit for
// bit); the overflowed rows are rebuilt by the caller.  A captured graph
// holds the old list pointer and capacity and is dropped.
md_status grow_capacity(md_ctx c) {
  std::vector<int32_t> cnt(c->ntot);
  HIPCHECK(c, hipMemcpy(cnt.data(), c->ncount, sizeof(int32_t) * c->ntot, hipMemcpyDeviceToHost));
  int32_t m = 0;
  for (int32_t v : cnt) m = std::max(m, v);
  if (c->brick) {
    // chunks of rows built in several passes are not all full
    std::vector<int32_t> ch(c->ntot);
    HIPCHECK(c, hipMemcpy(ch.data(), c->ba.nchunk, sizeof(int32_t) * c->ntot,
                          hipMemcpyDeviceToHost));
    for (int32_t v : ch)
      if (v > c->ba.capc) m = std::max(m, v * kChunkEntries);
  }
  if (m <= c->cap) return fail(c, MD_EOVERFLOW, "overflow flagged with every row within capacity");
  const int32_t cap = std::max(c->cap, ((m + 16 + 7) / 8) * 8);
  if (c->brick) {
    uint4* fresh = nullptr;
    const int32_t capc = chunk_capacity(c, cap);
    if (!list_span_fits(c->brick_layer, capc)) return leave_brick(c);
    md_status rc = dalloc(c, &fresh, chunk_elems(c->ntot, capc));
    if (rc) return rc;
    launch_relayout_chunks(c->stream, c->ntot, c->ba.nchunk, c->ba.capc, capc, c->ba.list, fresh);
    HIPCHECK(c, hipGetLastError());
    HIPCHECK(c, hipStreamSynchronize(c->stream));
    free_chunks(c);
    free_gather(c);  // of the old capacity, where a switch left one
    c->ba.list = fresh;
    c->ba.capc = capc;
    c->cap = cap;
    drop_graph(c);
    return MD_OK;
  }
  const int32_t elem = c->staged ? 2 : 4;
  void* old = c->staged ? (void*)c->nbr16 : (void*)c->nbr;
  md_status rc;
  void* fresh = nullptr;
  if (c->staged) {
    uint16_t* p = nullptr;
    rc = dalloc(c, &p, list_elems(c->ntot, cap));
    fresh = p;
  } else {
    uint32_t* p = nullptr;
    rc = dalloc(c, &p, list_elems(c->ntot, cap));
    fresh = p;
  }
  if (rc) return rc;
  launch_relayout_list(c->stream, c->ntot, c->ncount, c->cap, cap, elem, old, fresh);
  HIPCHECK(c, hipGetLastError());
  HIPCHECK(c, hipStreamSynchronize(c->stream));
  dfree(c, old);
  if (c->staged)
    c->nbr16 = (uint16_t*)fresh;
  else
    c->nbr = (uint32_t*)fresh;
  c->cap = cap;
  drop_graph(c);
  return MD_OK;
}

void plan_chunks(md_ctx c);

// Partial-sum blocks of the gather path: tpp blocks per tile.
void gather_blocks(md_ctx c) {
  for (RepDesc& d : c->reps_h) {
    d.fb0 = d.tile0 * c->tpp;
    d.fb1 = d.tile1 * c->tpp;
  }
}

// ... and of the row tiles, which the replicas' tiles follow each other in.
void row_tile_blocks(md_ctx c) {
  int32_t t = 0;
  for (int32_t r = 0; r < c->nrep; ++r) {
    RepDesc& d = c->reps_h[r];
    d.fb0 = t;
    while (t < c->nrt && c->rtiles_h[t].rep == r) ++t;
    d.fb1 = t;
  }
}

md_status upload_blocks(md_ctx c) {
  plan_chunks(c);
  if (c->nchunks)
    HIPCHECK(c, hipMemcpyAsync(c->chunks, c->chunks_h.data(), sizeof(RedChunk) * c->nchunks,
                               hipMemcpyHostToDevice, c->stream));
  HIPCHECK(c, hipMemcpyAsync(c->reps, c->reps_h.data(), sizeof(RepDesc) * c->nrep,
                             hipMemcpyHostToDevice, c->stream));
  // the host vectors are re-planned only after the copies finished
  HIPCHECK(c, hipStreamSynchronize(c->stream));
  return MD_OK;
}

// The buffers of the gather path, all of them or none.
md_status alloc_gather(md_ctx c) {
  if (c->nbr) return MD_OK;
  uint32_t* nbr = nullptr;
  int4 *rec = nullptr, *alt = nullptr;
  md_status rc = dalloc(c, &nbr, list_elems(c->ntot, c->cap));
  if (!rc && c->mixed) rc = dalloc(c, &rec, (size_t)c->stride);
  if (!rc && c->mixed) rc = dalloc(c, &alt, (size_t)c->stride);
  if (rc) {
    dfree(c, nbr);
    dfree(c, rec);
    return rc;
  }
  c->nbr = nbr;
  c->pos16 = rec;
  c->pos16_alt = alt;
  return MD_OK;
}

void free_gather(md_ctx c) {
  dfree(c, c->nbr);
  dfree(c, c->pos16);
  dfree(c, c->pos16_alt);
  c->nbr = nullptr;
  c->pos16 = c->pos16_alt = nullptr;
}

void free_chunks(md_ctx c) {
  dfree(c, c->ba.list);
  c->ba.list = nullptr;
}

// The buffers of the path that the context is on; a switch that failed for want
// of memory may have given them back.
md_status path_buffers(md_ctx c) {
  if (c->brick && !c->ba.list)
    return dalloc(c, &c->ba.list, chunk_elems(c->ntot, c->ba.capc));
  return c->brick || c->staged || c->cells ? MD_OK : alloc_gather(c);
}

// A tile whose neighbourhood outgrew the LDS slots (a box that condensed far
// above its mean density): the context, with all its replicas, goes on with
// gather lists, which take any density, until the next md_set_state
// (enter_tiles).  Every replica is marked for a rebuild.  Nothing is switched
// before the gather buffers are there: a call that fails here leaves the context
// on its tiles, to try again at the next build.  Both lists are kept from then
// on, as long as they fit side by side.
md_status leave_brick(md_ctx c) {
  HIPCHECK(c, hipStreamSynchronize(c->stream));
  md_status rc = alloc_gather(c);
  if (rc) {
    free_chunks(c);
    rc = alloc_gather(c);
  }
  if (rc) {
    c->built = c->forces_valid = false;
    return rc;
  }
  c->ba.ntiles = 0;
  c->ba.nbricks = 0;
  c->brick = false;
  c->brick_tpp = c->tpp;
  c->brick_unroll = c->unroll;
  c->tpp = 2;
  c->unroll = 4;
  gather_blocks(c);
  drop_graph(c);
  launch_mark_rebuild(c->stream, c->nrep, c->rebuild, c->st);
  return upload_blocks(c);
}

// The same on the list-free path: row tiles take any density.
md_status leave_search(md_ctx c) {
  HIPCHECK(c, hipStreamSynchronize(c->stream));
  c->search = false;
  c->ba.ntiles = 0;
  row_tile_blocks(c);
  drop_graph(c);
  launch_mark_rebuild(c->stream, c->nrep, c->rebuild, c->st);
  return upload_blocks(c);
}

// A new state starts on the tiles again if the context left them, so that it is
// evaluated as in a new context.  (Without memory for their list it stays on
// gather lists.)
md_status enter_tiles(md_ctx c) {
  if (c->brick || c->search || c->btiles_h.empty()) return MD_OK;
  HIPCHECK(c, hipStreamSynchronize(c->stream));
  if (!c->cells) {
    const int32_t capc = chunk_capacity(c, c->cap);  // it may have grown since
    if (!list_span_fits(c->brick_layer, capc)) return MD_OK;
    if (capc != c->ba.capc) free_chunks(c);
    c->ba.capc = capc;
    if (!c->ba.list && dalloc(c, &c->ba.list, chunk_elems(c->ntot, capc))) {
      free_gather(c);
      if (dalloc(c, &c->ba.list, chunk_elems(c->ntot, capc))) return MD_OK;
    }
    c->tpp = c->brick_tpp;
    c->unroll = c->brick_unroll;
  }
  c->brick = !c->cells;
  c->search = c->cells;
  c->ba.ntiles = (int32_t)c->btiles_h.size();
  c->ba.nbricks = (int32_t)c->bricks_h.size();
  for (const BrickTile& t : c->btiles_h) {  // a replica's tiles follow each other
    RepDesc& d = c->reps_h[t.rep];
    if (t.cx == 0 && t.cy == 0 && t.cz == 0) d.fb0 = t.part;
    d.fb1 = t.part + t.units;
  }
  drop_graph(c);
  return upload_blocks(c);
}

// Full rebuild of every replica (md_build_cells and the first build after
// md_set_state); grows the neighbour capacity once on overflow.
md_status build_all(md_ctx c) {
  if (const md_status rc = path_buffers(c)) return rc;
  for (bool grown = false;;) {
    launch_mark_rebuild(c->stream, c->nrep, c->rebuild, c->st);
    run_chain(c, c->stream);
    md_status rc = sync_and_check(c);
    // counted as a build, unless the context leaves its tiles for it
    if (!(c->err_bits & kErrSlots) || c->staged)
      launch_after_build(c->stream, c->nrep, c->rebuild, c->obs, c->st);
    if (rc == MD_OK) {
      c->built = true;
      c->forces_valid = false;
      return MD_OK;
    }
    if (rc != MD_EOVERFLOW) return rc;
    if (c->err_bits & kErrSlots) {  // not a capacity
      if (!c->brick && !c->search) return rc;
      rc = c->brick ? leave_brick(c) : leave_search(c);
    } else {
      if (grown) return rc;
      const bool tiles = c->brick;
      rc = grow_capacity(c);
      grown = c->brick == tiles;  // or it went on with gather lists
    }
    if (rc) return rc;
  }
}

ThermoArgs no_thermo() {
  ThermoArgs t{};
  return t;
}

void launch_reductions(md_ctx c, hipStream_t s, int32_t step, const ThermoArgs& ta,
                       int32_t energy = 1, int32_t drift_src = 0, int32_t next = 0) {
  if (c->nchunks)
    launch_reduce_chunks(s, c->nchunks, c->chunks, c->part, c->dmax, step, next, c->part2,
                         c->st);
  launch_reduce(s, c->nrep, c->reps, c->part, c->dmax, c->nchunks ? c->part2 : nullptr, step,
                energy, DriftArgs{drift_src, next, c->dpend}, ta, c->kcall, c->lam, c->rebuild,
                c->obs, c->st);
}

// Split every replica's partial blocks [fb0, fb1) (and drift tiles) into
// chunks of about kRedChunk when some replica has more than 16 chunks' worth;
// otherwise the per-replica pass reads the partials directly (one launch
// instead of two: up to 16 partials per thread of its block).  Host side
// only: the caller uploads reps and chunks.
void plan_chunks(md_ctx c) {
  int32_t most = 0;
  for (const RepDesc& d : c->reps_h) most = std::max(most, d.fb1 - d.fb0);
  c->chunks_h.clear();
  if (most <= 16 * kRedChunk) {
    c->nchunks = 0;
    for (RepDesc& d : c->reps_h) d.cb0 = d.cb1 = 0;
    return;
  }
  for (RepDesc& d : c->reps_h) {
    const int64_t nb = d.fb1 - d.fb0, nt = d.tile1 - d.tile0;
    const int64_t nch = std::max<int64_t>(1, (nb + kRedChunk - 1) / kRedChunk);
    d.cb0 = (int32_t)c->chunks_h.size();
    for (int64_t j = 0; j < nch; ++j) {
      RedChunk ch;
      ch.b0 = d.fb0 + (int32_t)(nb * j / nch);
      ch.b1 = d.fb0 + (int32_t)(nb * (j + 1) / nch);
      ch.t0 = d.tile0 + (int32_t)(nt * j / nch);
      ch.t1 = d.tile0 + (int32_t)(nt * (j + 1) / nch);
      c->chunks_h.push_back(ch);
    }
    d.cb1 = (int32_t)c->chunks_h.size();
  }
  c->nchunks = (int32_t)c->chunks_h.size();
}

void launch_forces0(md_ctx c) {
  launch_forces(c, 0, c->stream);
  launch_reductions(c, c->stream, 0, no_thermo());
}


// Directly launched NVE steps of a one-replica context on gather lists or tiles
// of cells can fuse the next step's kick and drift into the force launch (md_params.split_kick).
bool can_fuse(md_ctx c, int32_t thermo) {
  return !thermo && c->nrep == 1 && (!c->cells || c->search) && !c->staged && c->p.split_kick == 0;
}

// One velocity-Verlet step on stream s (also used while capturing a graph).
// energy: the step forms PE and W (the observables refreshed on it).
// kick: launch this step's first half kick and drift (false when the
// previous step's fused force launch applied them).  fuse: this step's force
// launch applies the next step's kick and drift (force mode 2); the next
// step is then enqueued with kick = false.
// resume: finish a step whose list build overflowed (kHalt): its kick and
// drift are done and its histogram is stale, so the chain clears the counts
// itself; drift_src (0: kick tile maxima, 1: the maximum the previous fused
// force launch stored) is then the one of the interrupted step.
md_status enqueue_step(md_ctx c, hipStream_t s, const ThermoArgs& ta, int32_t thermo, int32_t k,
                       int32_t energy, bool kick = true, bool fuse = false, bool resume = false,
                       int32_t drift_src = -1) {
  // one replica: its histogram is read only inside a rebuild, so the kick
  // (or the fused force launch before it) clears it when its threads cover
  // the cells (not in very dilute boxes) and the chain skips a launch (the
  // one-block chain of a small box keeps its histogram in LDS)
  const bool zero_in_kick = c->nrep == 1 && !c->small_chain &&
                            (int64_t)c->ncells <= (int64_t)c->ntiles * kTile;
  const int32_t nzero = zero_in_kick ? c->ncells : 0;
  if (kick && !resume)
    launch_kick_drift(s, c->mixed, thermo, c->ntiles, c->tiles, c->reps, c->tab, c->pos,
                      c->brick ? nullptr : c->pos16, c->vel, c->frc, c->xref, c->stride, c->p.dt,
                      c->lam, c->rebuild, c->dmax, c->st, c->counts, nzero);
  run_chain(c, s, zero_in_kick && !resume);
  const bool timed = c->prof_every > 0 && (k + 1) % c->prof_every == 0;
  if (timed) {
    if (c->ev_pool.size() < c->ev_used + 2) return fail(c, MD_EHIP, "event pool exhausted");
    HIPCHECK(c, hipEventRecord(c->ev_pool[c->ev_used], s));
  }
  launch_forces(c, fuse ? 2 : 1, s, energy, fuse ? nzero : 0);
  if (timed) {
    HIPCHECK(c, hipEventRecord(c->ev_pool[c->ev_used + 1], s));
    c->ev_used += 2;
  }
  if (fuse) {
    std::swap(c->pos, c->pos_tmp);
    std::swap(c->pos16, c->pos16_alt);
  }
  launch_reductions(c, s, 1, ta, energy, drift_src >= 0 ? drift_src : (kick ? 0 : 1),
                    fuse ? 1 : 0);
  return MD_OK;
}

// Steps that form PE and W: the logged ones and the last of the run (the
// observables md_observables returns).  Inside a K-step graph: the logged
// steps when the log cadence divides K (the same steps in every replay),
// every step otherwise, and always the graph's last step.
int32_t energy_step(const ThermoArgs& ta, int64_t k, int64_t last) {
  if (k == last) return 1;
  return ta.log_every > 0 && (k + 1) % ta.log_every == 0;
}
int32_t energy_step_graph(const ThermoArgs& ta, int32_t k, int32_t K) {
  if (k == K - 1) return 1;
  if (ta.log_every <= 0) return 0;
  return K % ta.log_every != 0 || (k + 1) % ta.log_every == 0;
}

md_status reserve_events(md_ctx c, int32_t nsteps);

// Whether directly launched step k also applies the next step's kick and drift.
// Not the last step of a call, and on the tiles of the mixed form no step that
// forms energies: that launch fused does not hold its registers at three blocks
// per CU (logged every step, 1,048,576 particles: 301 us a step fused at two,
// 276 not fused; FP64, two blocks either way: 326 against 343).
bool fuses(md_ctx c, const ThermoArgs& ta, int32_t k, int32_t nsteps, bool fusable) {
  return fusable && k + 1 < nsteps &&
         !(c->brick && c->mixed && energy_step(ta, k, nsteps - 1));
}

// Directly launched steps [k0, nsteps) of an md_step call whose steps
// [0, kg) ran inside graph replays.  A step launched here after another one
// of this loop had its kick and drift applied by that step's force launch
// when the call can fuse.  resume: step k0 was interrupted by an overflowed
// list build after its kick and drift; its drift maximum is where that kick
// left it, src = 1: the previous force launch's partials (a fused direct step),
// 0: the kick's tile maxima.
md_status enqueue_direct(md_ctx c, hipStream_t s, const ThermoArgs& ta, int32_t thermo,
                         int32_t k0, int32_t nsteps, bool fusable, bool resume, int32_t src) {
  md_status rc = reserve_events(c, nsteps - k0);
  if (rc) return rc;
  bool fused = false;  // the step before
  for (int32_t k = k0; k < nsteps; ++k) {
    const bool res = resume && k == k0, kick = !res && !fused;
    fused = fuses(c, ta, k, nsteps, fusable);
    rc = enqueue_step(c, s, ta, thermo, k, energy_step(ta, k, nsteps - 1), kick, fused, res,
                      res ? src : -1);
    if (rc) return rc;
  }
  return MD_OK;
}

md_status reserve_events(md_ctx c, int32_t nsteps) {
  if (c->prof_every <= 0) return MD_OK;
  const size_t need = c->ev_used + 2 * (size_t)(nsteps / c->prof_every + 1);
  while (c->ev_pool.size() < need) {
    hipEvent_t e;
    HIPCHECK(c, hipEventCreate(&e));
    c->ev_pool.push_back(e);
  }
  return MD_OK;
}

void drop_graph(md_ctx c) {
  if (c->gexec) (void)hipGraphExecDestroy(c->gexec);
  c->gexec = nullptr;
}

// A graph of K steps, captured once per launch configuration and replayed:
// every argument is fixed, the step number lives in device counters.
md_status ensure_graph(md_ctx c, const ThermoArgs& ta, int32_t thermo, int32_t K) {
  const int64_t key[16] = {K, thermo, ta.ramp, ta.log_every, ta.nlog, (int64_t)(intptr_t)ta.log,
                           (int64_t)(intptr_t)c->nbr, (int64_t)(intptr_t)c->nbr16,
                           c->prof_every, c->prof_epoch, (int64_t)(intptr_t)c->pos,
                           c->cap, c->lcap_f, c->tpp, c->unroll, (int64_t)(intptr_t)c->ba.list};
  if (c->gexec && std::equal(key, key + 16, c->gkey)) return MD_OK;
  drop_graph(c);
  if (!c->cap_stream) HIPCHECK(c, hipStreamCreateWithFlags(&c->cap_stream, hipStreamNonBlocking));
  md_status rc = reserve_events(c, K);
  if (rc) return rc;
  HIPCHECK(c, hipStreamBeginCapture(c->cap_stream, hipStreamCaptureModeRelaxed));
  for (int32_t k = 0; k < K && rc == MD_OK; ++k)
    rc = enqueue_step(c, c->cap_stream, ta, thermo, k, energy_step_graph(ta, k, K));
  hipGraph_t g = nullptr;
  hipError_t e = hipStreamEndCapture(c->cap_stream, &g);
  if (rc) {
    if (g) (void)hipGraphDestroy(g);
    return rc;
  }
  if (e != hipSuccess) return fail(c, MD_EHIP, "graph capture failed");
  e = hipGraphInstantiate(&c->gexec, g, nullptr, nullptr, 0);
  (void)hipGraphDestroy(g);
  if (e != hipSuccess) {
    c->gexec = nullptr;
    return fail(c, MD_EHIP, "graph instantiation failed");
  }
  std::copy(key, key + 16, c->gkey);
  return MD_OK;
}

}  // namespace

extern "C" {

const char* md_last_error(md_ctx c) { return c ? c->err.c_str() : g_init_error.c_str(); }

md_status md_init(md_ctx* out, const md_params* p, int32_t nrep, const int64_t* n,
                  const double* L, void* hip_stream) {
  return md_init_alloc(out, p, nrep, n, L, hip_stream, nullptr);
}

md_status md_init_alloc(md_ctx* out, const md_params* p, int32_t nrep, const int64_t* n,
                        const double* L, void* hip_stream, const md_allocator* alloc) {
  if (!out) return fail(nullptr, MD_EINVAL, "out is NULL");
  if (alloc && (!alloc->alloc || !alloc->free))
    return fail(nullptr, MD_EINVAL, "allocator needs both alloc and free");
  *out = nullptr;
  std::string why;
  if (validate(p, &why)) return fail(nullptr, MD_EINVAL, why);
  if (nrep < 1 || !n || !L) return fail(nullptr, MD_EINVAL, "need nrep >= 1 and n, L arrays");
  const double rcmax = max_rc(*p);
  int64_t ntot = 0;
  for (int r = 0; r < nrep; ++r) {
    if (n[r] < 2) return fail(nullptr, MD_EINVAL, "every replica needs at least 2 particles");
    if (!std::isfinite(L[r]) || !(L[r] >= 2.0 * (rcmax + p->skin)))
      return fail(nullptr, MD_EBOX, "box side L must be >= 2 (max rc + skin)");
    ntot += n[r];
  }
  // list entries carry a 26-bit particle index; the list-free path keeps no
  // list and indexes particles with 32-bit integers
  if (p->path != MD_PATH_CELLS && ntot > (int64_t)kIdxMask + 1)
    return fail(nullptr, MD_EINVAL,
                "total particle count must be <= 2^26 on the list paths (the list-free "
                "path takes up to 2^30)");
  // SoA components are addressed as stride + i in 32-bit arithmetic
  if (ntot > (int64_t)1 << 30)
    return fail(nullptr, MD_EINVAL, "total particle count must be <= 2^30");

  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return fail(nullptr, MD_EHIP, "hipGetDevice failed");
  {
    const hipError_t e = scratch_setup(dev);
    if (e != hipSuccess)
      return fail(nullptr, MD_EHIP,
                  std::string("hipGetSymbolAddress(scratch) failed: ") + hipGetErrorString(e));
  }
  md_ctx c = new md_ctx_s();
  c->p = *p;
  c->device = dev;
  c->nrep = nrep;
  c->ntot = (int32_t)ntot;
  c->stride = (int32_t)(((ntot + 63) / 64) * 64);
  c->mixed = p->precision == MD_MIXED;
  c->tpp = p->tpp == 0 ? 2 : p->tpp;
  c->unroll = p->unroll == 0 ? 4 : p->unroll;
  c->stream = (hipStream_t)hip_stream;
  if (alloc) c->alloc = *alloc;
  for (int r = 0; r < nrep; ++r) c->nmax_rep = std::max<int32_t>(c->nmax_rep, (int32_t)n[r]);

  // replica geometry: cells of side >= max rc + skin (nc < 3 -> one cell)
  const double side = rcmax + p->skin;
  int32_t off = 0, coff = 0, tile = 0;
  double rho_max = 0.0;
  for (int r = 0; r < nrep; ++r) {
    RepDesc d{};
    int32_t nc = (int32_t)std::floor(L[r] / side);
    if (nc < 3) nc = 1;
    d.L = L[r];
    d.inv_cell = (double)nc / L[r];
    d.half_skin2 = (0.5 * p->skin) * (0.5 * p->skin);
    d.dof = 3.0 * (double)n[r] - 3.0;
    d.volume = L[r] * L[r] * L[r];
    d.cside = L[r] / nc;
    // mixed records: the largest power of two scale s.t. half a cell side
    // plus the skin plus one unit of drift stays below 2^30 fixed-point units
    d.qs = 1.0;
    while ((0.5 * d.cside + p->skin + 1.0) * (2.0 * d.qs) <= 1073741824.0) d.qs *= 2.0;
    d.qinv = 1.0 / d.qs;
    d.off = off;
    d.n = (int32_t)n[r];
    d.coff = coff;
    d.nc = nc;
    d.tile0 = tile;
    for (int32_t s0 = off; s0 < off + d.n; s0 += kTile) {
      Tile t{};
      t.rep = r;
      t.start = s0;
      t.end = std::min(s0 + kTile, off + d.n);
      c->tiles_h.push_back(t);
      ++tile;
    }
    d.tile1 = tile;
    c->reps_h.push_back(d);
    off += d.n;
    int64_t cells = (int64_t)nc * nc * nc;
    if ((int64_t)coff + cells > (int64_t)0x7fffffff) {
      delete c;
      return fail(nullptr, MD_EINVAL, "too many cells");
    }
    coff += (int32_t)cells;
    rho_max = std::max(rho_max, (double)n[r] / d.volume);
  }
  c->ncells = coff;
  c->ntiles = tile;
  c->small_chain = p->small_box == 0 && nrep == 1 && ntot <= kSmallN && c->ncells <= kSmallCells;
  c->small_list = p->small_box == 0 && nrep == 1 && ntot <= kSmallListN;

  // kernel path: the staged path needs >= 3 cells per side in every replica
  bool all3 = true;
  for (const RepDesc& d : c->reps_h) {
    all3 = all3 && d.nc >= 3;
    if (d.nc != 1) c->any_multi = 1;
  }
  std::vector<Tile> tiles1;
  for (const Tile& t : c->tiles_h)
    if (c->reps_h[t.rep].nc == 1) tiles1.push_back(t);
  c->ntiles1 = (int32_t)tiles1.size();
  if ((p->path == MD_PATH_STAGED || p->path == MD_PATH_CELLS) && !all3) {
    delete c;
    return fail(nullptr, MD_EINVAL, "the staged and cell paths need >= 3 cells per box side");
  }
  c->staged = p->path == MD_PATH_STAGED;
  c->cells = p->path == MD_PATH_CELLS;
  if (c->mixed && !c->staged && !c->cells)
    for (const RepDesc& d : c->reps_h)
      if (d.nc > 1023) {
        delete c;
        return fail(nullptr, MD_EINVAL,
                    "mixed precision on the gather path supports up to 1023 cells per side");
      }
  if (p->max_neighbors > 0) {
    c->cap = p->max_neighbors;
  } else {
    const double expect = rho_max * 4.0 / 3.0 * M_PI * side * side * side;
    c->cap = (int32_t)(((int64_t)std::ceil(1.5 * expect) + 16 + 7) / 8 * 8);
  }
  int32_t lds_max = 65536;
  {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) == hipSuccess &&
        v > 0)
      lds_max = v;
    (void)hipGetLastError();
    lds_max = std::min(lds_max, 65536);  // stay within the default per-block limit
  }
  if (c->staged || c->cells) {
    if (c->staged && c->tpp == 8) {
      delete c;
      return fail(nullptr, MD_EINVAL, "the staged path takes tpp 1, 2 or 4");
    }
    // row tiles of about 128 home particles; on the staged path LDS holds the
    // tile's 9 x (nx + 2) cells with 30 % headroom (denser tiles spill to
    // global memory)
    const int32_t homes = c->cells ? cells_homes_per_block() : staged_homes_per_group();
    double need = 0.0;
    for (int r = 0; r < nrep; ++r) {
      RepDesc& d = c->reps_h[r];
      const int32_t nc = d.nc;
      const double ppc = (double)d.n / ((double)nc * nc * nc);
      int32_t cpt = p->tile_cells;
      if (cpt <= 0) cpt = (int32_t)std::floor(0.85 * homes / ppc);
      cpt = std::max(1, std::min(cpt, std::min(nc, (int32_t)kMaxRowCells)));
      const int32_t ntr = (nc + cpt - 1) / cpt;
      d.fb0 = (int32_t)c->rtiles_h.size();
      int32_t nxmax = 0;
      for (int32_t row = 0; row < nc * nc; ++row)
        for (int32_t t = 0; t < ntr; ++t) {
          RowTile rt{};
          rt.rep = r;
          rt.row = row;
          rt.a = (int32_t)((int64_t)t * nc / ntr);
          rt.nx = (int32_t)((int64_t)(t + 1) * nc / ntr) - rt.a;
          nxmax = std::max(nxmax, rt.nx);
          c->rtiles_h.push_back(rt);
        }
      d.fb1 = (int32_t)c->rtiles_h.size();
      need = std::max(need, 9.0 * (nxmax + 2) * ppc);
    }
    c->nrt = (int32_t)c->rtiles_h.size();
    const int32_t want = (int32_t)((int64_t)std::ceil(1.3 * need + 64) / 64 * 64);
    const int32_t room = lds_max - 8192;  // static LDS of the kernel
    c->lcap_f = std::max(64, std::min(want, (int32_t)(room / 24)));
    if (p->stage_slots > 0) c->lcap_f = std::min(c->lcap_f, p->stage_slots);
    if (c->cells) plan_bricks(c);
  } else if (plan_bricks(c)) {
    // lanes per particle: four fill the chip sooner (per NVE launch 32,000
    // particles FP64 24 us against 33 with two, 131,072: 42 us both), two
    // walk large boxes faster (1,048,576: 202 against 223 us, mixed 146
    // against 184); results do not depend on it
    c->tpp = ntot < 200000 ? 4 : 2;
    c->unroll = kChunkEntries / c->tpp;
  } else {
    gather_blocks(c);
  }
  // pair table: shift constants of Eq. (3) computed on the host in FP64
  PairTab tab{};
  for (int a = 0; a < MD_MAXT; ++a)
    for (int b = 0; b < MD_MAXT; ++b) {
      const int ab = a * MD_MAXT + b;
      if (a >= p->ntypes || b >= p->ntypes) {
        tab.rc2[ab] = 0.0;  // never used
        tab.thr[ab] = 0.0;
        tab.sig2[ab] = 1.0;
        continue;
      }
      const double rc = p->rc[ab];
      const double t = rc + p->skin;
      tab.rc2[ab] = rc * rc;
      tab.thr[ab] = t * t;
      tab.sig2[ab] = p->sig[ab] * p->sig[ab];
      const double e = p->eps[ab];
      tab.c12[ab] = 4.0 * e;
      tab.c6[ab] = p->potential == MD_POT_SOFT ? 0.0 : -4.0 * e;
      tab.f12[ab] = 48.0 * e;
      tab.f6[ab] = p->potential == MD_POT_SOFT ? 0.0 : -24.0 * e;
      double vc, dvc;
      plain_v(*p, ab, rc, &vc, &dvc);
      tab.vc[ab] = vc;
      tab.fs[ab] = p->trunc == MD_TRUNC_SHIFTED_FORCE ? dvc : 0.0;
      tab.rc[ab] = rc;
    }
  for (int a = 0; a < MD_MAXT; ++a) {
    tab.mass[a] = a < p->ntypes ? p->mass[a] : 1.0;
    tab.inv_mass[a] = 1.0 / tab.mass[a];
  }
  if (c->brick || c->search) c->bp_h = brick_pair(*p, tab);
  c->thr_form = fma_pair_form(tab.thr, p->ntypes);
  c->rc2_form = fma_pair_form(tab.rc2, p->ntypes);

  std::vector<int32_t> cell_rep(c->ncells);
  for (int r = 0; r < nrep; ++r) {
    const RepDesc& d = c->reps_h[r];
    std::fill(cell_rep.begin() + d.coff, cell_rep.begin() + d.coff + d.nc * d.nc * d.nc, r);
  }

  const size_t N = c->ntot, S = c->stride;
  md_status rc = MD_OK;
#define ALLOC(ptr, count)                       \
  if ((rc = dalloc(c, &(ptr), (count))) != 0) { \
    std::string m_ = c->err;                    \
    md_destroy(c);                              \
    return fail(nullptr, rc, m_);               \
  }
  // Tables and counters: one allocation, and one copy of all the short ones.  A
  // copy and an allocation take about 10 us each: a context of 1,000, 16,384 or
  // 131,072 particles is made in 41, 66 or 235 us; 150, 176 or 346 with one of
  // each per table.
  struct Part {
    const void* src;  // nullptr: zeros
    size_t bytes, off;
    std::function<void(char*)> place;
  };
  std::vector<Part> parts;
  size_t total = 0;
  auto table = [&](auto& ptr, const void* src, size_t count) {
    using T = std::remove_reference_t<decltype(*ptr)>;
    if (!count) return;
    parts.push_back(Part{src, count * sizeof(T), total, [&ptr](char* p) { ptr = (T*)p; }});
    total += (count * sizeof(T) + 255) / 256 * 256;
  };
  std::vector<double> ones(nrep, 1.0);
  std::vector<int32_t> cell_tile;
  if (c->staged) {
    cell_tile.assign(c->ncells, 0);
    for (int32_t t = 0; t < c->nrt; ++t) {
      const RowTile& rt = c->rtiles_h[t];
      const RepDesc& d = c->reps_h[rt.rep];
      for (int32_t x = rt.a; x < rt.a + rt.nx; ++x) cell_tile[d.coff + rt.row * d.nc + x] = t;
    }
  }
  const size_t most_blocks =
      std::max({(size_t)c->ntiles * 8, (size_t)c->nrt, (size_t)c->brick_parts});
  plan_chunks(c);
  c->max_chunks = (int32_t)((most_blocks + kRedChunk - 1) / kRedChunk) + nrep;
  c->chunks_h.resize(c->max_chunks);  // what a later plan may need; the first nchunks are this one's
  table(c->reps, c->reps_h.data(), (size_t)nrep);
  table(c->tiles, c->tiles_h.data(), (size_t)c->ntiles);
  table(c->tiles1, tiles1.data(), tiles1.size());
  table(c->tab, &tab, 1);
  table(c->cell_rep, cell_rep.data(), (size_t)c->ncells);
  table(c->lam, ones.data(), (size_t)nrep);
  if (c->brick || c->search) {
    c->ba.capc = chunk_capacity(c, c->cap);
    table(c->ba.tiles, c->btiles_h.data(), (size_t)c->ba.ntiles);
    table(c->ba.bricks, c->bricks_h.data(), (size_t)c->ba.nbricks);
    table(c->bp, &c->bp_h, 1);
  }
  if (c->staged || c->cells) table(c->rtiles, c->rtiles_h.data(), (size_t)c->nrt);
  if (c->staged) table(c->cell_tile, cell_tile.data(), (size_t)c->ncells);
  table(c->chunks, c->chunks_h.data(), (size_t)c->max_chunks);
  table(c->st, nullptr, 1);
  table(c->rebuild, nullptr, (size_t)nrep);
  table(c->obs, nullptr, (size_t)nrep);
  table(c->kcall, nullptr, (size_t)nrep);
  table(c->dpend, nullptr, (size_t)nrep);
  table(c->therm, nullptr, 2 * (size_t)nrep);
  char* base = nullptr;
  ALLOC(base, total);
  for (const Part& q : parts) q.place(base + q.off);

  ALLOC(c->counts, (size_t)c->ncells);
  ALLOC(c->cell_start, (size_t)c->ncells + 1);
  ALLOC(c->bsum, scan_bsum_elems(c->ncells));
  ALLOC(c->cell_of, N);
  ALLOC(c->slot, N);
  ALLOC(c->tmp_src, N);
  ALLOC(c->pos, N);
  ALLOC(c->pos_tmp, N);
  ALLOC(c->vel, 3 * S);
  ALLOC(c->vel_tmp, 3 * S);
  ALLOC(c->xref, 3 * S);
  if (c->mixed) {
    float* f = nullptr;
    ALLOC(f, 3 * S);
    c->frc = f;
  } else {
    double* f = nullptr;
    ALLOC(f, 3 * S);
    c->frc = f;
  }
  ALLOC(c->id, N);
  ALLOC(c->id_tmp, N);
  ALLOC(c->img, 3 * N);
  if (c->brick || c->search) {
    ALLOC(c->ba.head, (size_t)c->ba.ntiles);
    ALLOC(c->ba.row, (size_t)c->ba.ntiles * c->ba.rows);
    ALLOC(c->ba.hrow, (size_t)c->ba.ntiles * c->ba.hrows);
  }
  if (c->brick) {
    ALLOC(c->ba.list, chunk_elems(c->ntot, c->ba.capc));
    ALLOC(c->ba.nchunk, N);
  } else if (c->staged) {
    ALLOC(c->nbr16, list_elems(c->ntot, c->cap));
  } else if (!c->cells) {
    ALLOC(c->nbr, list_elems(c->ntot, c->cap));
    if (c->mixed) {
      ALLOC(c->pos16, S);
      ALLOC(c->pos16_alt, S);
    }
  }
  if (!c->cells) ALLOC(c->ncount, N);  // list lengths (the list-free path has none)
  ALLOC(c->part, 4 * most_blocks);
  ALLOC(c->dmax, (size_t)c->ntiles);
  ALLOC(c->part2, (size_t)kPart2 * c->max_chunks);
#undef ALLOC
  // long tables are copied from where they are, the others from one block
  constexpr size_t kShort = 128 << 10;
  bool ok = hipMemset(c->counts, 0, sizeof(int32_t) * c->ncells) == hipSuccess &&
            hipMemset(c->frc, 0, (c->mixed ? 4 : 8) * 3 * S) == hipSuccess;
  std::vector<char> block;
  auto flush = [&](size_t end) {
    if (!block.empty())
      ok = ok && hipMemcpy(base + (end - block.size()), block.data(), block.size(),
                           hipMemcpyHostToDevice) == hipSuccess;
    block.clear();
  };
  for (const Part& q : parts) {
    const size_t padded = (q.bytes + 255) / 256 * 256;
    if (q.src && q.bytes > kShort) {
      flush(q.off);
      ok = ok && hipMemcpy(base + q.off, q.src, q.bytes, hipMemcpyHostToDevice) == hipSuccess;
      continue;
    }
    block.resize(block.size() + padded, 0);
    if (q.src) std::memcpy(block.data() + block.size() - padded, q.src, q.bytes);
  }
  flush(total);
  if (!ok) {
    md_destroy(c);
    return fail(nullptr, MD_EHIP, "uploading context tables failed");
  }
  *out = c;
  return MD_OK;
}

md_status md_destroy(md_ctx c) {
  if (!c) return MD_OK;
  (void)hipStreamSynchronize(c->stream);
  drop_graph(c);
  if (c->cap_stream) (void)hipStreamDestroy(c->cap_stream);
  for (hipEvent_t e : c->ev_pool) (void)hipEventDestroy(e);
  for (void* p : c->owned) {
    if (c->alloc.alloc)
      c->alloc.free(c->alloc.u, p, (void*)c->stream);
    else
      (void)hipFree(p);
  }
  c->owned.clear();
  delete c;
  return MD_OK;
}

md_status md_set_state(md_ctx c, const double* x, const double* v, const int32_t* type) {
  if (!c) return MD_EINVAL;
  if (!x || !v || !type) return fail(c, MD_EINVAL, "x, v and type are required");
  if (const md_status e = enter_tiles(c)) return e;
  launch_set_state(c->stream, c->ntot, c->stride, x, v, type, c->p.ntypes, c->pos, c->vel, c->id,
                   c->img, c->st);
  HIPCHECK(c, hipMemsetAsync(c->obs, 0, sizeof(md_obs) * c->nrep, c->stream));
  HIPCHECK(c, hipMemsetAsync(c->frc, 0, (c->mixed ? 4 : 8) * 3 * (size_t)c->stride, c->stream));
  md_status rc = sync_and_check(c);
  // positions are checked against the box at the first wrap
  c->has_state = rc == MD_OK;
  c->built = false;
  c->forces_valid = false;
  return rc;
}

md_status md_get_state(md_ctx c, double* x, double* v, int32_t* img) {
  if (!c) return MD_EINVAL;
  if (!c->has_state) return fail(c, MD_ESTATE, "no state set");
  if (x || v) launch_get_state(c->stream, c->ntot, c->stride, c->pos, c->vel, c->id, x, v);
  if (img)
    HIPCHECK(c, hipMemcpyAsync(img, c->img, sizeof(int32_t) * 3 * (size_t)c->ntot,
                               hipMemcpyDeviceToDevice, c->stream));
  return sync_and_check(c);
}

md_status md_build_cells(md_ctx c) {
  if (!c) return MD_EINVAL;
  if (!c->has_state) return fail(c, MD_ESTATE, "no state set");
  return build_all(c);
}

md_status md_forces(md_ctx c) {
  if (!c) return MD_EINVAL;
  if (!c->has_state) return fail(c, MD_ESTATE, "no state set");
  if (!c->built) {
    md_status rc = build_all(c);
    if (rc) return rc;
  }
  launch_forces0(c);
  c->forces_valid = true;
  return MD_OK;
}

md_status md_get_forces(md_ctx c, void* F) {
  if (!c) return MD_EINVAL;
  if (!F) return fail(c, MD_EINVAL, "F is NULL");
  if (!c->forces_valid) return fail(c, MD_ESTATE, "no forces computed");
  launch_get_forces(c->stream, c->ntot, c->stride, c->frc, c->mixed, c->id, F);
  return sync_and_check(c);
}

md_status md_step(md_ctx c, int32_t nsteps, const double* T0, const double* T1,
                  int64_t ramp_steps, md_obs* log, int32_t log_every) {
  if (!c) return MD_EINVAL;
  if (!c->has_state) return fail(c, MD_ESTATE, "no state set");
  if (nsteps < 0) return fail(c, MD_EINVAL, "nsteps must be >= 0");
  if (log && log_every <= 0) return fail(c, MD_EINVAL, "log needs log_every > 0");
  const int32_t thermo = T0 != nullptr;
  if (thermo) {
    for (int r = 0; r < c->nrep; ++r) {
      const double t1 = T1 ? T1[r] : T0[r];
      if (!(T0[r] > 0.0) || !(t1 > 0.0) || !std::isfinite(T0[r]) || !std::isfinite(t1))
        return fail(c, MD_EINVAL, "thermostat targets must be finite and > 0");
    }
  }
  c->last_thermo = thermo;
  if (!c->built) {
    md_status rc = build_all(c);
    if (rc) return rc;
  }
  if (!c->forces_valid) {
    launch_forces0(c);
    c->forces_valid = true;
  }
  ThermoArgs ta{};
  if (thermo) {
    std::vector<double> th(2 * c->nrep);
    for (int r = 0; r < c->nrep; ++r) {
      th[r] = T0[r];
      th[c->nrep + r] = T1 ? T1[r] : T0[r];
    }
    HIPCHECK(c, hipMemcpyAsync(c->therm, th.data(), sizeof(double) * th.size(),
                               hipMemcpyHostToDevice, c->stream));
    HIPCHECK(c, hipStreamSynchronize(c->stream));  // th is a local buffer
    ta.T0 = c->therm;
    ta.T1 = c->therm + c->nrep;
    ta.ramp = ramp_steps;
    ta.thermo = 1;
  }
  int64_t nlog = 0;
  if (log) {
    nlog = nsteps / log_every;
    if (nlog * c->nrep > c->log_cap) {
      dfree(c, c->log_dev);
      c->log_dev = nullptr;
      c->log_cap = 0;
      md_status rc = dalloc(c, &c->log_dev, (size_t)std::max<int64_t>(nlog * c->nrep, 1));
      if (rc) return rc;
      c->log_cap = nlog * c->nrep;
    }
    ta.log_every = log_every;
    ta.log = c->log_dev;
    ta.nlog = (int32_t)nlog;
  }
  hipStream_t s = c->stream;
  launch_begin_call(s, c->nrep, c->kcall, c->lam);
  int32_t k = 0;
  // events recorded inside a captured graph cannot be timed, so profiled
  // steps are launched directly
  const int32_t K = c->prof_every > 0 ? 0 : c->p.graph_steps;
  if (K > 0 && nsteps >= K) {
    md_status rc = ensure_graph(c, ta, thermo, K);
    if (rc) return rc;
    for (; k + K <= nsteps; k += K) HIPCHECK(c, hipGraphLaunch(c->gexec, s));
  }
  const int32_t kg = k;  // steps [0, kg) ran inside graph replays
  // the last step of a call is never fused: the state it leaves (positions,
  // velocities, forces) is complete
  bool fusable = can_fuse(c, thermo);
  md_status rc = enqueue_direct(c, s, ta, thermo, kg, nsteps, fusable, false, 0);
  if (rc) return rc;
  if (thermo) launch_apply_lambda(s, c->ntiles, c->tiles, c->stride, c->vel, c->lam, c->nrep, c->st);
  HIPCHECK(c, hipGetLastError());
  // a list build that overflowed halted the queued steps (kHalt): grow the
  // capacity, rebuild the interrupted step's lists on its state and finish
  // the call from there -- the trajectory of a context with enough capacity
  int32_t at = -1, src = 0;
  for (int attempt = 0;; ++attempt) {
    HIPCHECK(c, hipStreamSynchronize(s));
    DevState st{};
    HIPCHECK(c, hipMemcpy(&st, c->st, sizeof(DevState), hipMemcpyDeviceToHost));
    const int32_t mend = kErrOverflow | (c->brick || c->search ? kErrSlots : 0);
    if (!(st.err & mend) || (st.err & ~mend) || attempt == 8) break;
    int64_t done = 0;
    HIPCHECK(c, hipMemcpy(&done, c->kcall, sizeof(int64_t), hipMemcpyDeviceToHost));
    // how the interrupted step was queued: its kick by the step before or by
    // itself; one that is interrupted again was queued as before
    if ((int32_t)done != at)
      src = (int32_t)done > kg && fuses(c, ta, (int32_t)done - 1, nsteps, fusable) ? 1 : 0;
    at = (int32_t)done;
    if (st.err & kErrSlots) {
      rc = c->brick ? leave_brick(c) : leave_search(c);
    } else {
      rc = grow_capacity(c);
    }
    if (rc) {
      c->built = false;
      c->forces_valid = false;
      const DevState z{};  // reported by this call
      HIPCHECK(c, hipMemcpy(c->st, &z, sizeof(DevState), hipMemcpyHostToDevice));
      return rc;
    }
    st.err = 0;
    st.any_rebuild = 1;  // the interrupted step's rebuild flags are still set
    HIPCHECK(c, hipMemcpy(c->st, &st, sizeof(DevState), hipMemcpyHostToDevice));
    // the kernels that a context goes on with may not fuse (row tiles)
    fusable = can_fuse(c, thermo);
    rc = enqueue_direct(c, s, ta, thermo, at, nsteps, fusable, true, src);
    if (rc) return rc;
    if (thermo)
      launch_apply_lambda(s, c->ntiles, c->tiles, c->stride, c->vel, c->lam, c->nrep, c->st);
    HIPCHECK(c, hipGetLastError());
  }
  rc = sync_and_check(c);
  if (rc == MD_EOVERFLOW) {
    // not recoverable by growing the list (staged tile slots, or repeated
    // growth): the state is the interrupted step's
    c->built = false;
    c->forces_valid = false;
    return rc;
  }
  if (rc) return rc;
  if (log && nlog > 0)
    HIPCHECK(c, hipMemcpy(log, c->log_dev, sizeof(md_obs) * nlog * c->nrep,
                          hipMemcpyDeviceToHost));
  return MD_OK;
}

md_status md_observables(md_ctx c, md_obs* out) {
  if (!c) return MD_EINVAL;
  if (!out) return fail(c, MD_EINVAL, "out is NULL");
  md_status rc = sync_and_check(c);
  if (rc) return rc;
  HIPCHECK(c, hipMemcpy(out, c->obs, sizeof(md_obs) * c->nrep, hipMemcpyDeviceToHost));
  return MD_OK;
}

md_status md_get_cells(md_ctx c, int32_t rep, int32_t* cell_start, int32_t* order_ids) {
  if (!c) return MD_EINVAL;
  if (rep < 0 || rep >= c->nrep) return fail(c, MD_EINVAL, "replica index out of range");
  if (!c->built) return fail(c, MD_ESTATE, "cells not built");
  md_status rc = sync_and_check(c);
  if (rc) return rc;
  const RepDesc& d = c->reps_h[rep];
  const int64_t ncell = (int64_t)d.nc * d.nc * d.nc;
  if (cell_start) {
    HIPCHECK(c, hipMemcpy(cell_start, c->cell_start + d.coff, sizeof(int32_t) * (ncell + 1),
                          hipMemcpyDeviceToHost));
    for (int64_t k = 0; k <= ncell; ++k) cell_start[k] -= d.off;
  }
  if (order_ids) {
    HIPCHECK(c, hipMemcpy(order_ids, c->id + d.off, sizeof(int32_t) * d.n,
                          hipMemcpyDeviceToHost));
    for (int32_t k = 0; k < d.n; ++k) order_ids[k] -= d.off;
  }
  return MD_OK;
}

md_status md_get_neighbors(md_ctx c, int32_t rep, int32_t* count, int32_t* ids, int32_t cap) {
  if (!c) return MD_EINVAL;
  if (c->cells) return fail(c, MD_ESTATE, "the cell path keeps no neighbour list");
  if (rep < 0 || rep >= c->nrep) return fail(c, MD_EINVAL, "replica index out of range");
  if (!c->built) return fail(c, MD_ESTATE, "list not built");
  if (!count || (cap > 0 && !ids) || cap < 0) return fail(c, MD_EINVAL, "bad output buffers");
  md_status rc = sync_and_check(c);
  if (rc) return rc;
  const RepDesc& d = c->reps_h[rep];
  std::vector<int32_t> cnt(d.n), idv(c->ntot);
  HIPCHECK(c, hipMemcpy(cnt.data(), c->ncount + d.off, sizeof(int32_t) * d.n,
                        hipMemcpyDeviceToHost));
  HIPCHECK(c, hipMemcpy(idv.data(), c->id, sizeof(int32_t) * c->ntot, hipMemcpyDeviceToHost));
  // the list slices that hold the replica's particles, one contiguous block
  // (decoded from the tiles: as many entries as a row there can have)
  const int32_t lcap = c->brick ? std::min(c->cap, c->ba.capc * kChunkEntries) : c->cap;
  const int32_t s0 = (int32_t)(d.off / kSlice), s1 = (int32_t)((d.off + d.n - 1) / kSlice);
  const size_t lo = (size_t)s0 * kSlice * lcap, nel = (size_t)(s1 - s0 + 1) * kSlice * lcap;
  std::vector<uint32_t> sl(cap > 0 && d.n > 0 ? nel : 1);
  if (cap > 0 && d.n > 0) {
    const uint32_t* src = c->nbr;
    uint32_t* tmp = nullptr;
    if (c->brick) {
      md_status a_rc = dalloc(c, &tmp, list_elems(c->ntot, lcap));
      if (a_rc) return a_rc;
      launch_decode_brick(c->stream, c->ba, lcap, c->ncount, tmp);
      HIPCHECK(c, hipStreamSynchronize(c->stream));
      src = tmp;
    } else if (c->staged) {
      // staged entries are LDS slots of the home tile: decode to particle indices
      md_status a_rc = dalloc(c, &tmp, list_elems(c->ntot, c->cap));
      if (a_rc) return a_rc;
      launch_decode_staged(c->stream, c->nrt, c->rtiles, c->reps, c->cell_start, c->cap,
                           c->nbr16, c->ncount, tmp);
      src = tmp;
    }
    hipError_t e = hipMemcpy(sl.data(), src + lo, sizeof(uint32_t) * nel, hipMemcpyDeviceToHost);
    if (tmp) dfree(c, tmp);
    if (e != hipSuccess) return fail(c, MD_EHIP, "copying the neighbour list failed");
  }
  for (int32_t i = 0; i < d.n; ++i) {
    const int32_t g = (int32_t)d.off + i;
    const int32_t orig = idv[g] - d.off;
    count[orig] = cnt[i];
    const int32_t m = std::min(std::min(cnt[i], lcap), cap);
    const size_t b = list_base(g, lcap) - lo;
    for (int32_t k = 0; k < m; ++k) {
      const uint32_t e = sl[b + (size_t)k * kSlice];
      ids[(size_t)orig * cap + k] = idv[e & kIdxMask] - d.off;
    }
  }
  return MD_OK;
}

md_status md_replica_info(md_ctx c, int32_t rep, int32_t* nc, double* inv_cell, int64_t* n,
                          int64_t* offset, int32_t* max_neighbors) {
  if (!c) return MD_EINVAL;
  if (rep < 0 || rep >= c->nrep) return fail(c, MD_EINVAL, "replica index out of range");
  const RepDesc& d = c->reps_h[rep];
  if (nc) *nc = d.nc;
  if (inv_cell) *inv_cell = d.inv_cell;
  if (n) *n = d.n;
  if (offset) *offset = d.off;
  if (max_neighbors) *max_neighbors = c->cap;
  return MD_OK;
}

md_status md_profile(md_ctx c, int32_t every) {
  if (!c) return MD_EINVAL;
  if (every < 0) return fail(c, MD_EINVAL, "every must be >= 0");
  HIPCHECK(c, hipStreamSynchronize(c->stream));
  c->prof_every = every;
  c->ev_used = 0;
  c->prof_epoch += 1;  // captured graphs hold events of the previous setting
  return MD_OK;
}

md_status md_profile_read(md_ctx c, md_prof* out) {
  if (!c) return MD_EINVAL;
  if (!out) return fail(c, MD_EINVAL, "out is NULL");
  HIPCHECK(c, hipStreamSynchronize(c->stream));
  out->force_launches = (int64_t)(c->ev_used / 2);
  out->force_ms = 0.0;
  for (size_t k = 0; k + 1 < c->ev_used; k += 2) {
    float ms = 0.0f;
    HIPCHECK(c, hipEventElapsedTime(&ms, c->ev_pool[k], c->ev_pool[k + 1]));
    out->force_ms += ms;
  }
  return MD_OK;
}

md_status md_autotune(md_ctx c, int32_t reps, md_tune* out) {
  if (!c) return MD_EINVAL;
  if (!out || reps < 1) return fail(c, MD_EINVAL, "need out and reps >= 1");
  if (!c->has_state) return fail(c, MD_ESTATE, "no state set");
  if (!c->built) {
    md_status rc = build_all(c);
    if (rc) return rc;
  }
  std::vector<std::pair<int32_t, int32_t>> cand;
  if (c->cells)
    cand = {{1, 1}};  // one kernel variant: nothing to choose
  else if (c->brick)
    cand = {{2, 4}, {4, 2}};  // lanes per particle, entries of a chunk per lane
  else if (c->staged)
    cand = {{1, 4}, {1, 8}, {2, 2}, {2, 4}, {2, 8}, {4, 2}};
  else
    cand = {{1, 4}, {1, 8}, {2, 2}, {2, 4}, {4, 1}, {4, 2}, {8, 1}};
  hipEvent_t e0, e1;
  HIPCHECK(c, hipEventCreate(&e0));
  HIPCHECK(c, hipEventCreate(&e1));
  *out = md_tune{};
  double best = 1e300;
  int32_t btpp = c->tpp, bun = c->unroll;
  // the form that the steps run (their registers differ): without energies, and
  // fused with the next kick where directly launched NVE steps are; its
  // velocities and positions go to the scratch of the rebuild chain.  A context
  // that last stepped under the thermostat is tuned for such steps (soft
  // spheres, 1,048,576: the fused form chose a variant of 61 us, 58 this way).
  const int32_t mode = can_fuse(c, c->last_thermo) && c->p.graph_steps == 0 ? 2 : 1;
  double* const vel = c->vel;
  auto timed = [&](float* ms) {
    c->vel = c->vel_tmp;
    launch_forces(c, mode, c->stream, 0);  // warm
    (void)hipEventRecord(e0, c->stream);
    for (int r = 0; r < reps; ++r) launch_forces(c, mode, c->stream, 0);
    (void)hipEventRecord(e1, c->stream);
    c->vel = vel;
    const hipError_t e = hipEventSynchronize(e1);
    return e == hipSuccess ? hipEventElapsedTime(ms, e0, e1) : e;
  };
  for (auto& tu : cand) {
    c->tpp = tu.first;
    c->unroll = tu.second;
    float ms = 0.0f;
    HIPCHECK(c, timed(&ms));
    const double avg = ms / reps;
    if (out->ntried < 16) {
      out->tried_tpp[out->ntried] = tu.first;
      out->tried_unroll[out->ntried] = tu.second;
      out->tried_ms[out->ntried] = avg;
      out->ntried += 1;
    }
    if (avg < best) {
      best = avg;
      btpp = tu.first;
      bun = tu.second;
    }
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  c->tpp = btpp;
  c->unroll = bun;
  if (!c->brick && !c->staged && !c->cells) {
    // partial-sum blocks per replica follow the lanes per particle
    gather_blocks(c);
    md_status rc = upload_blocks(c);
    if (rc) return rc;
  }
  drop_graph(c);
  launch_forces0(c);
  c->forces_valid = true;
  out->tpp = btpp;
  out->unroll = bun;
  out->force_ms = best;
  return sync_and_check(c);
}

md_status md_msd_reference(md_ctx c) {
  if (!c) return MD_EINVAL;
  if (!c->has_state) return fail(c, MD_ESTATE, "no state set");
  if (!c->u0) {
    md_status rc = dalloc(c, &c->u0, 3 * (size_t)c->ntot);
    if (!rc) rc = dalloc(c, &c->msd_part, (size_t)c->ntiles);
    if (!rc) rc = dalloc(c, &c->msd_out, (size_t)c->nrep);
    if (rc) return rc;
  }
  launch_msd_ref(c->stream, c->ntiles, c->tiles, c->reps, c->pos, c->id, c->img, c->u0);
  return sync_and_check(c);
}

md_status md_msd(md_ctx c, double* out) {
  if (!c) return MD_EINVAL;
  if (!out) return fail(c, MD_EINVAL, "out is NULL");
  if (!c->u0) return fail(c, MD_ESTATE, "no MSD reference set");
  launch_msd(c->stream, c->ntiles, c->nrep, c->tiles, c->reps, c->pos, c->id, c->img, c->u0,
             c->msd_part, c->msd_out);
  md_status rc = sync_and_check(c);
  if (rc) return rc;
  HIPCHECK(c, hipMemcpy(out, c->msd_out, sizeof(double) * c->nrep, hipMemcpyDeviceToHost));
  return MD_OK;
}

namespace {
// g(r) of replica rep into g (HOST [nbins]) from the pair histogram hist
// (DEVICE, >= nbins counters, cleared here).  The counts are copied into g's
// own storage (8 bytes each) and normalised in place.  may_build: build the
// cells first when the cell sweep needs them.
md_status rdf_with(md_ctx c, int32_t rep, double rmax, int32_t nbins, double* g,
                   unsigned long long* hist, bool may_build) {
  const RepDesc& d = c->reps_h[rep];
  // the cell sweep covers every pair closer than the cell side minus the
  // skin while the skin rule holds; otherwise all pairs are visited
  const bool by_cells = d.nc >= 3 && rmax <= d.L / d.nc - c->p.skin;
  if (!by_cells && d.n > 262144)
    return fail(c, MD_EINVAL,
                "md_rdf: rmax above the cell side minus the skin needs a replica of at most "
                "262144 particles");
  if (by_cells && !c->built) {
    if (!may_build) return fail(c, MD_ESTATE, "md_rdf_static: cells not built");
    md_status b = build_all(c);
    if (b) return b;
  }
  // Longer ranges take more cells to each side while these are distinct
  // (2 h + 1 <= nc) and built; the number of pairs tested then follows the
  // range instead of the box.  Unbuilt cells are not built for it: that call
  // keeps visiting all pairs.  (The margin covers rounding in the cell of a
  // particle, as the skin test does for h = 1.)
  int32_t h = by_cells ? 1 : 0;
  if (!by_cells && c->built)
    for (int32_t q = 2; 2 * q + 1 <= d.nc && !h; ++q)
      if (rmax <= (q * (d.L / d.nc) - c->p.skin) * (1.0 - 1e-12)) h = q;
  launch_zero_u64(c->stream, hist, nbins);
  if (h)
    launch_rdf_cells(c->stream, d.coff, d.nc, h, c->cell_start, c->pos, d.L, c->p.skin, rmax,
                     nbins, hist);
  else
    launch_rdf(c->stream, c->pos, d.off, d.n, d.L, rmax, nbins, hist);
  HIPCHECK(c, hipGetLastError());
  md_status rc = sync_and_check(c);
  if (rc) return rc;
  HIPCHECK(c, hipMemcpy(g, hist, sizeof(unsigned long long) * nbins, hipMemcpyDeviceToHost));
  const double dr = rmax / nbins, V = d.L * d.L * d.L, n = (double)d.n;
  const double pi = 3.14159265358979323846;
  for (int32_t b = 0; b < nbins; ++b) {
    unsigned long long h;
    std::memcpy(&h, &g[b], sizeof h);
    const double r0 = b * dr, r1 = (b + 1) * dr;
    const double shell = 4.0 / 3.0 * pi * (r1 * r1 * r1 - r0 * r0 * r0);
    g[b] = 2.0 * V * (double)h / (n * n * shell);
  }
  return MD_OK;
}

md_status rdf_args(md_ctx c, int32_t rep, double rmax, int32_t nbins, const double* g) {
  if (rep < 0 || rep >= c->nrep) return fail(c, MD_EINVAL, "replica index out of range");
  if (!c->has_state) return fail(c, MD_ESTATE, "no state set");
  const RepDesc& d = c->reps_h[rep];
  if (!g || nbins < 1 || nbins > kStaticBins || !(rmax > 0.0) || rmax > 0.5 * d.L)
    return fail(c, MD_EINVAL, "need g, 1 <= nbins <= 8192 and 0 < rmax <= L/2");
  return MD_OK;
}
}  // namespace

md_status md_rdf(md_ctx c, int32_t rep, double rmax, int32_t nbins, double* g) {
  if (!c) return MD_EINVAL;
  md_status rc = rdf_args(c, rep, rmax, nbins, g);
  if (rc) return rc;
  if (!c->rdf_hist) {  // 64 KiB, kept: an allocation and its release cost more than the counts
    rc = dalloc(c, &c->rdf_hist, (size_t)kStaticBins);
    if (rc) return rc;
  }
  return rdf_with(c, rep, rmax, nbins, g, c->rdf_hist, true);
}

md_status md_rdf_static(md_ctx c, int32_t rep, double rmax, int32_t nbins, double* g) {
  if (!c) return MD_EINVAL;
  md_status rc = rdf_args(c, rep, rmax, nbins, g);
  if (rc) return rc;
  unsigned long long* hist = scratch_dev(c->device);
  if (!hist) return fail(c, MD_EHIP, "md_rdf_static: no scratch address for this device");
  return rdf_with(c, rep, rmax, nbins, g, hist, false);
}

md_status md_list_stats(md_ctx c, int32_t rep, double* mean, int32_t* max) {
  if (!c) return MD_EINVAL;
  if (c->cells) return fail(c, MD_ESTATE, "the cell path keeps no neighbour list");
  if (rep < -1 || rep >= c->nrep) return fail(c, MD_EINVAL, "replica index out of range");
  if (!c->built) return fail(c, MD_ESTATE, "list not built");
  md_status rc = sync_and_check(c);
  if (rc) return rc;
  const int32_t off = rep < 0 ? 0 : c->reps_h[rep].off;
  const int32_t n = rep < 0 ? c->ntot : c->reps_h[rep].n;
  std::vector<int32_t> cnt(n);
  HIPCHECK(c, hipMemcpy(cnt.data(), c->ncount + off, sizeof(int32_t) * n, hipMemcpyDeviceToHost));
  int64_t sum = 0;
  int32_t m = 0;
  for (int32_t v : cnt) {
    sum += v;
    m = std::max(m, v);
  }
  if (mean) *mean = (double)sum / (double)n;
  if (max) *max = m;
  return MD_OK;
}

}  // extern "C"
