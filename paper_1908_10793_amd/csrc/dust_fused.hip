// Fused tile step: plan (tile table), the dispatcher over geometries and the
// partial reduction, and the rebinning kernels (half-step keys and packing,
// level-major permutation).  The kernels themselves are in
// dust_fused_kern.h.
#include <algorithm>
#include <vector>

#include "dust_cells_kern.h"
#include "dust_fused_kern.h"

namespace dust {

// Workgroups of the particle-per-lane kernel that the chip holds at once (its
// LDS: three on each of 256 CUs, two with FP64 arithmetic).
static constexpr int CELLS_BLOCKS = 768, CELLS_BLOCKS_F64 = 512;


// Supported tile shapes (cells per axis, 256 cells each).
struct Shape3 { int x, y, z; };
static const Shape3 kShapes3[] = {{8, 8, 4}, {16, 4, 4}, {4, 16, 4}, {4, 4, 16}, {8, 4, 8}, {4, 8, 8}};
static const Shape3 kShapes2[] = {{16, 16, 1}, {32, 8, 1}, {8, 32, 1}};

static int shape_id(int ndim, TileShape t) {
  if (ndim > 2) {
    for (int s = 0; s < 6; ++s)
      if (kShapes3[s].x == t.t[0] && kShapes3[s].y == t.t[1] && kShapes3[s].z == t.t[2]) return s;
  } else {
    for (int s = 0; s < 3; ++s)
      if (kShapes2[s].x == t.t[0] && kShapes2[s].y == t.t[1]) return s;
  }
  return -1;
}

dust_status_t fused_plan_init(FusedPlan& plan, const Box* boxes, int nbox, TileShape tile, int slack) {
  (void)slack;
  fused_plan_free(plan);
  plan.tile = tile;
  plan.halo = FUSED_HALO;
  if (nbox < 1) return DUST_EINVAL;
  int ndim = boxes[0].ndim;
  if (ndim == 2) plan.tile.t[2] = 1;
  plan.shape = shape_id(ndim, plan.tile);
  if (plan.shape < 0) return DUST_EUNSUPPORTED;
  std::vector<TileDesc> tiles;
  plan.small = plan.tsc = true;
  for (int b = 0; b < nbox; ++b) {
    const Box& B = boxes[b];
    if (B.ncell >= (1 << 24)) plan.small = false;
    for (int d = 0; d < B.ndim; ++d)
      if (B.ax[d].shape != SHAPE_TSC) plan.tsc = false;
    int n[3] = {B.ax[0].n, B.ax[1].n, B.ndim > 2 ? B.ax[2].n : 1};
    int t[3] = {plan.tile.t[0], plan.tile.t[1], B.ndim > 2 ? plan.tile.t[2] : 1};
    int nt[3];
    for (int d = 0; d < 3; ++d) nt[d] = (n[d] + t[d] - 1) / t[d];
    int64_t key = B.cell_base;
    for (int tk = 0; tk < nt[2]; ++tk)
      for (int tj = 0; tj < nt[1]; ++tj)
        for (int ti = 0; ti < nt[0]; ++ti) {
          TileDesc d{};
          d.box = b;
          d.i0 = ti * t[0];
          d.j0 = tj * t[1];
          d.k0 = tk * t[2];
          d.ex = std::min(t[0], n[0] - d.i0);
          d.ey = std::min(t[1], n[1] - d.j0);
          d.ez = std::min(t[2], n[2] - d.k0);
          d.key0 = key;
          key += (int64_t)d.ex * d.ey * d.ez;
          tiles.push_back(d);
        }
  }
  int h2 = 2 * FUSED_HALO;
  plan.rmax[0] = plan.tile.t[0] + h2;
  plan.rmax[1] = plan.tile.t[1] + h2;
  plan.rmax[2] = ndim > 2 ? plan.tile.t[2] + h2 : 1;
  plan.lds_cells = (size_t)plan.rmax[0] * plan.rmax[1] * plan.rmax[2];
  plan.ntiles = (int)tiles.size();
  if (hipMalloc((void**)&plan.tiles_d, sizeof(TileDesc) * tiles.size()) != hipSuccess)
    return DUST_ENOMEM;
  if (hipMemcpy(plan.tiles_d, tiles.data(), sizeof(TileDesc) * tiles.size(), hipMemcpyHostToDevice) !=
      hipSuccess)
    return DUST_EDEVICE;
  if (hipMalloc((void**)&plan.part_d, sizeof(double) * PART_WORDS * (tiles.size() + CELLS_BLOCKS + DEFER_BLOCKS)) !=
          hipSuccess ||
      hipMalloc((void**)&plan.tile_map, 256 * tiles.size()) != hipSuccess ||
      hipMalloc((void**)&plan.defer_count, 256) != hipSuccess)
    return DUST_ENOMEM;
  if (hipMemset(plan.defer_count, 0, 256) != hipSuccess) return DUST_EDEVICE;
  plan.ok = true;
  return DUST_OK;
}

void fused_plan_free(FusedPlan& plan) {
  if (plan.tiles_d) (void)hipFree(plan.tiles_d);
  if (plan.part_d) (void)hipFree(plan.part_d);
  if (plan.defer_count) (void)hipFree(plan.defer_count);
  if (plan.defer_list) (void)hipFree(plan.defer_list);
  if (plan.tile_map) (void)hipFree(plan.tile_map);
  plan.tile_map = nullptr;
  plan.tiles_d = nullptr;
  plan.part_d = nullptr;
  plan.defer_count = nullptr;
  plan.defer_list = nullptr;
  plan.defer_cap = 0;
  plan.ok = false;
  plan.ntiles = 0;
}

// LDS of one workgroup: the FP64 deposit window ((nc+1) channels, padded to
// 32 bytes), then the gas window as one 4-vector of the storage type per cell
// (a single 16- or 32-byte LDS read gives every component of a cell).
static size_t fused_dep_doubles(size_t cells, int nc) { return (cells * (nc + 1) + 3) & ~(size_t)3; }

dust_status_t fused_plan_reserve(FusedPlan& plan, int64_t n) {
  if ((size_t)n <= plan.defer_cap && plan.defer_list) return DUST_OK;
  if (plan.defer_list) (void)hipFree(plan.defer_list);
  plan.defer_list = nullptr;
  plan.defer_cap = 0;
  size_t cap = (size_t)std::max<int64_t>(n, 1);
  if (hipMalloc((void**)&plan.defer_list, cap * sizeof(uint32_t)) != hipSuccess) return DUST_ENOMEM;
  plan.defer_cap = cap;
  return DUST_OK;
}

size_t fused_lds_bytes(const FusedPlan& plan, int nc, int ts_bytes) {
  return fused_dep_doubles(plan.lds_cells, nc) * sizeof(double) + plan.lds_cells * 4 * (size_t)ts_bytes;
}

// A fused launch's end in a launch of its own (see FusedEnd).
static constexpr int REDUCE_THREADS = 1024;
static constexpr int REDUCE_TAIL_BLOCKS = 31;
template <typename TS>
__global__ void __launch_bounds__(REDUCE_THREADS) k_fused_end(FusedEnd<TS> fe) {
  fused_end_block<TS, REDUCE_THREADS>(fe, blockIdx.x);
}

DUST_FUSED_G_ALL(extern, float, double)
DUST_FUSED_G_ALL(extern, float, float)
DUST_FUSED_G_ALL(extern, double, double)
DUST_CELLS_ALL(extern, float, double)
DUST_CELLS_ALL(extern, float, float)
DUST_CELLS_ALL(extern, double, double)


template <typename TS, typename A>
void launch_fused(const FusedPlan& plan, const PView<TS>& p, const FusedMove<TS>& mv, const Box* boxes_d, int nbox, int geom, int ndim, int unif, const FView<TS>& fl,
                  const Forces& f, const Species* sp, int drag_mode, double dt, const double* tdev,
                  const int64_t* bin_start, const double* xg, DiagDev* dg, bool sums, FusedEnd<TS>& fe,
                  hipEvent_t ev0, hipEvent_t ev1, hipStream_t st) {
  if (plan.ntiles == 0) return;
  double* part = plan.part_d;
  // (the deferred-particle count is zero here: set at set-up, and reset by
  // the partial reduction that ends every launch)
  if (mv.sh.rec && mv.slot_of) {
    const int nparts = plan.ntiles * cells_split(plan.ntiles, p.n, sizeof(A) == 8);
    if (ev0) (void)hipEventRecord(ev0, st);
#define DUST_G(G, D, UU)                                                                                   \
  do {                                                                                                     \
    launch_cells_g<TS, A, G, D, UU>(plan, p, mv, boxes_d, fl, f, sp, drag_mode, dt, tdev, bin_start, xg, dg, \
                                    sums, st);                                                             \
    if (ev1) (void)hipEventRecord(ev1, st);                                                                \
    hipLaunchKernelGGL((k_fused_deferred<TS, A, G, D, UU>), dim3(DEFER_BLOCKS), dim3(256), 0, st, p,       \
                       ShadowView<TS>{nullptr, nullptr}, (const uint32_t*)nullptr, boxes_d, nbox, fl, f, sp, \
                       drag_mode, A(dt), tdev, xg, (const uint32_t*)plan.defer_list,                       \
                       (const uint32_t*)plan.defer_count, part, nparts, (int)sums, dg);                    \
  } while (0)
    if (geom == GEOM_CART && ndim == 2 && unif) DUST_G(GEOM_CART, 2, true);
    else if (geom == GEOM_CART && ndim == 2) DUST_G(GEOM_CART, 2, false);
    else if (geom == GEOM_CART && unif) DUST_G(GEOM_CART, 3, true);
    else if (geom == GEOM_CART) DUST_G(GEOM_CART, 3, false);
    else if (geom == GEOM_CYL) DUST_G(GEOM_CYL, 3, false);
    else DUST_G(GEOM_SPH, 3, false);
#undef DUST_G
    fe = fused_end<TS>(plan, nparts, dg, sums, p, mv, bin_start);
    return;
  }
#define DUST_G(G, D, UU)                                                                          \
  launch_fused_g<TS, A, G, D, UU>(plan, p, mv, boxes_d, fl, f, sp, drag_mode, dt, tdev,            \
                                  bin_start, xg, dg, part, sums, plan.defer_list,                  \
                                  plan.defer_count, nbox, ev0, ev1, st)
  if (geom == GEOM_CART && ndim == 2 && unif) DUST_G(GEOM_CART, 2, true);
  else if (geom == GEOM_CART && ndim == 2) DUST_G(GEOM_CART, 2, false);
  else if (geom == GEOM_CART && unif) DUST_G(GEOM_CART, 3, true);
  else if (geom == GEOM_CART) DUST_G(GEOM_CART, 3, false);
  else if (geom == GEOM_CYL) DUST_G(GEOM_CYL, 3, false);
  else DUST_G(GEOM_SPH, 3, false);
#undef DUST_G
  fe = fused_end<TS>(plan, plan.ntiles, dg, sums, p, mv, bin_start);
}

template <typename TS>
FusedEnd<TS> fused_end(const FusedPlan& plan, int nparts, DiagDev* dg, bool sums, const PView<TS>& p,
                       const FusedMove<TS>& mv, const int64_t* bin_start) {
  return {plan.part_d, nparts + DEFER_BLOCKS, dg, (int)sums, plan.defer_count, p, mv, bin_start,
          mv.sh.rec ? REDUCE_TAIL_BLOCKS : 0};
}

template <typename TS> void launch_fused_end(const FusedEnd<TS>& fe, hipStream_t st) {
  if (fe.blocks() > 0) hipLaunchKernelGGL((k_fused_end<TS>), dim3(fe.blocks()), dim3(REDUCE_THREADS), 0, st, fe);
}

// ---------------------------------------------------------------- rebinning by half-step cell

// Tile-major key of the cell each particle reaches in the first half drift
// (the same drift the fused kernel does, so a particle is normally processed
// by the thread of the cell it kicks in).  A particle that leaves through an
// open face keeps the key of its current cell (the fused kernel removes it);
// a particle without a valid cell gets key nbins.  (The sort takes the
// particle indices as values.)  The particles are packed into sh on the way:
// the tile kernel, at its 2 waves per SIMD, reads them in sorted order, where
// seven to nine arrays cost it as many scattered reads each.  (A separate
// pass that moved the arrays into sorted order, at 7 waves per SIMD, took
// longer than the packing and the kernel's own reads: 8.7 ms for 120 M
// particles.)
template <typename TS, typename A, int GEOM, int NDIM, bool U>
__global__ void __launch_bounds__(256)
    k_halfstep_keys(PView<TS> p, const Box* __restrict__ boxes, int nbox, Forces f, A dt,
                    const double* __restrict__ tdev, uint32_t nbins, TileShape ts,
                    uint32_t* __restrict__ key, ShadowView<TS> sh) {
  constexpr int nc = GEOM == GEOM_CART ? NDIM : 3;
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= p.n) return;
  // every load issued before the cell is examined (one memory latency)
  const int64_t c = p.cell[i];
  A off[3], mom[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    off[d] = d < NDIM ? A(p.off[d][i]) : A(0);
    mom[d] = d < nc ? A(p.mom[d][i]) : A(0);
  }
  pack_particle(p, i, c, off, mom, sh);
  uint32_t k = nbins;
  auto key_in = [&](const Box& B) {
    int idx[3];
    unravel(B, c - B.cell_base, idx);
    const A h = A(0.5) * dt;
    int here[3] = {idx[0], idx[1], idx[2]};
    return drift_any<A, GEOM, NDIM, U>(B, f, true, h, *tdev + double(h), idx, off, mom)
               ? tile_key_idx(B, idx, ts) : tile_key_idx(B, here, ts);
  };
  if (c >= 0 && c < (int64_t)nbins) {
    // one box (the common case): its descriptor is uniform, read with
    // scalar loads; several boxes: the particle's box per lane
    if (nbox == 1)
      k = key_in(boxes[0]);
    else
      k = key_in(boxes[find_box(boxes, nbox, c)]);
  }
  // a key beyond the bins would break the sort's bin starts
  key[i] = k < nbins ? k : nbins;
}

template <typename TS, typename A>
void launch_halfstep_keys(const PView<TS>& p, const Box* boxes_d, int nbox, int geom, int ndim,
                          int unif, const Forces& f, double dt, const double* tdev, int64_t nbins,
                          TileShape ts, uint32_t* key, const ShadowView<TS>& sh, hipStream_t st) {
  if (p.n == 0) return;
  unsigned g = (unsigned)((p.n + 255) / 256);
#define DUST_K(G, D, UU)                                                                          \
  hipLaunchKernelGGL((k_halfstep_keys<TS, A, G, D, UU>), dim3(g), dim3(256), 0, st, p, boxes_d,     \
                     nbox, f, A(dt), tdev, (uint32_t)nbins, ts, key, sh)
  if (geom == GEOM_CART && ndim == 2 && unif) DUST_K(GEOM_CART, 2, true);
  else if (geom == GEOM_CART && ndim == 2) DUST_K(GEOM_CART, 2, false);
  else if (geom == GEOM_CART && unif) DUST_K(GEOM_CART, 3, true);
  else if (geom == GEOM_CART) DUST_K(GEOM_CART, 3, false);
  else if (geom == GEOM_CYL) DUST_K(GEOM_CYL, 3, false);
  else DUST_K(GEOM_SPH, 3, false);
#undef DUST_K
}

// The level-major order of each tile's binned particles as a permutation:
// lm[slot] = perm[ps + j] for the j-th particle of a cell whose sorted range
// starts at ps (one workgroup per tile, one thread per cell: the fused
// kernel's mapping); inverse: lm[ps + j] = slot.
__global__ void __launch_bounds__(256)
    k_level_perm(const TileDesc* __restrict__ tiles, TileShape ts, const uint32_t* __restrict__ perm,
                 const int64_t* __restrict__ bin_start, uint32_t* __restrict__ lm, int inverse) {
  const TileDesc td = tiles[blockIdx.x];
  const int TX = ts.t[0], TY = ts.t[1];
  const int lx = threadIdx.x % TX, ly = (threadIdx.x / TX) % TY, lz = threadIdx.x / (TX * TY);
  const bool own = lx < td.ex && ly < td.ey && lz < td.ez;
  int64_t ps = 0, pe = 0;
  if (own) {
    const int64_t key = td.key0 + lx + (int64_t)td.ex * (ly + (int64_t)td.ey * lz);
    ps = bin_start[key];
    pe = bin_start[key + 1];
  }
  const WaveLevels wl = wave_levels(own ? (int)(pe - ps) : 0, ps);
  uint32_t lvl = wl.base;
  for (int j = 0; j < wl.nlev; ++j) {
    const uint32_t to = level_slot(wl, j, lvl);
    if (wl.cnt > j) {
      if (inverse) lm[ps + j] = to;
      else lm[to] = perm[ps + j];
    }
  }
}

void launch_level_perm(const FusedPlan& plan, int64_t n, const uint32_t* perm, const int64_t* bin_start,
                       uint32_t* lm, bool inverse, hipStream_t st) {
  if (n == 0 || plan.ntiles == 0) return;
  hipLaunchKernelGGL(k_level_perm, dim3(plan.ntiles), dim3(256), 0, st, plan.tiles_d, plan.tile, perm, bin_start, lm,
                     (int)inverse);
}

// A fused rebinning step's us with a particle per lane and a cell per thread:
//  * 64x96x16 cylindrical disk, FP32, 136 and 200 at 4 particles per cell, 471
//    and 624 at 32, 731 and 841 at 48, 1026 and 1056 at 64; 64x32x48 spherical
//    disk 140 and 216, 498 and 633, 807 and 864, 1165 and 1081 (FP64: 1516 and
//    2146 at 64);
//  * Cartesian, where the tile kernel's arithmetic is shorter: 256^2, FP32, 105
//    and 121 at 4, 183 and 219 at 24, 232 and 250 at 32, 402 and 322 at 48; FP64
//    235 and 259 at 24, 357 and 328 at 32; 48^3, FP64, 184 and 243 at 4, 519 and
//    625 at 24, 1057 and 1044 at 48;
//  * FP32 uniform Cartesian (c3), shorter again: 96^3 525 and 581 at 4, 835 and
//    812 at 8, 1309 and 1040 at 12; shearing boxes whose particles have gathered,
//    at 8, 116 and 139 (32^3), 852 and 873 (100x96x72), 1472 and 1529 (128^3).
bool cells_path(int64_t n, int64_t cells, int geom, bool c3) {
  return n <= (c3 ? 9 : geom == GEOM_CART ? 28 : 56) * cells;
}

// As many workgroups a tile as the chip holds at once, each with a chunk of
// particles at least.  us with one and with more: 64^2 FP64 square of 65 k
// particles, 16 tiles, the kernel 65 and (16) 17; 32^3 shearing box of 262 k, 128
// tiles, 54 and (4) 33; 64x96x16 cylindrical disk at 8 per cell, FP32, 384 tiles,
// the step 189 and (2) 167.  More than the chip holds lose: that disk in FP64 225
// and (2) 243, 48^3 shearing box at 8 per cell, FP32, 432 tiles, 205 and (2) 224.
int cells_split(int ntiles, int64_t n, bool f64) {
  if (ntiles <= 0) return 1;
  const int64_t fill = (f64 ? CELLS_BLOCKS_F64 : CELLS_BLOCKS) / ntiles,
                chunks = (n + (int64_t)ntiles * 256 - 1) / ((int64_t)ntiles * 256);
  return (int)std::max<int64_t>(1, std::min(fill, chunks));
}

#define DUST_FUSED_INST(TS, A)                                                                    \
  template void launch_fused<TS, A>(const FusedPlan&, const PView<TS>&, const FusedMove<TS>&,       \
                                    const Box*, int, int, int, int, const FView<TS>&,              \
                                    const Forces&, const Species*, int, double, const double*,     \
                                    const int64_t*, const double*, DiagDev*, bool, FusedEnd<TS>&,  \
                                    hipEvent_t, hipEvent_t, hipStream_t);                          \
  template void launch_halfstep_keys<TS, A>(const PView<TS>&, const Box*, int, int, int, int,       \
                                            const Forces&, double, const double*, int64_t,         \
                                            TileShape, uint32_t*, const ShadowView<TS>&, hipStream_t);

DUST_FUSED_INST(float, double)
DUST_FUSED_INST(float, float)
DUST_FUSED_INST(double, double)

template FusedEnd<float> fused_end<float>(const FusedPlan&, int, DiagDev*, bool, const PView<float>&,
                                         const FusedMove<float>&, const int64_t*);
template void launch_fused_end<float>(const FusedEnd<float>&, hipStream_t);
template void launch_fused_end<double>(const FusedEnd<double>&, hipStream_t);

}  // namespace dust
