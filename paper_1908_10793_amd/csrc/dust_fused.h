// Fused tile kernel of the dust hot path: plan (tile table) and launcher.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dust_launch.h"
#include "dust_types.h"

namespace dust {

struct TileDesc {
  int32_t box;
  int32_t i0, j0, k0;    // first active cell of the tile
  int32_t ex, ey, ez;    // tile extents (clipped at the box edge)
  int32_t pad;
  int64_t key0;          // first tile-major key of the tile
};

struct FusedPlan {
  bool ok = false;
  TileShape tile{{8, 8, 4}};
  int shape = 0;          // index of the compiled tile shape
  bool small = false;     // every box has fewer than 2^24 cells
  bool tsc = false;       // and TSC shape on every axis
  int halo = 2;           // LDS window beyond the tile: stencil + half drift
  int ntiles = 0;
  int rmax[3] = {0, 0, 0};  // largest region extents
  size_t lds_cells = 0;
  TileDesc* tiles_d = nullptr;
  double* part_d = nullptr;   // per-tile diagnostic partials (+ the deferred kernel's)
  uint32_t* defer_count = nullptr;   // deferred particles of the current launch
  uint32_t* defer_list = nullptr;    // their slots (capacity defer_cap)
  size_t defer_cap = 0;
  uint8_t* tile_map = nullptr;       // per tile, 256 tile-local cells in thread order (FP32
                                     // Cartesian path: ranked by particle count at each rebinning)
};

// A particle's state as a rebinning packs it (the shadow copy of the fused
// step): one place to read per particle for the tile kernel, which takes them
// in sorted order.  Ext: the attributes that not every run has.
template <typename TS> struct __attribute__((aligned(16))) ShadowRec {
  int32_t cell, species;
  TS off[3], mom[3];
};
template <typename TS> struct __attribute__((aligned(16))) ShadowExt {
  int32_t id;
  TS drag, mass;
};
static_assert(sizeof(ShadowRec<float>) == 32 && sizeof(ShadowExt<float>) == 16, "FP32 records");
static_assert(sizeof(ShadowRec<double>) == 64 && sizeof(ShadowExt<double>) == 32, "FP64 records");
template <typename TS> struct ShadowView {
  ShadowRec<TS>* rec;   // null: no rebinning in this step
  ShadowExt<TS>* ext;   // null where the particles have no id, drag and mass
};

// Capacity of the deferred-particle list for n particles.
dust_status_t fused_plan_reserve(FusedPlan& plan, int64_t n);

dust_status_t fused_plan_init(FusedPlan& plan, const Box* boxes, int nbox, TileShape tile, int slack);
void fused_plan_free(FusedPlan& plan);
// LDS of one fused workgroup: the dynamic part (windows), and the static
// part (per-thread diagnostic sums, species tables) as an upper bound.
size_t fused_lds_bytes(const FusedPlan& plan, int nc, int ts_bytes);
static constexpr size_t FUSED_STATIC_LDS = 5 * 256 * sizeof(double) + 3 * DUST_MAX_SPECIES * sizeof(double) + 256;

// One fused step over every tile (binned by tile-major key, bin_start).
// After a rebinning (sh.rec given): slot s of p receives the update of the
// packed particle src_index[s] (or slot slot_of[t] that of perm[t]: a particle
// per lane, dust_cells_kern.h), attributes too, and the slots from
// bin_start[nbins] on (no tile visits them) the packed particles perm[s];
// else the particles of p are updated in place.  clear_removed: a particle
// that leaves in the second half drift of a rebinning step keeps whatever its
// new slot held; this zeroes that instead.  xg: the context's FP64 x-ghost
// gas layers (filled this step), or null.  ev0 / ev1 (nullable) are recorded
// around the tile kernel alone (not the deferred-particle kernel).
template <typename TS> struct FusedMove {
  ShadowView<TS> sh;
  const uint32_t* src_index;   // null: slot_of is given instead
  const uint32_t* perm;
  const uint32_t* slot_of;     // slot of each sorted position (FP32 uniform-Cartesian path: of each of
  const uint32_t* order_src;   // order_src, the same particles lane by lane of the layout)
  int64_t nbins;
  int clear_removed;
};
// What is left of a fused launch (a launch_fused or launch_c3, which fill it
// in): the per-workgroup diagnostic partials (tile kernel and deferred
// kernel) to be added to the diagnostics block and the deferred-particle
// count to be reset, by one workgroup, and after a rebinning the slots without
// a cell to be filled (see launch_fused), by tail_blocks more.  A step that
// sums over its grid does it in that launch (launch_grid_sums), else
// launch_fused_end.
template <typename TS> struct FusedEnd {
  const double* part;
  int nparts;
  DiagDev* dg;
  int sums;
  uint32_t* defer_count;
  PView<TS> p;
  FusedMove<TS> mv;
  const int64_t* bin_start;
  int tail_blocks;
  int blocks() const { return nparts > 0 ? 1 + tail_blocks : 0; }
};
template <typename TS, typename A>
void launch_fused(const FusedPlan& plan, const PView<TS>& p, const FusedMove<TS>& mv,
                  const Box* boxes_d, int nbox, int geom, int ndim, int unif, const FView<TS>& fl,
                  const Forces& f, const Species* sp, int drag_mode, double dt, const double* tdev,
                  const int64_t* bin_start, const double* xg, DiagDev* dg, bool sums,
                  FusedEnd<TS>& fe, hipEvent_t ev0, hipEvent_t ev1, hipStream_t st);

// A rebinning's first pass: keys (tile-major) of the cells the particles
// reach in the first half drift of a step of length dt starting at *tdev, and
// the particles packed into sh.
template <typename TS, typename A>
void launch_halfstep_keys(const PView<TS>& p, const Box* boxes_d, int nbox, int geom, int ndim,
                          int unif, const Forces& f, double dt, const double* tdev, int64_t nbins,
                          TileShape ts, uint32_t* key, const ShadowView<TS>& sh, hipStream_t st);

// After the sort (perm, bin_start): lm = the source index of every binned
// slot in the fused kernel's level-major layout within each wave's range of
// slots; inverse: instead the slot of every sorted position.
void launch_level_perm(const FusedPlan& plan, int64_t n, const uint32_t* perm, const int64_t* bin_start,
                       uint32_t* lm, bool inverse, hipStream_t st);

// Whether a rebinning step of n particles over `cells` active cells runs a
// particle per lane (dust_cells_kern.h) or a cell per thread.
bool cells_path(int64_t n, int64_t cells, int geom, bool c3);
// Workgroups per tile of that kernel, which share its particles (each with a
// window of its own): few tiles would leave CUs idle.
int cells_split(int ntiles, int64_t n, bool f64);

template <typename TS> void launch_fused_end(const FusedEnd<TS>& fe, hipStream_t st);
template <typename TS>
FusedEnd<TS> fused_end(const FusedPlan& plan, int nparts, DiagDev* dg, bool sums, const PView<TS>& p,
                       const FusedMove<TS>& mv, const int64_t* bin_start);

// The fused step of uniform 3-D Cartesian boxes in FP32 storage and
// arithmetic (dust_cart3.hip), with forces none, constant or standard
// shearing box: the tile kernel (ev0 / ev1 around it), the deferred-particle
// kernel and the reduction of their diagnostic partials.
void launch_c3(const FusedPlan& plan, const PView<float>& p, const FusedMove<float>& mv,
               const Box* boxes_d, int nbox, const FView<float>& fl, const Forces& f, const Species* sp,
               int drag_mode, double dt, const double* tdev, const int64_t* bin_start, const double* xg,
               DiagDev* dg, bool sums, FusedEnd<float>& fe, hipEvent_t ev0, hipEvent_t ev1, hipStream_t st);
// The same after a rebinning with a particle per lane (dust_cart3_cells.hip).
void launch_c3_cells(const FusedPlan& plan, const PView<float>& p, const FusedMove<float>& mv, const Box* boxes_d,
                     const FView<float>& fl, const Forces& f, const Species* sp, double dt, const double* tdev,
                     const int64_t* bin_start, const double* xg, DiagDev* dg, bool sums, hipStream_t st);
// Its rebinning: half-step tile keys with its own drift (and the packed
// particles), and after the sort the per-tile ranking of cells by count
// (plan.tile_map) with the source index of every slot (lm), or with order_slot
// given: lm the source indices lane by lane, order_slot their slots.
void launch_c3_keys(const PView<float>& p, const Box* boxes_d, int nbox, double dt, int64_t nbins,
                    TileShape ts, uint32_t* key, const ShadowView<float>& sh, hipStream_t st);
void launch_c3_level_perm(const FusedPlan& plan, const uint32_t* perm, const int64_t* bin_start, uint32_t* lm,
                          uint32_t* order_slot, hipStream_t st);
// Predictor drag source (mass: dust density) on the binned layout of the
// last fused step (see k_c3_aux): out[0..2] the momentum deposit channels
// (mass: out[0] the density array).
void launch_c3_aux(const FusedPlan& plan, const PView<float>& p, const Box* boxes_d, int nbox,
                   const FView<float>& fl, float* const out[3], bool mass, const Forces& f, const Species* sp,
                   double dt, const int64_t* bin_start, int64_t nbins, DiagDev* dg, hipStream_t st);
size_t c3_lds_bytes(const FusedPlan& plan);

}  // namespace dust
