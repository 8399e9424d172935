// Particle-to-grid sums over particles sorted by tile: the interface of
// dust_sorted_kern.h.
#pragma once

#include "dust_launch.h"

namespace dust {

// What a launch sums: the deposit stage (caller's values), the predictor's
// drag source, the dust density, or the unfused step (gather, kick, deposit).
enum { SORTED_DEPOSIT = 0, SORTED_SOURCE = 1, SORTED_MASS = 2, SORTED_STEP = 3 };

template <typename TW> struct SortedIn {
  const TW* q[4];   // SORTED_DEPOSIT: the channels' values per particle
};

// Cells of the kernel's tile along axis d (the sort's keys are tile-major in
// this shape).
constexpr int sorted_tile_extent(bool f64, int ndim, int d) {
  return ndim < 3 ? (d < 2 ? 16 : 1) : d == 0 ? (f64 ? 4 : 8) : d == 1 ? 8 : 4;
}
inline TileShape sorted_tile(bool f64, int ndim) {
  return TileShape{{sorted_tile_extent(f64, ndim, 0), sorted_tile_extent(f64, ndim, 1),
                    sorted_tile_extent(f64, ndim, 2)}};
}

// The sums of one launch, added to fl.dep (SORTED_MASS: fl.dep[0]).  key,
// perm: the particles sorted by the tile-major key of their current cell in
// sorted_tile(A is double, ndim), key nbins last (launch_bin).  dt: the step
// (SORTED_SOURCE: its reciprocal).  xg: as in launch_gather.  sums: add the
// kick's diagnostic sums to dg (SORTED_STEP); flags go to dg in every mode.
template <typename TS, typename A, typename TW, int MODE>
void launch_sorted(const PView<TS>& p, const Box* boxes, int nbox, int geom, int ndim, int unif,
                   const FView<TS>& fl, const SortedIn<TW>& in, const double* xg, const Forces& f,
                   const Species* sp, int drag_mode, double dt, const uint32_t* key, const uint32_t* perm,
                   int64_t nbins, DiagDev* dg, bool sums, hipStream_t st);

}  // namespace dust
