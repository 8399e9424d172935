// Particle-to-grid sums over particles sorted by tile: the interface of
// dust_sorted_kern.h.
#pragma once

#include "dust_launch.h"

namespace dust {

// What a launch sums: the deposit stage (caller's values), the predictor's
// drag source, the dust density, or the unfused step (gather, kick, deposit).
enum { SORTED_DEPOSIT = 0, SORTED_SOURCE = 1, SORTED_MASS = 2, SORTED_STEP = 3 };

// A particle's state within an unfused step (positions at x^{n+1/2}), packed
// so that any order reads it as 16-byte words of one place: 48 bytes in FP32,
// 80 in FP64.
template <typename TS> struct __attribute__((aligned(16))) StepRecord {
  int32_t cell, species;
  TS off[3], mom[3], drag, mass;
};
static_assert(sizeof(StepRecord<float>) == 48 && sizeof(StepRecord<double>) == 80, "record sizes");

template <typename TS, typename TW> struct SortedIn {
  const TW* q[4];        // SORTED_DEPOSIT: the channels' values per particle
  StepRecord<TS>* rec;   // SORTED_STEP: the particles (momenta are updated)
};

// Cells of the kernel's tile along axis d (the sort's keys are tile-major in
// this shape).
constexpr int sorted_tile_extent(int ndim, int d) { return ndim < 3 ? (d < 2 ? 16 : 1) : d < 2 ? 8 : 4; }
inline TileShape sorted_tile(int ndim) {
  return TileShape{{sorted_tile_extent(ndim, 0), sorted_tile_extent(ndim, 1), sorted_tile_extent(ndim, 2)}};
}

// The sums of one launch, added to fl.dep (SORTED_MASS: fl.dep[0]).  key,
// perm: the particles sorted by the tile-major key of their current cell in
// sorted_tile(ndim), key nbins last (launch_bin).  dt: the step
// (SORTED_SOURCE: its reciprocal).  xg: as in launch_gather.  sums: add the
// kick's diagnostic sums to dg (SORTED_STEP); flags go to dg in every mode.
template <typename TS, typename A, typename TW, int MODE>
void launch_sorted(const PView<TS>& p, const Box* boxes, int nbox, int geom, int ndim, int unif,
                   const FView<TS>& fl, const SortedIn<TS, TW>& in, const double* xg, const Forces& f,
                   const Species* sp, int drag_mode, double dt, const uint32_t* key, const uint32_t* perm,
                   int64_t nbins, DiagDev* dg, bool sums, hipStream_t st);

// The half drifts around SORTED_STEP: the first from the arrays to records
// and sort keys (in the input order), the second from records to the arrays.
template <typename TS, typename A>
void launch_step_pack(const PView<TS>& p, const Box* boxes, int nbox, int geom, int ndim, int unif,
                      const Forces& f, double h, const double* tdev, double toff, StepRecord<TS>* rec,
                      uint32_t* key, int64_t nbins, DiagDev* dg, hipStream_t st);
template <typename TS, typename A>
void launch_step_unpack(const PView<TS>& p, const Box* boxes, int nbox, int geom, int ndim, int unif,
                        const Forces& f, double h, const double* tdev, double toff, const StepRecord<TS>* rec,
                        DiagDev* dg, hipStream_t st);

}  // namespace dust
