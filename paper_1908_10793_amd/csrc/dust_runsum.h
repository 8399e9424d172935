// Sums of a chunk of particles over their stencils, by runs of one host cell
// (gfx950): one particle per thread of a 256-thread workgroup, in an order in
// which the particles of a cell follow one another.
//
// Each thread puts its particle's weights and channel values in LDS; then
// nine lanes take a particle, one lane per row of three cells of its stencil
// (2-D: per cell), seven particles of a wave at a time, and sum in registers
// until the host cell changes.  A run is then added to the FP64 window with
// LDS atomics.  A lane holds one row's channels (12 registers where a thread
// per host cell needs 108), so FP64 sums cost no occupancy, and lanes never
// wait for the fullest cell of a wave.  A lane per cell, two particles at a
// time, took three times the LDS reads: 800 us for the density of 30 M
// particles against 390.
#pragma once

#include "dust_device.h"
#include "dust_particle.h"

namespace dust {

static constexpr int RUN_THREADS = 256;

template <typename A, int NDIM> struct RunSums {
  static constexpr int NA = NDIM > 2 ? 3 : 1;     // cells of a lane
  static constexpr int GROUPS = 7;                // particles that a wave takes at a time
  // a wave's 64 particles go through its records in one round, FP64 in two
  // (with the records of 64, one workgroup less would fit a CU's LDS)
  static constexpr int ROUNDS = sizeof(A) == 4 ? 1 : 2;
  static constexpr int RP = 64 / ROUNDS;          // particles of a round
  static constexpr int PG = (RP + GROUPS - 1) / GROUPS;   // a group's share of them
  // one particle's words: q[4], w0[3], then FP32 the window index and the 9
  // products w1 w2 at a stride of 20 words, FP64 w1[3], w2[3] and the window
  // index at 14: consecutive lanes' 16-byte writes, and the seven groups'
  // reads, on distinct banks
  static constexpr bool F32 = sizeof(A) == 4;
  static constexpr int RS = F32 ? 20 : 14;
  static constexpr int W0 = 4, W1 = F32 ? 8 : 7, W2 = 10, HOST = F32 ? 7 : 13;
  static constexpr int WR = GROUPS * PG;          // records of a wave (those past RP stay zero)
  static constexpr int WORDS = (RUN_THREADS / 64) * WR * RS;
};

// The calling workgroup's piece of its tile's particles [s0, s1), whole chunks
// of RUN_THREADS: piece blockIdx.x mod split of `split` (the last ones may be
// empty, s0 >= s1).
template <typename I> __device__ __forceinline__ void tile_piece(I& s0, I& s1, int split) {
  if (s0 >= s1) return;
  const uint32_t chunks = (uint32_t)((s1 - s0 + RUN_THREADS - 1) / RUN_THREADS);
  const uint32_t per = (chunks + split - 1) / split, q = blockIdx.x % (unsigned)split;
  const uint32_t a = q * per;
  const I end = s1;
  s0 = a < chunks ? s0 + (I)a * RUN_THREADS : end;
  s1 = end - s0 < (I)per * RUN_THREADS ? end : s0 + (I)per * RUN_THREADS;
}

// A wave's LDS writes before this, its reads after (its LDS operations
// complete in order; this keeps the compiler's order).
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Once per workgroup, before the first run_sums: the records past a round's
// particles are zero.
template <typename A, int NDIM> __device__ __forceinline__ void run_sums_init(A* rec) {
  using S = RunSums<A, NDIM>;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  for (int r = lane; r < (S::WR - S::RP) * S::RS; r += 64) rec[(wave * S::WR + S::RP) * S::RS + r] = A(0);
}

// Adds the particles of the calling workgroup's threads to the window win
// (NCH channels of WC cells, RX by RY a layer; compile-time or uniform).  Every thread calls; has: it
// has a particle, whose host cell has window index r0, channel values q and
// weights st (all zero without one).  rec: RunSums::WORDS;
// a wave uses its own part only.
template <typename A, int NDIM, int NCH>
__device__ __forceinline__ void run_sums(double* win, int RX, int RY, int WC, A* rec, int r0, bool has,
                                         const A q[4], const Stencil<A>& st) {
  using S = RunSums<A, NDIM>;
  constexpr int NA = S::NA, PG = S::PG;
  constexpr int c2 = NDIM > 2 ? 1 : 0;
  constexpr bool F32 = S::F32;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  // this lane's row of the stencil (2-D: cell), relative to the host cell
  const int grp = lane / 9, row = lane % 9;
  const bool sums_lane = grp < S::GROUPS;
  const int rb = NDIM > 2 ? row % 3 : row / 3, rc = NDIM > 2 ? row / 3 : 0;   // y and z of the row
  const int ra = NDIM > 2 ? 0 : row % 3;                                      // x of its first cell
  const int soff = (ra - 1) + RX * ((rb - 1) + RY * (rc - c2));
  // where runs of one host cell start (the first particle of a group's
  // share always does)
  const int prev = __shfl_up(has ? r0 : -1, 1);
  const uint64_t starts_all = __ballot(has && ((lane % S::RP) % PG == 0 || r0 != prev));
#pragma unroll
  for (int rd = 0; rd < S::ROUNDS; ++rd) {
    const uint64_t starts = S::ROUNDS == 1 ? starts_all : (starts_all >> (rd * S::RP)) & 0xffffffffull;
    if (starts == 0) continue;   // (wave-uniform: no particle in this round)
    uint32_t any = 0;   // iterations at which a run starts in some group
#pragma unroll
    for (int g = 0; g < S::GROUPS; ++g) any |= (uint32_t)(starts >> (g * PG)) & ((1u << PG) - 1);
    // the records (a thread without a particle: zeros, which add nothing)
    if (S::ROUNDS == 1 || lane / S::RP == rd) {
      A* rw = rec + (wave * S::WR + lane % S::RP) * S::RS;
#pragma unroll
      for (int m = 0; m < 4; ++m) rw[m] = q[m];
#pragma unroll
      for (int a = 0; a < 3; ++a) rw[S::W0 + a] = st.w[0][a];
      rw[S::HOST] = A(r0);   // (exact)
      if constexpr (F32) {
#pragma unroll
        for (int a = 0; a < 9; ++a) rw[S::W1 + a] = st.w[1][a % 3] * st.w[2][NDIM > 2 ? a / 3 : 1];
      } else {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          rw[S::W1 + a] = st.w[1][a];
          rw[S::W2 + a] = st.w[2][a];
        }
      }
    }
    wave_lds_fence();
    const uint32_t mine = sums_lane ? (uint32_t)(starts >> (grp * PG)) & ((1u << PG) - 1) : 0u;
    const A* rr = rec + (wave * S::WR + (sums_lane ? grp : 0) * PG) * S::RS;
    // FP32: a run that ended waits in `done` until some group's next one ends,
    // or the last particle: the groups' runs end at different particles, and
    // the adds of one wave cost the same for one group as for seven.  128^3
    // box at 8 particles per cell: 771 -> 734 us.  (FP64 lacks the registers:
    // the drag source of 14 M particles took 1592 us so, 1353 without.)
    A acc[NA][NCH], done[NA][NCH];
    int host = -1, done_host = -1;
    auto flush = [&](const A (&v)[NA][NCH], int at) {
#pragma unroll
      for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int m = 0; m < NCH; ++m) atomicAdd(&win[m * WC + at + soff + a], double(v[a][m]));
    };
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
      for (int m = 0; m < NCH; ++m) acc[a][m] = done[a][m] = A(0);
#pragma unroll 5
    for (int j = 0; j < PG; ++j) {
      const A* w = rr + j * S::RS;
      A qj[NCH], wx[NA], wyz;
#pragma unroll
      for (int m = 0; m < NCH; ++m) qj[m] = w[m];
#pragma unroll
      for (int a = 0; a < NA; ++a) wx[a] = w[S::W0 + ra + a];
      if constexpr (F32) wyz = w[S::W1 + rb + 3 * rc];
      else wyz = w[S::W1 + rb] * w[S::W2 + (NDIM > 2 ? rc : 1)];
      if ((any >> j) & 1u) {   // (wave-uniform)
        const bool starts_here = (mine >> j) & 1u;
        if (!F32) {
          if (starts_here && host >= 0) flush(acc, host);
        } else if (__any(starts_here && done_host >= 0)) {
          if (done_host >= 0) flush(done, done_host);
          done_host = -1;
        }
        if (starts_here) {
          if (F32) done_host = host;
          host = (int)w[S::HOST];
#pragma unroll
          for (int a = 0; a < NA; ++a)
#pragma unroll
            for (int m = 0; m < NCH; ++m) {
              if (F32) done[a][m] = acc[a][m];
              acc[a][m] = A(0);
            }
        }
      }
#pragma unroll
      for (int m = 0; m < NCH; ++m) {
        const A t = wyz * qj[m];
#pragma unroll
        for (int a = 0; a < NA; ++a) acc[a][m] += wx[a] * t;
      }
    }
    if (F32 && done_host >= 0) flush(done, done_host);
    if (host >= 0) flush(acc, host);
    wave_lds_fence();   // (the records of the next round or call)
  }
}

}  // namespace dust
