// Particle-to-grid sums over particles sorted by tile (gfx950): the deposit
// stage, the predictor's drag source, the dust density, and the unfused
// step's gather, kick and deposit in one pass.  Any particle order, any
// geometry; the caller's arrays are read through the sort's permutation and
// stay where they are.
//
// What bounds these sums is the atomics: one particle adds to 27 cells times
// up to 4 channels.  Added to HBM one by one they ran at 0.15 G particles/s
// (a deposit of 8.5 M particles in cell order 61 ms; a wave's 64 particles
// share a cell, and its adds queue on the same words).  Here
//  * a workgroup takes a fixed number of consecutive slots of the sorted
//    order, whatever their cells hold (no imbalance where dust collects),
//    and walks them in chunks of 256, tile by tile, with an FP64 LDS window
//    over the tile and one cell around it;
//  * one lane per particle forms its weights and its channels' values (the
//    next chunk's particles are loaded meanwhile), and the chunk is summed by
//    runs of one host cell (dust_runsum.h);
//  * a run of one host cell is then added to the window, and the window to
//    HBM once per tile.
#pragma once

#include <type_traits>

#include "dust_device.h"
#include "dust_launch.h"
#include "dust_particle.h"
#include "dust_runsum.h"
#include "dust_sorted.h"

namespace dust {

static constexpr int SORTED_THREADS = RUN_THREADS;   // also the particles of a chunk

// Three velocity components and the density of a window's cell, in the
// storage type; the unfused step in Cartesian boxes takes the arithmetic type
// (the x ghosts of a shear-periodic box are FP64 values).
template <typename T> struct GasCell { T v[4]; };

// Compile-time layout of a kernel.
template <typename TS, typename A, int GEOM, int NDIM, int MODE> struct SortedShape {
  static constexpr int NC = GEOM == GEOM_CART ? NDIM : 3;
  static constexpr int NCH = MODE == SORTED_MASS ? 1 : MODE == SORTED_SOURCE ? NC : NC + 1;
  static constexpr bool GAS = MODE == SORTED_SOURCE || MODE == SORTED_STEP;
  using TG = typename std::conditional<MODE == SORTED_STEP && GEOM == GEOM_CART, A, TS>::type;
  static constexpr int T0 = sorted_tile_extent(NDIM, 0), T1 = sorted_tile_extent(NDIM, 1),
                       T2 = sorted_tile_extent(NDIM, 2);
  static constexpr int RX = T0 + 2, RY = T1 + 2, RZ = NDIM > 2 ? T2 + 2 : 1;
  static constexpr int WC = RX * RY * RZ;
  static constexpr int NT = NDIM > 2 ? 27 : 9;    // cells of a stencil
};

// Stored state of one particle, as loaded a chunk ahead.
template <typename TS, typename TW> struct SortedRaw {
  int32_t cell, species;
  TS off[3], mom[3], drag, mass;
  TW q[4];
};

template <typename TS, typename TW, int GEOM, int NDIM, int MODE>
__device__ __forceinline__ void sorted_load(const PView<TS>& p, const SortedIn<TS, TW>& in, int drag_mode, int64_t i,
                                            SortedRaw<TS, TW>& r) {
  constexpr int NC = GEOM == GEOM_CART ? NDIM : 3;
  if constexpr (MODE == SORTED_STEP) {
    // the packed record of the unfused step: one line of memory per particle
    const StepRecord<TS> s = in.rec[i];
    r.cell = s.cell;
    r.species = s.species;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      r.off[d] = s.off[d];
      r.mom[d] = s.mom[d];
    }
    r.drag = s.drag;
    r.mass = s.mass;
    return;
  }
  r.cell = p.cell[i];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    r.off[d] = d < NDIM ? p.off[d][i] : TS(0);
    // (the deposit reads momenta only to flag non-finite ones, where given)
    r.mom[d] = MODE != SORTED_MASS && d < NC && (MODE != SORTED_DEPOSIT || p.mom[d]) ? p.mom[d][i] : TS(0);
  }
  r.species = 0;
  r.mass = r.drag = TS(0);
  if constexpr (MODE == SORTED_DEPOSIT) {
#pragma unroll
    for (int m = 0; m < 4; ++m) r.q[m] = m <= NC ? in.q[m][i] : TW(0);
  } else {
    if (p.species) r.species = p.species[i];
    if (p.mass) r.mass = p.mass[i];
    if (MODE != SORTED_MASS && drag_mode != DRAG_SPECIES) r.drag = p.drag[i];
  }
}

template <typename TS, typename A, typename TW, int GEOM, int NDIM, bool U, int MODE>
__global__ void __launch_bounds__(SORTED_THREADS) __attribute__((amdgpu_waves_per_eu(MODE == SORTED_STEP ? 2 : 1)))
    k_sorted(PView<TS> p, const Box* __restrict__ boxes, int nbox, FView<TS> fl, SortedIn<TS, TW> in,
             const double* __restrict__ xg, Forces f, const Species* __restrict__ sp, int drag_mode, A dt,
             const uint32_t* __restrict__ key, const uint32_t* __restrict__ perm, uint32_t nbins, int ppb,
             DiagDev* dg, int sums) {
  using S = SortedShape<TS, A, GEOM, NDIM, MODE>;
  using TG = typename S::TG;
  constexpr int NC = S::NC, NCH = S::NCH, RX = S::RX, RY = S::RY, WC = S::WC;
  constexpr int c2 = NDIM > 2 ? 1 : 0;
  __shared__ double win[NCH * WC];
  __shared__ __align__(16) A rec[RunSums<A, NDIM>::WORDS];
  __shared__ GasCell<TG> gas[S::GAS ? WC : 1];
  const int tid = threadIdx.x;
  const int64_t s0 = (int64_t)blockIdx.x * ppb;
  const int64_t s1 = s0 + ppb < p.n ? s0 + ppb : p.n;
  uint32_t flags = 0;
  double sum[5] = {0, 0, 0, 0, 0}, cells = 0.0;   // SORTED_STEP: the kick's diagnostics
  run_sums_init<A, NDIM>(rec);

  // the tile in the window: its box, cells, first window cell, end of its keys
  int ub = 0, e0 = 0, e1 = 0, e2 = 0, o0 = 0, o1 = 0, o2 = 0;
  uint32_t kend = 0;
  auto window_to_grid = [&]() {
    const Box& B = boxes[ub];
    for (int r = tid; r < WC; r += SORTED_THREADS) {
      const int a = r % RX, b = (r / RX) % RY, c = r / (RX * RY);
      if (a >= e0 + 2 || b >= e1 + 2 || (NDIM > 2 && c >= e2 + 2)) continue;
      const int64_t id = stored_index(B, o0 + a, o1 + b, o2 + c);
      const double iv = inv_volume(B, o0 + a, o1 + b, o2 + c);
#pragma unroll
      for (int m = 0; m < NCH; ++m) {
        const double x = win[m * WC + r];
        if (x != 0.0) unsafeAtomicAdd(&fl.dep[m][id], TS(x * iv));
      }
    }
  };
  auto next_tile = [&](uint32_t k0) {
    // the tile of key k0 (its cells are consecutive keys), its window
    ub = __builtin_amdgcn_readfirstlane(nbox == 1 ? 0 : find_box(boxes, nbox, k0));
    const Box& B = boxes[ub];
    const int n0 = B.ax[0].n, n1 = B.ax[1].n, n2 = NDIM > 2 ? B.ax[2].n : 1;
    uint32_t r = k0 - (uint32_t)B.cell_base;
    const uint32_t layer = (uint32_t)n0 * (uint32_t)n1 * (uint32_t)min(S::T2, n2);   // (at most the box)
    const int tk = NDIM > 2 ? (int)(r / layer) : 0;
    r -= (uint32_t)tk * layer;
    e2 = min(S::T2, n2 - tk * S::T2);
    const uint32_t line = (uint32_t)n0 * (uint32_t)min(S::T1, n1) * (uint32_t)e2;
    const int tj = (int)(r / line);
    r -= (uint32_t)tj * line;
    e1 = min(S::T1, n1 - tj * S::T1);
    const uint32_t col = (uint32_t)S::T0 * (uint32_t)(e1 * e2);
    const int ti = (int)(r / col);
    r -= (uint32_t)ti * col;
    e0 = min(S::T0, n0 - ti * S::T0);
    kend = k0 - r + (uint32_t)(e0 * e1 * e2);
    o0 = ti * S::T0 - 1;
    o1 = tj * S::T1 - 1;
    o2 = tk * S::T2 - c2;
    for (int w = tid; w < WC; w += SORTED_THREADS) {
#pragma unroll
      for (int m = 0; m < NCH; ++m) win[m * WC + w] = 0.0;
      if constexpr (S::GAS) {
        const int a = w % RX, b = (w / RX) % RY, c = w / (RX * RY);
        GasCell<TG> g{};
        if (a < e0 + 2 && b < e1 + 2 && (NDIM < 3 || c < e2 + 2)) {
#pragma unroll
          for (int m = 0; m < NC; ++m) g.v[m] = TG(gas_comp(B, fl, xg, m, o0 + a, o1 + b, o2 + c));
          if (drag_mode == DRAG_EPSTEIN) g.v[3] = TG(fl.rho[stored_index(B, o0 + a, o1 + b, o2 + c)]);
        }
        gas[w] = g;
      }
    }
  };

  // the particles of a chunk are loaded one chunk ahead, their places two
  // (past the block's last slot: the last one again, not used)
  auto slot = [&](int64_t e) { return e < s1 ? e : s1 - 1; };
  SortedRaw<TS, TW> nxt;
  uint32_t i_nxt = perm[slot(s0 + tid)], k_nxt = key[slot(s0 + tid)];
  sorted_load<TS, TW, GEOM, NDIM, MODE>(p, in, drag_mode, i_nxt, nxt);
  uint32_t i_far = perm[slot(s0 + SORTED_THREADS + tid)];
  bool last = false;
  for (int64_t cb = s0; cb < s1 && !last; cb += SORTED_THREADS) {
    const SortedRaw<TS, TW> cur = nxt;
    const uint32_t i = i_nxt, k = k_nxt;
    const int nv = (int)(s1 - cb < SORTED_THREADS ? s1 - cb : SORTED_THREADS);
    i_nxt = i_far;
    k_nxt = key[slot(cb + SORTED_THREADS + tid)];
    sorted_load<TS, TW, GEOM, NDIM, MODE>(p, in, drag_mode, i_nxt, nxt);
    i_far = perm[slot(cb + 2 * SORTED_THREADS + tid)];
    int done = 0;   // threads of the chunk whose particles are summed
    while (done < nv) {
      // those of the window's tile (sorted: threads done .. done + cnt - 1)
      const bool has = tid >= done && tid < nv && k < kend;
      const int cnt = __syncthreads_count(has);
      if (cnt == 0) {
        if (kend) window_to_grid();
        const uint32_t k0 = key[cb + done];
        if (k0 >= nbins) {
          // sorted last: particles without a cell, and cell ids out of range
          // (the step flagged those in its first drift)
          if (MODE != SORTED_STEP)
            for (int64_t e = cb + done + tid; e < s1; e += SORTED_THREADS)
              if (p.cell[perm[e]] >= 0) flags |= DUST_FLAG_BAD_CELL;
          kend = 0;
          last = true;
          break;
        }
        __syncthreads();   // (the window is cleared by other threads than read it)
        next_tile(k0);
        continue;
      }
      const Box& B = boxes[ub];
      int r0 = -1;
      A q[4] = {A(0), A(0), A(0), A(0)};
      Stencil<A> st;
#pragma unroll
      for (int d = 0; d < 3; ++d)
#pragma unroll
        for (int a = 0; a < 3; ++a) st.w[d][a] = A(0);
      if (has) {
        int idx[3];
        A off[3], mom[3];
        unravel(B, cur.cell - B.cell_base, idx);
        bool bad = false, nonfinite = false;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          off[d] = A(cur.off[d]);
          bad |= !(off[d] >= A(-0.5) && off[d] < A(0.5));
          mom[d] = A(cur.mom[d]);
          nonfinite |= !isfinite(double(mom[d]));
        }
        flags |= bad ? (uint32_t)DUST_FLAG_OFFSET_RANGE : 0u;
        flags |= nonfinite ? (uint32_t)DUST_FLAG_NONFINITE : 0u;
        r0 = (idx[0] - o0) + RX * ((idx[1] - o1) + RY * (idx[2] - o2));
        stencil_weights<A, GEOM, NDIM, U>(B, idx, off, st);
        if constexpr (MODE == SORTED_DEPOSIT) {
#pragma unroll
          for (int m = 0; m < NCH; ++m) q[m] = -A(cur.q[m]);
        } else {
          int spc = cur.species;
          if (spc >= sp->n) {
            flags |= DUST_FLAG_BAD_CELL;
            spc = 0;
          }
          const A m = p.mass ? A(cur.mass) : A(sp->mass[spc]);
          if constexpr (MODE == SORTED_MASS) {
            q[0] = m;
          } else {
            const A dval = drag_mode == DRAG_SPECIES ? A(1) : A(cur.drag);
            Where<A> w;
            where<A, GEOM, NDIM, U>(B, idx, off, w);
            // SOURCE: the slip as a weighted sum of differences; STEP: the
            // gathered velocity
            A v[3] = {A(0), A(0), A(0)}, rg = A(0);
            // (one plane of the stencil per iteration: straight-line code would
            // issue every read first, and hold its registers)
#pragma unroll 1
            for (int cc = -c2; cc <= c2; ++cc) {
              const A wz = NDIM < 3 ? A(1) : cc < 0 ? st.w[2][0] : cc == 0 ? st.w[2][1] : st.w[2][2];
#pragma unroll
              for (int bb = -1; bb <= 1; ++bb) {
                const A wbc = st.w[1][bb + 1] * wz;
#pragma unroll
                for (int a = -1; a <= 1; ++a) {
                  const A wt = st.w[0][a + 1] * wbc;
                  const GasCell<TG> g = gas[r0 + a + RX * (bb + RY * cc)];
                  if (drag_mode == DRAG_EPSTEIN) rg += wt * A(g.v[3]);
#pragma unroll
                  for (int d = 0; d < NC; ++d) {
                    if constexpr (MODE == SORTED_SOURCE) v[d] += wt * (A(g.v[d]) * w.sc[d] - mom[d]);
                    else v[d] += wt * A(g.v[d]);
                  }
                }
              }
            }
            const A it = drag_mode == DRAG_EPSTEIN
                             ? rg / dval
                             : inverse_tau<A, GEOM>(f, drag_mode, dval, A(sp->inv_tau[spc]), w);
            if constexpr (MODE == SORTED_SOURCE) {
              const A kq = m * (it < dt ? it : dt);   // dt: the reciprocal of the step here
#pragma unroll
              for (int d = 0; d < NC; ++d) q[d] = -(kq * v[d]);
            } else {
              A sl[3] = {v[0] * w.sc[0] - mom[0], v[1] * w.sc[1] - mom[1], NC > 2 ? v[2] * w.sc[2] - mom[2] : A(0)};
              A c, psi;
              propagator<A>(dt * it, c, psi);
              KickOut<A> o;
              kick_any<A, GEOM, NDIM>(B, f, dt, it, c, psi, w, mom, sl, o);
              bool fin = isfinite(double(o.e));
#pragma unroll
              for (int d = 0; d < NC; ++d) {
                const A vbar = (mom[d] + A(0.5) * o.dp[d]) / w.sc[d];
                const A dl = cell_width<A, U>(B.ax[d], idx[d]) * (GEOM == GEOM_CART || d == 0 ? A(1) : w.sc[d]);
                const double cps = fabs(double(vbar * dt / dl));
                cells = cps > cells ? cps : cells;
                mom[d] += o.dp[d];
                fin &= isfinite(double(mom[d]));
                in.rec[i].mom[d] = TS(mom[d]);
                q[d] = -(m * o.j[d]);
                sum[d] -= double(q[d]);
                sum[4] += fabs(double(q[d]));
              }
              q[NC] = -(m * o.e);
              sum[3] -= double(q[NC]);
              flags |= fin ? 0u : (uint32_t)DUST_FLAG_NONFINITE;
            }
          }
        }
      }
      run_sums<A, NDIM, NCH>(win, RX, RY, WC, rec, r0, has, q, st);
      done += cnt;
    }
  }
  __syncthreads();
  if (kend) window_to_grid();
  if (dg && flags) atomicOr(&dg->flags, (unsigned)flags);
  if constexpr (MODE == SORTED_STEP) {
    if (dg && sums) {
      // one set of atomics per workgroup
      __shared__ double red[SORTED_THREADS / 64][6];
#pragma unroll
      for (int k = 0; k < 5; ++k) sum[k] = wave_sum(sum[k]);
      cells = wave_max(cells);
      if ((tid & 63) == 0) {
#pragma unroll
        for (int k = 0; k < 5; ++k) red[tid >> 6][k] = sum[k];
        red[tid >> 6][5] = cells;
      }
      __syncthreads();
      if (tid == 0) {
        double t[6];
        for (int k = 0; k < 6; ++k) {
          t[k] = red[0][k];
          for (int w = 1; w < SORTED_THREADS / 64; ++w) t[k] = k == 5 ? fmax(t[k], red[w][k]) : t[k] + red[w][k];
        }
        for (int k = 0; k < 3; ++k) unsafeAtomicAdd(&dg->p_part[k], t[k]);
        unsafeAtomicAdd(&dg->e_part, t[3]);
        unsafeAtomicAdd(&dg->sum_abs_j, t[4]);
        atomic_max_nonneg(&dg->max_cells_bits, t[5]);
        if (t[5] > 1.8) atomicOr(&dg->flags, (unsigned)DUST_FLAG_CFL);
      }
    }
  }
}

// The two half drifts of the unfused step around launch_sorted (SORTED_STEP).
// In between, a particle's state is one packed record: the sorted pass reads
// it in an order that has nothing to do with the arrays', and nine arrays
// would cost it nine lines of memory per particle (5 GB for 4.3 M particles).
// First drift: arrays to records and sort keys (nbins without a cell; a
// particle that leaves through an open face loses its cell here).  Second
// drift: records to arrays.
template <typename TS, typename A, int GEOM, int NDIM, bool U>
__global__ void __launch_bounds__(256)
    k_step_pack(PView<TS> p, const Box* __restrict__ boxes, int nbox, Forces f, A h,
                const double* __restrict__ tdev, double toff, StepRecord<TS>* __restrict__ rec,
                uint32_t* __restrict__ key, uint32_t nbins, DiagDev* dg) {
  constexpr int NC = GEOM == GEOM_CART ? NDIM : 3;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= p.n) return;
  StepRecord<TS> r{};
  r.cell = -1;
  uint32_t k = nbins;
  int idx[3];
  A off[3], mom[3];
  const int b = load_particle<TS, A, GEOM, NDIM>(p, boxes, nbox, i, idx, off, mom, dg);
  if (b >= 0) {
    const Box& B = boxes[b];
    const double t = *tdev + toff;
    bool alive = drift_any<A, GEOM, NDIM, U>(B, f, true, h, t, idx, off, mom);
    TS o[3] = {TS(0), TS(0), TS(0)};
    if (alive)
      alive = GEOM == GEOM_CART && NDIM == 3 && f.kind == FORCE_FARGO
                  ? finalize<TS, A, GEOM, NDIM, GEOM == GEOM_CART>(B, f, t, idx, off, mom, o)
                  : finalize<TS, A, GEOM, NDIM, false>(B, f, t, idx, off, mom, o);
    if (alive) {
      r.cell = (int32_t)(B.cell_base + ravel(B, idx));
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        r.off[d] = d < NDIM ? o[d] : TS(0);
        r.mom[d] = d < NC ? TS(mom[d]) : TS(0);
      }
      r.species = p.species ? p.species[i] : 0;
      r.drag = p.drag ? p.drag[i] : TS(1);
      r.mass = p.mass ? p.mass[i] : TS(0);
      k = tile_key_idx(B, idx, TileShape{{sorted_tile_extent(NDIM, 0), sorted_tile_extent(NDIM, 1),
                                          sorted_tile_extent(NDIM, 2)}});
    } else {
      p.cell[i] = -1;
      if (dg) {
        atomicAdd(&dg->n_removed, 1ull);
        atomicOr(&dg->flags, (unsigned)DUST_FLAG_LEFT_OPEN);
      }
    }
  }
  rec[i] = r;
  key[i] = k;
}

template <typename TS, typename A, int GEOM, int NDIM, bool U>
__global__ void __launch_bounds__(256)
    k_step_unpack(PView<TS> p, const Box* __restrict__ boxes, int nbox, Forces f, A h,
                  const double* __restrict__ tdev, double toff, const StepRecord<TS>* __restrict__ rec, DiagDev* dg) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= p.n) return;
  const StepRecord<TS> r = rec[i];
  if (r.cell < 0) return;
  const Box& B = boxes[find_box(boxes, nbox, r.cell)];
  int idx[3];
  A off[3], mom[3];
  unravel(B, r.cell - B.cell_base, idx);
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    off[d] = A(r.off[d]);
    mom[d] = A(r.mom[d]);
  }
  const double t = *tdev + toff;
  const bool alive = drift_any<A, GEOM, NDIM, U>(B, f, false, h, t, idx, off, mom);
  if (!alive) {
    // (it keeps the state at the end of the kick)
    constexpr int NC = GEOM == GEOM_CART ? NDIM : 3;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      if (d < NDIM) p.off[d][i] = r.off[d];
      if (d < NC) p.mom[d][i] = r.mom[d];
    }
  }
  store_particle_any<TS, A, GEOM, NDIM>(p, B, f, t, i, alive, idx, off, mom, dg);
}

#define DUST_STEP_SWITCH(KERN, ...)                                                                             \
  do {                                                                                                          \
    const dim3 g_((unsigned)((p.n + 255) / 256)), b_(256);                                                      \
    if (geom == GEOM_CART && ndim == 2 && unif)                                                                 \
      hipLaunchKernelGGL((KERN<TS, A, GEOM_CART, 2, true>), g_, b_, 0, st, __VA_ARGS__);                        \
    else if (geom == GEOM_CART && ndim == 2)                                                                    \
      hipLaunchKernelGGL((KERN<TS, A, GEOM_CART, 2, false>), g_, b_, 0, st, __VA_ARGS__);                       \
    else if (geom == GEOM_CART && unif)                                                                         \
      hipLaunchKernelGGL((KERN<TS, A, GEOM_CART, 3, true>), g_, b_, 0, st, __VA_ARGS__);                        \
    else if (geom == GEOM_CART)                                                                                 \
      hipLaunchKernelGGL((KERN<TS, A, GEOM_CART, 3, false>), g_, b_, 0, st, __VA_ARGS__);                       \
    else if (geom == GEOM_CYL)                                                                                  \
      hipLaunchKernelGGL((KERN<TS, A, GEOM_CYL, 3, false>), g_, b_, 0, st, __VA_ARGS__);                        \
    else                                                                                                        \
      hipLaunchKernelGGL((KERN<TS, A, GEOM_SPH, 3, false>), g_, b_, 0, st, __VA_ARGS__);                        \
  } while (0)

template <typename TS, typename A>
void launch_step_pack(const PView<TS>& p, const Box* boxes, int nbox, int geom, int ndim, int unif,
                      const Forces& f, double h, const double* tdev, double toff, StepRecord<TS>* rec,
                      uint32_t* key, int64_t nbins, DiagDev* dg, hipStream_t st) {
  if (p.n == 0) return;
  DUST_STEP_SWITCH(k_step_pack, p, boxes, nbox, f, A(h), tdev, toff, rec, key, (uint32_t)nbins, dg);
}
template <typename TS, typename A>
void launch_step_unpack(const PView<TS>& p, const Box* boxes, int nbox, int geom, int ndim, int unif,
                        const Forces& f, double h, const double* tdev, double toff, const StepRecord<TS>* rec,
                        DiagDev* dg, hipStream_t st) {
  if (p.n == 0) return;
  DUST_STEP_SWITCH(k_step_unpack, p, boxes, nbox, f, A(h), tdev, toff, rec, dg);
}

template <typename TS, typename A, typename TW, int MODE>
void launch_sorted(const PView<TS>& p, const Box* boxes, int nbox, int geom, int ndim, int unif,
                   const FView<TS>& fl, const SortedIn<TS, TW>& in, const double* xg, const Forces& f,
                   const Species* sp, int drag_mode, double dt, const uint32_t* key, const uint32_t* perm,
                   int64_t nbins, DiagDev* dg, bool sums, hipStream_t st) {
  if (p.n == 0) return;
  // slots per workgroup: up to 4096 (few window flushes), fewer while the
  // launch would not give every CU several workgroups
  int64_t ppb = (p.n / 2048 + SORTED_THREADS - 1) / SORTED_THREADS * SORTED_THREADS;
  ppb = ppb < SORTED_THREADS ? SORTED_THREADS : ppb > 4096 ? 4096 : ppb;
  const unsigned nb = (unsigned)((p.n + ppb - 1) / ppb);
#define DUST_S(G_, D_, U_)                                                                                \
  hipLaunchKernelGGL((k_sorted<TS, A, TW, G_, D_, U_, MODE>), dim3(nb), dim3(SORTED_THREADS), 0, st, p,    \
                     boxes, nbox, fl, in, xg, f, sp, drag_mode, A(dt), key, perm, (uint32_t)nbins, (int)ppb, \
                     dg, (int)sums)
  if (geom == GEOM_CART && ndim == 2 && unif) DUST_S(GEOM_CART, 2, true);
  else if (geom == GEOM_CART && ndim == 2) DUST_S(GEOM_CART, 2, false);
  else if (geom == GEOM_CART && unif) DUST_S(GEOM_CART, 3, true);
  else if (geom == GEOM_CART) DUST_S(GEOM_CART, 3, false);
  else if (geom == GEOM_CYL) DUST_S(GEOM_CYL, 3, false);
  else DUST_S(GEOM_SPH, 3, false);
#undef DUST_S
}

#define DUST_SORTED_INST(TS, A, TW, MODE)                                                                  \
  template void launch_sorted<TS, A, TW, MODE>(                                                            \
      const PView<TS>&, const Box*, int, int, int, int, const FView<TS>&, const SortedIn<TS, TW>&, const double*, \
      const Forces&, const Species*, int, double, const uint32_t*, const uint32_t*, int64_t, DiagDev*, bool, \
      hipStream_t);

#define DUST_SORTED_STEP_INST(TS, A)                                                                         \
  DUST_SORTED_INST(TS, A, TS, SORTED_STEP)                                                                   \
  template void launch_step_pack<TS, A>(const PView<TS>&, const Box*, int, int, int, int, const Forces&,     \
                                        double, const double*, double, StepRecord<TS>*, uint32_t*, int64_t,  \
                                        DiagDev*, hipStream_t);                                              \
  template void launch_step_unpack<TS, A>(const PView<TS>&, const Box*, int, int, int, int, const Forces&,   \
                                          double, const double*, double, const StepRecord<TS>*, DiagDev*,    \
                                          hipStream_t);

}  // namespace dust
