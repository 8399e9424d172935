// Unfused per-phase kernels of the dust hot path (gfx950): drift, gather,
// exponential-midpoint kick, deposit, ghost fill / fold, feedback and FP64
// conservation sums.  One thread per particle (or per grid cell); all the
// per-particle arithmetic lives in dust_device.h and is shared with the
// fused kernel.
#include "dust_device.h"
#include "dust_fused_kern.h"
#include "dust_launch.h"
#include "dust_particle.h"

namespace dust {

// ---------------------------------------------------------------- particle kernels
// Templated on the geometry and dimension of the context's boxes so that the
// stencil and component loops unroll into registers.

template <typename TS, typename A, int GEOM, int NDIM, bool U>
__global__ void __launch_bounds__(256) k_drift(PView<TS> p, const Box* boxes, int nbox, Forces f,
                                               A h, const double* tdev, double toff, int first,
                                               DiagDev* dg) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= p.n) return;
  const double t_after = *tdev + toff;
  int idx[3];
  A off[3], mom[3];
  int b = load_particle<TS, A, GEOM, NDIM>(p, boxes, nbox, i, idx, off, mom, dg);
  if (b < 0) return;
  const Box& B = boxes[b];
  bool alive = drift_any<A, GEOM, NDIM, U>(B, f, first != 0, h, t_after, idx, off, mom);
  store_particle_any<TS, A, GEOM, NDIM>(p, B, f, t_after, i, alive, idx, off, mom, dg);
}

template <typename TS, typename A, typename TW, int GEOM, int NDIM, bool U>
__global__ void __launch_bounds__(256) k_gather(PView<TS> p, const Box* boxes, int nbox,
                                                FView<TS> fl, const double* xg, TW* rho_p,
                                                TW* vg0, TW* vg1, TW* vg2, DiagDev* dg) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= p.n) return;
  int idx[3];
  A off[3], mom[3];
  int b = load_particle<TS, A, GEOM, NDIM>(p, boxes, nbox, i, idx, off, mom, dg);
  if (b < 0) return;
  const Box& B = boxes[b];
  Stencil<A> s;
  stencil_weights<A, GEOM, NDIM, U>(B, idx, off, s);
  constexpr int nc = GEOM == GEOM_CART ? NDIM : 3;
  constexpr int c2 = NDIM > 2 ? 1 : 0;
  A r = A(0), v[3] = {A(0), A(0), A(0)};
#pragma unroll
  for (int c = -c2; c <= c2; ++c)
#pragma unroll
    for (int bb = -1; bb <= 1; ++bb) {
      A wbc = s.w[1][bb + 1] * s.w[2][c + 1];
#pragma unroll
      for (int a = -1; a <= 1; ++a) {
        A w = s.w[0][a + 1] * wbc;
        int64_t id = stored_index(B, idx[0] + a, idx[1] + bb, idx[2] + c);
        if (rho_p) r += w * A(fl.rho[id]);
#pragma unroll
        for (int m = 0; m < nc; ++m) v[m] += w * A(gas_comp(B, fl, xg, m, idx[0] + a, idx[1] + bb, idx[2] + c));
      }
    }
  if (rho_p) rho_p[i] = TW(r);
  if (vg0) vg0[i] = TW(v[0]);
  if (vg1) vg1[i] = TW(v[1]);
  if (nc > 2 && vg2) vg2[i] = TW(v[2]);
}

// Workgroups of the kick: a grid-stride loop, so that the diagnostic sums
// take one set of atomics per workgroup.  One per wave, as before, had 64
// particles share five contended FP64 atomics: 6.5 ms for 8.5 M particles,
// of which the particles' own traffic is 0.1 ms.
static constexpr int KICK_BLOCKS = 1024;

template <typename TS, typename A, typename TW, int GEOM, int NDIM, bool U>
__global__ void __launch_bounds__(256) k_kick(PView<TS> p, const Box* boxes, int nbox, Forces f,
                                              const Species* sp, int drag_mode, A dt, const TW* rho_p,
                                              const TW* vg0,
                                              const TW* vg1, const TW* vg2, TW* imp0, TW* imp1,
                                              TW* imp2, TW* imp3, DiagDev* dg, double* part) {
  constexpr int nc = GEOM == GEOM_CART ? NDIM : 3;
  double sums[5] = {0, 0, 0, 0, 0};
  double cells = 0.0;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < p.n; i += stride) {
    int idx[3];
    A off[3], mom[3];
    int b = load_particle<TS, A, GEOM, NDIM>(p, boxes, nbox, i, idx, off, mom, dg);
    if (b >= 0) {
      const Box& B = boxes[b];
      Where<A> w;
      where<A, GEOM, NDIM, U>(B, idx, off, w);
      // slip: canonical gas momentum at the particle minus p
      A sl[3] = {A(vg0[i]) * w.sc[0] - mom[0], A(vg1[i]) * w.sc[1] - mom[1],
                 nc > 2 ? A(vg2[i]) * w.sc[2] - mom[2] : A(0)};
      int s = p.species ? p.species[i] : 0;
      if (s >= sp->n) {
        flag(dg, DUST_FLAG_BAD_CELL);
        s = 0;
      }
      A dval = drag_mode == DRAG_SPECIES ? A(1) : A(p.drag[i]);
      A m = p.mass ? A(p.mass[i]) : A(sp->mass[s]);
      // Epstein: tau = C / rho_g with the density gathered at x^{n+1/2}
      A it = drag_mode == DRAG_EPSTEIN ? A(rho_p[i]) / dval
                                       : inverse_tau<A, GEOM>(f, drag_mode, dval, A(sp->inv_tau[s]), w);
      A c, psi;
      propagator<A>(dt * it, c, psi);
      KickOut<A> o;
      kick_any<A, GEOM, NDIM>(B, f, dt, it, c, psi, w, mom, sl, o);
      TW* imp[4] = {imp0, imp1, imp2, imp3};
      bool fin = isfinite(double(o.e));
#pragma unroll
      for (int k = 0; k < nc; ++k) {
        A vbar = (mom[k] + A(0.5) * o.dp[k]) / w.sc[k];
        A dl = cell_width<A, U>(B.ax[k], idx[k]) * (GEOM == GEOM_CART || k == 0 ? A(1) : w.sc[k]);
        double cps = fabs(double(vbar * dt / dl));
        cells = cps > cells ? cps : cells;
        mom[k] += o.dp[k];
        fin &= isfinite(double(mom[k]));
        p.mom[k][i] = TS(mom[k]);
        if (imp[k]) imp[k][i] = TW(m * o.j[k]);
        sums[k] += double(m * o.j[k]);
        sums[4] += fabs(double(m * o.j[k]));
      }
      if (imp[nc]) imp[nc][i] = TW(m * o.e);
      sums[3] += double(m * o.e);
      if (!fin) flag(dg, DUST_FLAG_NONFINITE);
    }
  }
  if (dg) {
    __shared__ double red[4][6];
#pragma unroll
    for (int k = 0; k < 5; ++k) sums[k] = wave_sum(sums[k]);
    cells = wave_max(cells);
    if ((threadIdx.x & 63) == 0) {
      for (int k = 0; k < 5; ++k) red[threadIdx.x >> 6][k] = sums[k];
      red[threadIdx.x >> 6][5] = cells;
    }
    __syncthreads();
    // the block's sums in a fixed order: into its slot of part (deterministic,
    // added up by k_reduce_kick_partials), else to the diagnostics
    if (threadIdx.x < 5) {
      const int k = threadIdx.x;
      const double v = ((red[0][k] + red[1][k]) + red[2][k]) + red[3][k];
      if (part) part[(size_t)blockIdx.x * 5 + k] = v;
      else unsafeAtomicAdd(k < 3 ? &dg->p_part[k] : k == 3 ? &dg->e_part : &dg->sum_abs_j, v);
    }
    if (threadIdx.x == 0) {
      const double c = fmax(fmax(red[0][5], red[1][5]), fmax(red[2][5], red[3][5]));
      atomic_max_nonneg(&dg->max_cells_bits, c);
      if (c > 1.8) atomicOr(&dg->flags, (unsigned)DUST_FLAG_CFL);
    }
  }
}

// Sum of the kick's per-block partials (5 per block) in a fixed order, added
// to the diagnostics.
__global__ void __launch_bounds__(256)
    k_reduce_kick_partials(const double* __restrict__ part, int64_t nblocks, DiagDev* dg) {
  __shared__ double red[256][5];
  double acc[5] = {0, 0, 0, 0, 0};
  for (int64_t b = threadIdx.x; b < nblocks; b += 256)
#pragma unroll
    for (int k = 0; k < 5; ++k) acc[k] += part[(size_t)b * 5 + k];
#pragma unroll
  for (int k = 0; k < 5; ++k) red[threadIdx.x][k] = acc[k];
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if (threadIdx.x < h)
      for (int k = 0; k < 5; ++k) red[threadIdx.x][k] += red[threadIdx.x + h][k];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    for (int k = 0; k < 3; ++k) dg->p_part[k] += red[0][k];
    dg->e_part += red[0][3];
    dg->sum_abs_j += red[0][4];
  }
}

template <typename TS, typename A, typename TW, int GEOM, int NDIM, bool U>
__global__ void __launch_bounds__(256) k_deposit(PView<TS> p, const Box* boxes, int nbox,
                                                 FView<TS> fl, const TW* imp0, const TW* imp1,
                                                 const TW* imp2, const TW* imp3, DiagDev* dg) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= p.n) return;
  int idx[3];
  A off[3], mom[3];
  int b = load_particle<TS, A, GEOM, NDIM>(p, boxes, nbox, i, idx, off, mom, dg);
  if (b < 0) return;
  const Box& B = boxes[b];
  constexpr int nc = GEOM == GEOM_CART ? NDIM : 3;
  A q[4] = {A(imp0[i]), A(imp1[i]), A(imp2[i]), A(0)};
  if (nc > 2) q[3] = A(imp3[i]);
  Stencil<A> s;
  stencil_weights<A, GEOM, NDIM, U>(B, idx, off, s);
  constexpr int c2 = NDIM > 2 ? 1 : 0;
#pragma unroll
  for (int c = -c2; c <= c2; ++c)
#pragma unroll
    for (int bb = -1; bb <= 1; ++bb) {
      A wbc = s.w[1][bb + 1] * s.w[2][c + 1];
#pragma unroll
      for (int a = -1; a <= 1; ++a) {
        int ii = idx[0] + a, jj = idx[1] + bb, kk = idx[2] + c;
        A w = s.w[0][a + 1] * wbc * A(inv_volume(B, ii, jj, kk));
        int64_t id = stored_index(B, ii, jj, kk);
#pragma unroll
        for (int k = 0; k <= nc; ++k) unsafeAtomicAdd(&fl.dep[k][id], TS(-w * q[k]));
      }
    }
}

// Deposit without float atomics, for the deterministic mode (the step's
// Eq. dust_feedback_final, the predictor's drag source, the dust density):
// one thread per stored cell (active or ghost) of box B sums W q / dV of
// the particles whose stencil covers the cell -- those of the 3^d active
// cells around it, the offsets in a fixed order and each cell's particles
// in the order of a stable sort by cell (perm, bin_start over the global
// cell ids) -- in FP64, for the nch channels q0.. (per particle), and adds
// sgn times the sums to out.dep[0..nch).  Every word has one writer and a
// fixed summation order, so the result is the same bits on every run.
template <typename TS, typename A, typename TW, int GEOM, int NDIM, bool U>
__global__ void __launch_bounds__(256)
    k_deposit_pull(PView<TS> p, Box B, FView<TS> fl, int nch, double sgn, const TW* imp0, const TW* imp1,
                   const TW* imp2, const TW* imp3, const uint32_t* __restrict__ perm,
                   const int64_t* __restrict__ bin_start) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= B.nstore) return;
  constexpr int c2 = NDIM > 2 ? 1 : 0;
  const int i = (int)(t % B.g0) - 1;
  const int j = (int)((t / B.g0) % B.g1) - 1;
  const int k = (int)(t / ((int64_t)B.g0 * B.g1)) - B.k_off;
  const int n0 = B.ax[0].n, n1 = B.ax[1].n, n2 = NDIM > 2 ? B.ax[2].n : 1;
  const TW* imp[4] = {imp0, imp1, imp2, imp3};
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  // this cell is the particle's host cell shifted by (a, bb, c)
  for (int c = -c2; c <= c2; ++c) {
    const int sk = k - c;
    if (sk < 0 || sk >= n2) continue;
    for (int bb = -1; bb <= 1; ++bb) {
      const int sj = j - bb;
      if (sj < 0 || sj >= n1) continue;
      for (int a = -1; a <= 1; ++a) {
        const int si = i - a;
        if (si < 0 || si >= n0) continue;
        int src[3] = {si, sj, sk};
        const int64_t cid = B.cell_base + ravel(B, src);
        const int64_t e = bin_start[cid + 1];
        for (int64_t s = bin_start[cid]; s < e; ++s) {
          const int64_t ip = perm[s];
          A off[3];
#pragma unroll
          for (int d = 0; d < 3; ++d) off[d] = d < NDIM ? A(p.off[d][ip]) : A(0);
          Stencil<A> sw;
          stencil_weights<A, GEOM, NDIM, U>(B, src, off, sw);
          const double w = double(sw.w[0][a + 1] * sw.w[1][bb + 1] * sw.w[2][c + 1]);
#pragma unroll
          for (int m = 0; m < 4; ++m)
            if (m < nch) acc[m] += w * double(imp[m][ip]);
        }
      }
    }
  }
  const double iv = inv_volume(B, i, j, k);
  const int64_t id = B.store_base + t;
#pragma unroll
  for (int m = 0; m < 4; ++m)
    if (m < nch) fl.dep[m][id] = TS(double(fl.dep[m][id]) + sgn * (acc[m] * iv));
}

// Per-particle coefficients for the deterministic drag source and dust
// density (deposited by k_deposit_pull): q_m = m min(1/tau, 1/dt) times the
// slip sum_i W_i (s_m v_i - p_m), as ds_particles forms them (Epstein: tau
// from the gathered gas density), or the particle mass (MASS); zero for a
// particle without a cell (which no bin holds).
template <typename TS, typename A, int GEOM, int NDIM, bool U, bool MASS>
__global__ void __launch_bounds__(256)
    k_source_coeffs(PView<TS> p, const Box* boxes, int nbox, FView<TS> fl, Forces f, const Species* sp,
                    int drag_mode, A inv_dt, A* q0, A* q1, A* q2, DiagDev* dg) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= p.n) return;
  constexpr int nc = MASS ? 1 : (GEOM == GEOM_CART ? NDIM : 3);
  constexpr int c2 = NDIM > 2 ? 1 : 0;
  A* q[3] = {q0, q1, q2};
  int idx[3];
  A off[3], mom[3] = {A(0), A(0), A(0)};
  const int b = MASS ? load_position<TS, A, NDIM>(p, boxes, nbox, i, idx, off, dg)
                     : load_particle<TS, A, GEOM, NDIM>(p, boxes, nbox, i, idx, off, mom, dg);
  A out[3] = {A(0), A(0), A(0)};
  if (b >= 0) {
    const Box& B = boxes[b];
    int sidx = p.species ? p.species[i] : 0;
    if (sidx >= sp->n) {
      flag(dg, DUST_FLAG_BAD_CELL);
      sidx = 0;
    }
    const A m = p.mass ? A(p.mass[i]) : A(sp->mass[sidx]);
    if constexpr (MASS) {
      out[0] = m;
    } else {
      Stencil<A> s;
      stencil_weights<A, GEOM, NDIM, U>(B, idx, off, s);
      Where<A> w;
      where<A, GEOM, NDIM, U>(B, idx, off, w);
      A sl[3] = {A(0), A(0), A(0)};
      A rg = A(0);
#pragma unroll
      for (int cc = -c2; cc <= c2; ++cc)
#pragma unroll
        for (int bb = -1; bb <= 1; ++bb) {
          const A wbc = s.w[1][bb + 1] * s.w[2][cc + 1];
#pragma unroll
          for (int a = -1; a <= 1; ++a) {
            const A wt = s.w[0][a + 1] * wbc;
            if (drag_mode == DRAG_EPSTEIN)
              rg += wt * A(fl.rho[stored_index(B, idx[0] + a, idx[1] + bb, idx[2] + cc)]);
#pragma unroll
            for (int mm = 0; mm < nc; ++mm)
              sl[mm] += wt * (A(gas_comp(B, fl, nullptr, mm, idx[0] + a, idx[1] + bb, idx[2] + cc)) * w.sc[mm] -
                              mom[mm]);
          }
        }
      const A dval = drag_mode == DRAG_SPECIES ? A(1) : A(p.drag[i]);
      const A it = drag_mode == DRAG_EPSTEIN ? rg / dval
                                             : inverse_tau<A, GEOM>(f, drag_mode, dval, A(sp->inv_tau[sidx]), w);
      const A k = m * (it < inv_dt ? it : inv_dt);
#pragma unroll
      for (int mm = 0; mm < nc; ++mm) out[mm] = k * sl[mm];
    }
  }
#pragma unroll
  for (int mm = 0; mm < nc; ++mm) q[mm][i] = out[mm];
}

// Drag source of the gas predictor (Sec. 3.1, Eq. Delta_vp and f_D): at the
// particle's current position, the canonical slip between the weighted gas
// velocity and the particle, times m / max(tau, dt) (the stiffness limiter
// of Bai & Stone 2010), subtracted from the momentum channels with the
// gather's weights over the cell volume.  inv_dt = 1/dt.
// Each thread takes DS_PPT particles 64 slots apart (a workgroup covers
// 256 * DS_PPT consecutive slots) and sums the contributions of consecutive
// ones with the same host cell in registers (the particles of a cell sit 64
// slots apart in the level-major layout of the fused step), so a cell's
// stencil is deposited once per run instead of once per particle.  Where
// the workgroup's particles share a box and their stencils fit a window of
// ds_win_cells<TS>() cells, the box is workgroup-uniform, the window's gas
// velocity is staged in LDS, the gathers read it there, the deposits go to
// an FP64 LDS window (FP64 LDS atomics run ~20x faster than FP32 ones on
// gfx950) and that window is added to HBM once; otherwise gathers and
// deposits go to HBM.  Correct for any particle order.
static constexpr int DS_PPT = 4;
// window capacity in cells: 3 FP64 deposit channels + 3 gas components in
// storage precision within 64 KiB of LDS
template <typename TS> constexpr int ds_win_cells() { return sizeof(TS) == 4 ? 1600 : 1300; }

struct DsWindow {
  int o[3], ext[3];
  int64_t cells;
};

// Host cell and offsets of particle i (the dust density needs no momenta):
// the box index, or -1 without a cell (flags as load_particle).
template <typename TS, typename A, int NDIM>
__device__ __forceinline__ int load_position(const PView<TS>& p, const Box* boxes, int nbox, int64_t i,
                                             int idx[3], A off[3], DiagDev* dg) {
  const int64_t c = p.cell[i];
  if (c < 0) return -1;
  const int b = find_box(boxes, nbox, c);
  const Box& B = boxes[b];
  if (c >= B.cell_base + B.ncell) {
    flag(dg, DUST_FLAG_BAD_CELL);
    return -1;
  }
  unravel(B, c - B.cell_base, idx);
  bool bad = false;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    off[d] = d < NDIM ? A(p.off[d][i]) : A(0);
    bad |= !(off[d] >= A(-0.5) && off[d] < A(0.5));
  }
  if (bad) flag(dg, DUST_FLAG_OFFSET_RANGE);
  return b;
}

// The particles of one thread (see k_drag_source).  WIN: every particle
// with a cell lies in box ub (workgroup-uniform) inside window wd.
// MASS: the dust density instead (one channel, the particle mass, no gas).
// EPS: Epstein drag (stopping time from the gathered gas density).
template <typename TS, typename A, int GEOM, int NDIM, bool U, bool WIN, bool MASS, bool EPS>
__device__ __forceinline__ void ds_particles(const PView<TS>& p, const Box* boxes, int nbox, int ub,
                                             const FView<TS>& fl, const Forces& f, const Species* sp,
                                             int drag_mode, A inv_dt, DiagDev* dg, int64_t base,
                                             double* win, const TS* gwin, const DsWindow& wd) {
  constexpr int nc = MASS ? 1 : (GEOM == GEOM_CART ? NDIM : 3);
  constexpr int c2 = NDIM > 2 ? 1 : 0;
  constexpr int NT = NDIM > 2 ? 27 : 9;
  // register sums of the current run of particles with host cell `cur`
  A acc[NT][3];
  int64_t cur = -1;
  int cb = 0, cidx[3] = {0, 0, 0};
  auto flush = [&]() {
    const Box& B = WIN ? boxes[ub] : boxes[cb];
    double iv[3][3];
#pragma unroll
    for (int d = 0; d < 3; ++d)
#pragma unroll
      for (int a = 0; a < 3; ++a) iv[d][a] = d < NDIM ? B.ax[d].ivol[cidx[d] + a] : 1.0;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int a = t % 3, bb = (t / 3) % 3, cc = NDIM > 2 ? t / 9 : 1;
      const int ii = cidx[0] + a - 1, jj = cidx[1] + bb - 1, kk = cidx[2] + cc - 1;
      const A v = A(iv[0][a] * iv[1][bb] * iv[2][cc]);
      constexpr A sgn = MASS ? A(1) : A(-1);   // the drag source is subtracted
      if constexpr (WIN) {
        const int64_t e = (ii - wd.o[0]) + (int64_t)wd.ext[0] * ((jj - wd.o[1]) + (int64_t)wd.ext[1] * (kk - wd.o[2]));
#pragma unroll
        for (int m = 0; m < nc; ++m) atomicAdd(&win[m * wd.cells + e], double(sgn * acc[t][m] * v));
      } else {
        const int64_t id = stored_index(B, ii, jj, kk);
#pragma unroll
        for (int m = 0; m < nc; ++m) unsafeAtomicAdd(&fl.dep[m][id], TS(sgn * acc[t][m] * v));
      }
    }
  };
  for (int j = 0; j < DS_PPT; ++j) {
    const int64_t i = base + 64 * j;
    if (i >= p.n) break;
    int idx[3];
    A off[3], mom[3];
    int b;
    if constexpr (WIN) {
      // every particle with a valid cell is in box ub (the window test)
      const Box& B = boxes[ub];
      const int64_t c = p.cell[i];
      if (c < 0) continue;
      if (c < B.cell_base || c >= B.cell_base + B.ncell) {
        flag(dg, DUST_FLAG_BAD_CELL);
        continue;
      }
      unravel(B, c - B.cell_base, idx);
      constexpr int nm = MASS ? 0 : nc;
      bool bad = false, nonfinite = false;
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        off[d] = d < NDIM ? A(p.off[d][i]) : A(0);
        mom[d] = d < nm ? A(p.mom[d][i]) : A(0);
        bad |= !(off[d] >= A(-0.5) && off[d] < A(0.5));
        nonfinite |= !isfinite(double(mom[d]));
      }
      if (bad) flag(dg, DUST_FLAG_OFFSET_RANGE);
      if (nonfinite) flag(dg, DUST_FLAG_NONFINITE);
      b = ub;
    } else if constexpr (MASS) {
      b = load_position<TS, A, NDIM>(p, boxes, nbox, i, idx, off, dg);
      if (b < 0) continue;
    } else {
      b = load_particle<TS, A, GEOM, NDIM>(p, boxes, nbox, i, idx, off, mom, dg);
      if (b < 0) continue;
    }
    const Box& B = WIN ? boxes[ub] : boxes[b];
    const int64_t c = p.cell[i];
    if (c != cur) {
      if (cur >= 0) flush();
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int m = 0; m < 3; ++m) acc[t][m] = A(0);
      cur = c;
      cb = b;
      cidx[0] = idx[0];
      cidx[1] = idx[1];
      cidx[2] = idx[2];
    }
    Stencil<A> s;
    stencil_weights<A, GEOM, NDIM, U>(B, idx, off, s);
    A q[3] = {A(0), A(0), A(0)};
    if constexpr (MASS) {
      int sidx = p.species ? p.species[i] : 0;
      if (sidx >= sp->n) {
        flag(dg, DUST_FLAG_BAD_CELL);
        sidx = 0;
      }
      q[0] = p.mass ? A(p.mass[i]) : A(sp->mass[sidx]);
    } else {
      Where<A> w;
      where<A, GEOM, NDIM, U>(B, idx, off, w);
      // slip s_c v_g,c - p_c as a weighted sum of per-cell differences (keeps
      // its relative accuracy where the velocities are much larger than it)
      A sl[3] = {A(0), A(0), A(0)};
      A rg = A(0);   // gas density at the particle (Epstein drag)
      int64_t e0 = 0;
      if constexpr (WIN)
        e0 = (idx[0] - wd.o[0]) + (int64_t)wd.ext[0] * ((idx[1] - wd.o[1]) + (int64_t)wd.ext[1] * (idx[2] - wd.o[2]));
#pragma unroll
      for (int cc = -c2; cc <= c2; ++cc)
#pragma unroll
        for (int bb = -1; bb <= 1; ++bb) {
          A wbc = s.w[1][bb + 1] * s.w[2][cc + 1];
#pragma unroll
          for (int a = -1; a <= 1; ++a) {
            A wt = s.w[0][a + 1] * wbc;
            if constexpr (EPS) rg += wt * A(fl.rho[stored_index(B, idx[0] + a, idx[1] + bb, idx[2] + cc)]);
#pragma unroll
            for (int m = 0; m < nc; ++m) {
              A g;
              if constexpr (WIN)
                g = A(gwin[m * wd.cells + e0 + a + (int64_t)wd.ext[0] * (bb + (int64_t)wd.ext[1] * cc)]);
              else
                g = A(gas_comp(B, fl, nullptr, m, idx[0] + a, idx[1] + bb, idx[2] + cc));
              sl[m] += wt * (g * w.sc[m] - mom[m]);
            }
          }
        }
      int sidx = p.species ? p.species[i] : 0;
      if (sidx >= sp->n) {
        flag(dg, DUST_FLAG_BAD_CELL);
        sidx = 0;
      }
      A dval = drag_mode == DRAG_SPECIES ? A(1) : A(p.drag[i]);
      A m = p.mass ? A(p.mass[i]) : A(sp->mass[sidx]);
      A it;
      if constexpr (EPS)
        it = rg / dval;
      else
        it = inverse_tau<A, GEOM>(f, drag_mode, dval, A(sp->inv_tau[sidx]), w);
      A k = m * (it < inv_dt ? it : inv_dt);
#pragma unroll
      for (int mm = 0; mm < nc; ++mm) q[mm] = k * sl[mm];
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      A wt = s.w[0][t % 3] * s.w[1][(t / 3) % 3] * s.w[2][NDIM > 2 ? t / 9 : 1];
#pragma unroll
      for (int mm = 0; mm < nc; ++mm) acc[t][mm] += wt * q[mm];
    }
  }
  if (cur >= 0) flush();
}

// Window over the host cells [lo, hi] (plus one cell on each side) if it
// holds at most cap cells.
template <int NDIM>
__device__ __forceinline__ bool ds_window(const int lo[3], const int hi[3], int64_t cap, DsWindow& wd) {
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    wd.o[d] = d < NDIM ? lo[d] - 1 : 0;
    wd.ext[d] = d < NDIM ? hi[d] - lo[d] + 3 : 1;
  }
  wd.cells = (int64_t)wd.ext[0] * wd.ext[1] * wd.ext[2];
  return wd.cells <= cap;
}

template <typename TS, int NC, bool GAS>
__device__ __forceinline__ void ds_stage(const Box& B, const FView<TS>& fl, const DsWindow& wd, double* win,
                                         TS* gwin, int lane, int nlanes) {
  for (int64_t e = lane; e < wd.cells; e += nlanes) {
    int ii = wd.o[0] + (int)(e % wd.ext[0]);
    int jj = wd.o[1] + (int)((e / wd.ext[0]) % wd.ext[1]);
    int kk = wd.o[2] + (int)(e / ((int64_t)wd.ext[0] * wd.ext[1]));
    int64_t id = stored_index(B, ii, jj, kk);
#pragma unroll
    for (int m = 0; m < NC; ++m) {
      win[m * wd.cells + e] = 0.0;
      if constexpr (GAS) gwin[m * wd.cells + e] = fl.vel[m][id];
    }
  }
}

template <typename TS, int NC>
__device__ __forceinline__ void ds_add_window(const Box& B, const FView<TS>& fl, const DsWindow& wd,
                                              const double* win, int lane, int nlanes) {
  for (int64_t e = lane; e < wd.cells; e += nlanes) {
    int ii = wd.o[0] + (int)(e % wd.ext[0]);
    int jj = wd.o[1] + (int)((e / wd.ext[0]) % wd.ext[1]);
    int kk = wd.o[2] + (int)(e / ((int64_t)wd.ext[0] * wd.ext[1]));
    int64_t id = stored_index(B, ii, jj, kk);
#pragma unroll
    for (int m = 0; m < NC; ++m) {
      double v = win[m * wd.cells + e];
      if (v != 0.0) unsafeAtomicAdd(&fl.dep[m][id], TS(v));
    }
  }
}

// Windows: one for the workgroup when its particles' window fits the LDS
// capacity, else one per wave (a quarter of the capacity each) for the waves
// whose particles' window fits that; the other waves go to HBM.
template <typename TS, typename A, int GEOM, int NDIM, bool U, bool MASS, bool EPS>
__device__ __forceinline__ void ds_body(const PView<TS>& p, const Box* boxes, int nbox, const FView<TS>& fl,
                                        const Forces& f, const Species* sp, int drag_mode, A inv_dt,
                                        DiagDev* dg) {
  constexpr int nc = MASS ? 1 : (GEOM == GEOM_CART ? NDIM : 3);
  constexpr int CAP = ds_win_cells<TS>();
  __shared__ double win[3 * CAP];
  __shared__ TS gwin[3 * CAP];
  __shared__ int s_lo[4][3], s_hi[4][3], s_blo[4], s_bhi[4];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (lane == 0) {
    for (int d = 0; d < 3; ++d) {
      s_lo[wave][d] = 0x7fffffff;
      s_hi[wave][d] = -0x7fffffff;
    }
    s_blo[wave] = 0x7fffffff;
    s_bhi[wave] = -1;
  }
  __syncthreads();
  const int64_t base = (int64_t)blockIdx.x * (256 * DS_PPT) + (int64_t)wave * (64 * DS_PPT) + lane;
  // bounding box of each wave's host cells
  {
    int lo[3] = {0x7fffffff, 0x7fffffff, 0x7fffffff}, hi[3] = {-0x7fffffff, -0x7fffffff, -0x7fffffff};
    int blo = 0x7fffffff, bhi = -1;
    auto add = [&](const Box& B, int b, int64_t c) {
      if (c >= B.cell_base + B.ncell) return;
      int idx[3];
      unravel(B, c - B.cell_base, idx);
#pragma unroll
      for (int d = 0; d < NDIM; ++d) {
        lo[d] = idx[d] < lo[d] ? idx[d] : lo[d];
        hi[d] = idx[d] > hi[d] ? idx[d] : hi[d];
      }
      blo = b < blo ? b : blo;
      bhi = b > bhi ? b : bhi;
    };
    for (int j = 0; j < DS_PPT; ++j) {
      int64_t i = base + 64 * j;
      if (i >= p.n) break;
      int64_t c = p.cell[i];
      if (c < 0) continue;
      // one box: a uniform descriptor (scalar loads)
      if (nbox == 1)
        add(boxes[0], 0, c);
      else {
        const int b = find_box(boxes, nbox, c);
        add(boxes[b], b, c);
      }
    }
    if (bhi >= 0) {
#pragma unroll
      for (int d = 0; d < NDIM; ++d) {
        atomicMin(&s_lo[wave][d], lo[d]);
        atomicMax(&s_hi[wave][d], hi[d]);
      }
      atomicMin(&s_blo[wave], blo);
      atomicMax(&s_bhi[wave], bhi);
    }
  }
  __syncthreads();
  // workgroup window (uniform decision)
  int glo[3], ghi[3], gblo = 0x7fffffff, gbhi = -1;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    glo[d] = 0x7fffffff;
    ghi[d] = -0x7fffffff;
  }
  for (int w = 0; w < 4; ++w) {
    if (s_bhi[w] < 0) continue;
#pragma unroll
    for (int d = 0; d < NDIM; ++d) {
      glo[d] = s_lo[w][d] < glo[d] ? s_lo[w][d] : glo[d];
      ghi[d] = s_hi[w][d] > ghi[d] ? s_hi[w][d] : ghi[d];
    }
    gblo = s_blo[w] < gblo ? s_blo[w] : gblo;
    gbhi = s_bhi[w] > gbhi ? s_bhi[w] : gbhi;
  }
  DsWindow wd;
  const bool wg_win = gbhi >= 0 && gblo == gbhi && ds_window<NDIM>(glo, ghi, CAP * 3 / nc, wd);
  if (wg_win) {
    const int ub = __builtin_amdgcn_readfirstlane(gblo);
    const Box& B = boxes[ub];
    ds_stage<TS, nc, !MASS>(B, fl, wd, win, gwin, threadIdx.x, blockDim.x);
    __syncthreads();
    ds_particles<TS, A, GEOM, NDIM, U, true, MASS, EPS>(p, boxes, nbox, ub, fl, f, sp, drag_mode, inv_dt, dg, base,
                                             win, gwin, wd);
    __syncthreads();
    ds_add_window<TS, nc>(B, fl, wd, win, threadIdx.x, blockDim.x);
    return;   // uniform: the whole workgroup leaves here
  }
  // per-wave windows (each wave decides for itself; barriers stay uniform)
  int wlo[3], whi[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    wlo[d] = s_lo[wave][d];
    whi[d] = s_hi[wave][d];
  }
  const int qcap = CAP / 4;
  double* wwin = win + wave * 3 * qcap;
  TS* wgwin = gwin + wave * 3 * qcap;
  const bool w_win = s_bhi[wave] >= 0 && s_blo[wave] == s_bhi[wave] &&
                     ds_window<NDIM>(wlo, whi, qcap * 3 / nc, wd);
  const int ub = __builtin_amdgcn_readfirstlane(s_blo[wave]);
  if (w_win) ds_stage<TS, nc, !MASS>(boxes[ub], fl, wd, wwin, wgwin, lane, 64);
  __syncthreads();
  if (w_win)
    ds_particles<TS, A, GEOM, NDIM, U, true, MASS, EPS>(p, boxes, nbox, ub, fl, f, sp, drag_mode, inv_dt, dg, base,
                                             wwin, wgwin, wd);
  else
    ds_particles<TS, A, GEOM, NDIM, U, false, MASS, EPS>(p, boxes, nbox, 0, fl, f, sp, drag_mode, inv_dt, dg, base,
                                              wwin, wgwin, wd);
  __syncthreads();
  if (w_win) ds_add_window<TS, nc>(boxes[ub], fl, wd, wwin, lane, 64);
}

template <typename TS, typename A, int GEOM, int NDIM, bool U, bool EPS>
__global__ void __launch_bounds__(256) k_drag_source(PView<TS> p, const Box* boxes, int nbox,
                                                     FView<TS> fl, Forces f, const Species* sp,
                                                     int drag_mode, A inv_dt, DiagDev* dg) {
  ds_body<TS, A, GEOM, NDIM, U, false, EPS>(p, boxes, nbox, fl, f, sp, drag_mode, inv_dt, dg);
}

// Dust density: rho_d (fl.dep[0]) += m W / dV with the gather's weights.
template <typename TS, typename A, int GEOM, int NDIM, bool U>
__global__ void __launch_bounds__(256) k_mass_density(PView<TS> p, const Box* boxes, int nbox,
                                                      FView<TS> fl, const Species* sp, DiagDev* dg) {
  ds_body<TS, A, GEOM, NDIM, U, true, false>(p, boxes, nbox, fl, Forces{}, sp, DRAG_TAU, A(0), dg);
}

// Dispatch on the (geometry, dimension) shared by the context's boxes.
#define DUST_GEOM_SWITCH(geom, ndim, unif, CALL)                      \
  do {                                                                \
    if ((geom) == GEOM_CART && (ndim) == 2 && (unif)) {               \
      constexpr int G_ = GEOM_CART, D_ = 2;                           \
      constexpr bool U_ = true;                                       \
      CALL;                                                           \
    } else if ((geom) == GEOM_CART && (ndim) == 2) {                  \
      constexpr int G_ = GEOM_CART, D_ = 2;                           \
      constexpr bool U_ = false;                                      \
      CALL;                                                           \
    } else if ((geom) == GEOM_CART && (unif)) {                       \
      constexpr int G_ = GEOM_CART, D_ = 3;                           \
      constexpr bool U_ = true;                                       \
      CALL;                                                           \
    } else if ((geom) == GEOM_CART) {                                 \
      constexpr int G_ = GEOM_CART, D_ = 3;                           \
      constexpr bool U_ = false;                                      \
      CALL;                                                           \
    } else if ((geom) == GEOM_CYL) {                                  \
      constexpr int G_ = GEOM_CYL, D_ = 3;                            \
      constexpr bool U_ = false;                                      \
      CALL;                                                           \
    } else {                                                          \
      constexpr int G_ = GEOM_SPH, D_ = 3;                            \
      constexpr bool U_ = false;                                      \
      CALL;                                                           \
    }                                                                 \
  } while (0)

// ---------------------------------------------------------------- grid kernels
// Each ghost kernel treats several arrays of one box in one launch: the
// array is blockIdx.y.

template <typename TS> struct Arr4 {
  TS* a[4];
};

// One launch of a per-box kernel over several boxes: box[e] takes blocks
// [blk0[e], blk0[e+1]) of the grid (up to MB_BOXES boxes per launch); a
// block finds its entry by a scan of blk0 and reads its box descriptor from
// the device table (a block-uniform address).
static constexpr int MB_BOXES = 16;
static_assert(GRID_SUM_PARTS >= GRID_SUM_BLOCKS + MB_BOXES, "grid-sum partials");
struct BoxGrid {
  int n;
  int box[MB_BOXES];
  uint32_t blk0[MB_BOXES + 1];
};
__device__ __forceinline__ int grid_entry(const BoxGrid& g) {
  int e = 0;
  while (e + 1 < g.n && blockIdx.x >= g.blk0[e + 1]) ++e;
  return e;
}
// thread index within the box's range
__device__ __forceinline__ int64_t grid_thread(const BoxGrid& g, int e) {
  return (int64_t)(blockIdx.x - g.blk0[e]) * blockDim.x + threadIdx.x;
}

// The ghost cells of a box that boundary conditions fill or fold, in disjoint
// sets: z ghosts (all i, j), y ghosts (all i, active k), x ghosts (active j
// and k), of the axes whose faces are not open.
struct GhostSet {
  int n0, n1, n2, g0, g1;   // active cells; stored extents
  bool x, y, z;             // the axis has filled ghosts
  int64_t cx, cy, cz;       // cells of each set
};
__device__ __forceinline__ GhostSet ghost_set(const Box& B) {
  GhostSet s;
  s.n0 = B.ax[0].n;
  s.n1 = B.ax[1].n;
  s.n2 = B.ndim > 2 ? B.ax[2].n : 1;
  s.g0 = s.n0 + 2;
  s.g1 = s.n1 + 2;
  s.x = B.ax[0].bc_lo != BC_OPEN;
  s.y = B.ax[1].bc_lo == BC_PERIODIC;
  s.z = B.ndim > 2 && B.ax[2].bc_lo == BC_PERIODIC;
  s.cx = s.x ? 2 * (int64_t)s.n1 * s.n2 : 0;
  s.cy = s.y ? 2 * (int64_t)s.g0 * s.n2 : 0;
  s.cz = s.z ? 2 * (int64_t)s.g0 * s.g1 : 0;
  return s;
}
// t-th of them (t < cx + cy + cz), both sides of a face cell in turn last.
__device__ __forceinline__ void ghost_cell(const GhostSet& s, int64_t t, int& i, int& j, int& k) {
  if (t < s.cx) {
    const uint32_t half = (uint32_t)(s.cx / 2), u = (uint32_t)t, v = u < half ? u : u - half;
    i = u < half ? -1 : s.n0;
    k = (int)(v / (uint32_t)s.n1);
    j = (int)(v - (uint32_t)k * s.n1);
  } else if ((t -= s.cx) < s.cy) {
    const uint32_t half = (uint32_t)(s.cy / 2), u = (uint32_t)t, v = u < half ? u : u - half;
    j = u < half ? -1 : s.n1;
    k = (int)(v / (uint32_t)s.g0);
    i = (int)(v - (uint32_t)k * s.g0) - 1;
  } else {
    const uint32_t half = (uint32_t)(s.cz / 2), u = (uint32_t)(t - s.cy), v = u < half ? u : u - half;
    k = u < half ? -1 : s.n2;
    const int q = (int)(v / (uint32_t)s.g0);
    i = (int)(v - (uint32_t)q * s.g0) - 1;
    j = q - 1;
  }
}

// Shear-periodic x-ghost value of the row (j, k) of a field, FP64: the other
// face's active cells, interpolated in y.  (side 0: the ghost below x_lo,
// (x_{n-1}, y_j - s); 1: above x_hi, (x_0, y_j + s); dv: the boost of v_y.)
template <typename TS>
__device__ __forceinline__ double shear_ghost(const Box& B, const TS* a, const Shift& sh, int side, int j, int k,
                                              double dv) {
  const int n0 = B.ax[0].n, n1 = B.ax[1].n;
  const int jl = side ? j + sh.si : j - sh.si - (sh.sf > 0 ? 1 : 0);
  const double fr = side ? sh.sf : (sh.sf > 0 ? 1.0 - sh.sf : 0.0);
  const int i = side ? 0 : n0 - 1;
  const int j0 = ((jl % n1) + n1) % n1, j1 = ((jl + 1) % n1 + n1) % n1;
  const double v = (1.0 - fr) * double(a[stored_index(B, i, j0, k)]) + fr * double(a[stored_index(B, i, j1, k)]);
  return side ? v - dv : v + dv;
}

// What one step needs of the grid before its particles, in one launch (each
// of the five it replaces took 4 to 5 us on a small grid, whatever its work):
// the gas ghosts, the FP64 x-ghost gas of shear-periodic boxes, and cleared
// deposits.  A ghost cell takes its value from active cells directly: an
// image in z of an image in y of a row of the other x face is computed from
// that face, so no order among the ghosts is needed.
//
// Blocks of an entry: ghosts of rho and every velocity component, then the
// x-ghost layer of every component; past the last entry: deposits.
static constexpr int CLEAR_PER = 4;   // deposits that a thread clears
template <typename TS> struct Prepare {
  Arr4<TS> gas;        // rho, velocity components
  int na;              // arrays (0: no ghosts)
  double* xg;          // FP64 x-ghost layers, or null
  double qOmega, toff;
  const double* tdev;
  int boost;
  Arr4<TS> dep;        // to clear
  int nch;
  int64_t n;
};
__host__ __device__ __forceinline__ int64_t fill_cells(const Box& B) {
  const int64_t n0 = B.ax[0].n, n1 = B.ax[1].n, n2 = B.ndim > 2 ? B.ax[2].n : 1;
  return (B.ax[0].bc_lo != BC_OPEN ? 2 * n1 * n2 : 0) + (B.ax[1].bc_lo == BC_PERIODIC ? 2 * (n0 + 2) * n2 : 0) +
         (B.ndim > 2 && B.ax[2].bc_lo == BC_PERIODIC ? 2 * (n0 + 2) * (n1 + 2) : 0);
}
__host__ __device__ __forceinline__ int64_t xghost_cells(const Box& B) {
  return B.xg_base >= 0 ? (int64_t)(B.ax[1].n + 2) * (B.ax[2].n + 2) : 0;
}
__host__ __device__ __forceinline__ uint32_t blocks256(int64_t n) { return (uint32_t)((n + 255) / 256); }

template <typename TS> __global__ void __launch_bounds__(256) k_prepare(const Box* boxes, BoxGrid bg, Prepare<TS> pr) {
  if (blockIdx.x >= bg.blk0[bg.n]) {
    const uint32_t q = blockIdx.x - bg.blk0[bg.n], per = blocks256((pr.n + CLEAR_PER - 1) / CLEAR_PER);
    const uint32_t ch = q / per;
    TS* a = pr.dep.a[ch];
    const int64_t i0 = (int64_t)(q - ch * per) * (256 * CLEAR_PER) + threadIdx.x;
#pragma unroll
    for (int u = 0; u < CLEAR_PER; ++u)
      if (i0 + u * 256 < pr.n) a[i0 + u * 256] = TS(0);
    return;
  }
  const int e = grid_entry(bg);
  const Box& B = boxes[bg.box[e]];
  const uint32_t bf = blocks256(fill_cells(B));
  uint32_t q = blockIdx.x - bg.blk0[e];
  if (q < bf * (uint32_t)pr.na) {
    const int m = (int)(q / bf);
    const int64_t t = (int64_t)(q - (uint32_t)m * bf) * 256 + threadIdx.x;
    const GhostSet s = ghost_set(B);
    if (t >= s.cx + s.cy + s.cz) return;
    int i, j, k;
    ghost_cell(s, t, i, j, k);
    TS* a = pr.gas.a[m];
    const int64_t to = stored_index(B, i, j, k);
    if (s.z) k = k < 0 ? s.n2 - 1 : k >= s.n2 ? 0 : k;
    if (s.y) j = j < 0 ? s.n1 - 1 : j >= s.n1 ? 0 : j;
    // (an x ghost in a ghost row of an open y face is filled by nobody)
    const bool xgh = s.x && (i < 0 || i >= s.n0) && j >= 0 && j < s.n1;
    TS v;
    if (xgh && B.ax[0].bc_lo == BC_SHEAR) {
      const Shift sh = make_shift(B, pr.qOmega, *pr.tdev + pr.toff);
      v = TS(shear_ghost(B, a, sh, i < 0 ? 0 : 1, j, k, B.geom == GEOM_CART && pr.boost && m == 2 ? sh.u : 0.0));
    } else {
      if (xgh) i = i < 0 ? s.n0 - 1 : 0;
      v = a[stored_index(B, i, j, k)];
    }
    a[to] = v;
    return;
  }
  // FP64 copy of the shear-periodic x-ghost gas of velocity component m, with
  // the y and z ghost rows of the layer (periodic images): the interpolated
  // and boosted ghost values keep their FP64 rounding, so that a particle next
  // to the shear boundary sees the gas at the accuracy of the interior values.
  q -= bf * (uint32_t)pr.na;
  const int64_t layer = xghost_cells(B);
  const uint32_t bx = blocks256(layer);
  const int m = (int)(q / bx);
  const int64_t t = (int64_t)(q - (uint32_t)m * bx) * 256 + threadIdx.x;
  if (t >= layer) return;
  const int n1 = B.ax[1].n, n2 = B.ax[2].n, g1 = n1 + 2;
  const Shift sh = make_shift(B, pr.qOmega, *pr.tdev + pr.toff);
  const int jg = (int)(t % g1), kg = (int)(t / g1);
  const int j = ((jg - 1) % n1 + n1) % n1, k = ((kg - 1) % n2 + n2) % n2;
  const double dv = pr.boost && m == 1 ? sh.u : 0.0;
#pragma unroll
  for (int side = 0; side < 2; ++side)
    pr.xg[B.xg_base + (side * 3 + m) * layer + t] = shear_ghost(B, pr.gas.a[m + 1], sh, side, j, k, dv);
}

// Deposits of the ghost cells added to the active cells they are images of,
// written as a gather (each active cell next to a face reads the ghosts that
// feed it: those in z, then those in y with their own in z, then those in x
// with theirs, in this order of additions), so that one launch folds every
// axis; the ghosts are cleared by k_finish.  The energy channel of a
// shear-periodic box gains -/+ u D_y across x.  With FEED, v_c += D_c / (rho
// s_c) on every active cell with the folded deposits (read once).
// Targets: the cells next to a face, of the active cells of the folded axes
// and the stored cells of the others, in the first blocks of an entry; with
// FEED the other active cells follow, in blocks of their own (folding in the
// kernel's plain path took 81 us for a 128^3 FP32 shearing box; 35 so, as the
// feedback alone, with its FP64 division per cell).
struct FoldSet {
  int n[3], lo[3], T[3];   // active cells; first target; targets
  bool f[3];
  int64_t c[3];            // targets next to a z, y (of the rest), x face
};
__host__ __device__ __forceinline__ FoldSet fold_set(const Box& B) {
  FoldSet s;
  for (int d = 0; d < 3; ++d) {
    const bool ax = d < B.ndim;
    s.n[d] = ax ? B.ax[d].n : 1;
    s.f[d] = ax && (d == 0 ? B.ax[0].bc_lo != BC_OPEN : B.ax[d].bc_lo == BC_PERIODIC);
    s.lo[d] = ax && !s.f[d] ? -1 : 0;
  }
  // (an x ghost in a ghost row of an open y face keeps what z folds into it)
  if (s.f[2] && !s.f[1]) s.lo[0] = -1;
  for (int d = 0; d < 3; ++d) s.T[d] = s.n[d] - 2 * s.lo[d];
  const int64_t m0 = s.f[0] ? (s.n[0] > 1 ? 2 : 1) : 0, m1 = s.f[1] ? (s.n[1] > 1 ? 2 : 1) : 0,
                m2 = s.f[2] ? (s.n[2] > 1 ? 2 : 1) : 0;
  s.c[2] = m2 * s.T[0] * s.T[1];
  s.c[1] = m1 * s.T[0] * (s.T[2] - m2);
  s.c[0] = m0 * (s.T[1] - m1) * (s.T[2] - m2);
  return s;
}

template <typename TS> struct Fold {
  double qOmega, toff;
  const double* tdev;
  int boost_energy;
};

// v_c += D_c / (rho s_c) on an active cell, components [c0, c1).
template <typename TS>
__device__ __forceinline__ void feedback(const Box& B, const FView<TS>& fl, int c0, int c1, int i, int j, int64_t id,
                                         const double* D) {
  double sc[3] = {1.0, 1.0, 1.0};
  if (B.geom != GEOM_CART) {
    double x0 = cell_centre<double, false>(B.ax[0], i);
    sc[1] = x0;
    if (B.geom == GEOM_SPH) sc[2] = x0 * sin(cell_centre<double, false>(B.ax[1], j));
  }
  const double irho = 1.0 / double(fl.rho[id]);   // one division per cell
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    if (c < c0 || c >= c1) continue;
    const double q = D[c] * irho;
    fl.vel[c][id] = TS(double(fl.vel[c][id]) + (c == 0 ? q : q / sc[c]));
  }
}

template <typename TS, bool FOLD, bool FEED>
__global__ void __launch_bounds__(256) k_fold(const Box* boxes, BoxGrid bg, FView<TS> fl, Fold<TS> fo) {
  const int e = grid_entry(bg);
  const Box& B = boxes[bg.box[e]];
  int64_t t = grid_thread(bg, e);
  FoldSet s{};
  const int nc = B.geom == GEOM_CART ? B.ndim : 3;
  uint32_t be = 0, bc = 0;   // blocks of cells next to a face: in all, of a channel
  if constexpr (FOLD) {
    s = fold_set(B);
    bc = blocks256(s.c[0] + s.c[1] + s.c[2]);
    be = bc * (uint32_t)(nc + 1);
  }
  if (FEED && blockIdx.x - bg.blk0[e] >= be) {
    t -= (int64_t)be * 256;
    if (t >= B.ncell) return;
    int idx[3];
    unravel(B, t, idx);   // (active cell counts are below 2^31)
#pragma unroll
    for (int d = 0; d < 3; ++d)
      if (s.f[d] && (idx[d] == 0 || idx[d] == s.n[d] - 1)) return;
    const int64_t id = stored_index(B, idx[0], idx[1], idx[2]);
    double D[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) D[c] = c < nc ? double(fl.dep[c][id]) : 0.0;
    feedback(B, fl, 0, nc, idx[0], idx[1], id, D);
    return;
  }
  if constexpr (!FOLD) return;
  // a thread per cell and channel: its loads are behind branches, one after
  // the other (32^3 shearing box 9 us, 18 with the channels in turn)
  const int ch = (int)((blockIdx.x - bg.blk0[e]) / bc);
  t -= (int64_t)ch * bc * 256;
  int i, j, k;
  {
    const int m1 = s.f[1] ? (s.n[1] > 1 ? 2 : 1) : 0, m2 = s.f[2] ? (s.n[2] > 1 ? 2 : 1) : 0;
    // rows past the faces that are taken already
    const int r1 = s.T[1] - m1, j1 = s.f[1] ? 1 : s.lo[1], k1 = s.f[2] ? 1 : s.lo[2];
    if (t < s.c[2]) {
      const int64_t a = (int64_t)s.T[0] * s.T[1], side = t / a, v = t - side * a;
      k = side ? s.n[2] - 1 : 0;
      i = (int)(v % s.T[0]) + s.lo[0];
      j = (int)(v / s.T[0]) + s.lo[1];
    } else if ((t -= s.c[2]) < s.c[1]) {
      const int64_t a = (int64_t)s.T[0] * (s.T[2] - m2), side = t / a, v = t - side * a;
      j = side ? s.n[1] - 1 : 0;
      i = (int)(v % s.T[0]) + s.lo[0];
      k = (int)(v / s.T[0]) + k1;
    } else if ((t -= s.c[1]) < s.c[0]) {
      const int64_t a = (int64_t)r1 * (s.T[2] - m2), side = t / a, v = t - side * a;
      i = side ? s.n[0] - 1 : 0;
      j = (int)(v % r1) + j1;
      k = (int)(v / r1) + k1;
    } else {
      return;
    }
  }
  const int64_t id = stored_index(B, i, j, k);
  const bool in1 = j >= 0 && j < s.n[1], in2 = k >= 0 && k < s.n[2];
  if (s.f[0] && (i < 0 || i >= s.n[0]) && in1) return;   // (folded itself)
  const bool ex = s.f[0] && in1 && in2 && (i == 0 || i == s.n[0] - 1);
  const bool shear = B.ax[0].bc_lo == BC_SHEAR;
  Shift sh{0, 0.0, 0.0};
  if (ex && shear) sh = make_shift(B, fo.qOmega, *fo.tdev + fo.toff);
  // deposits of cell (ii, jj, kk), kk active, with its ghosts in z (all loads
  // of a face cell unconditional, to issue together: 29 us instead of 18 for
  // the 32^3 shearing box, most of them for nothing)
  auto dz = [&](const TS* a, int ii, int jj, int kk) -> TS {
    TS v = a[stored_index(B, ii, jj, kk)];
    if (s.f[2]) {
      if (kk == s.n[2] - 1) v += a[stored_index(B, ii, jj, -1)];
      if (kk == 0) v += a[stored_index(B, ii, jj, s.n[2])];
    }
    return v;
  };
  // and, jj active, with its ghosts in y
  auto dyz = [&](const TS* a, int ii, int jj, int kk) -> TS {
    TS v = dz(a, ii, jj, kk);
    if (s.f[1]) {
      if (jj == s.n[1] - 1) v += dz(a, ii, -1, kk);
      if (jj == 0) v += dz(a, ii, s.n[1], kk);
    }
    return v;
  };
  auto folded = [&](int ch) -> TS {
    const TS* a = fl.dep[ch];
    TS v = in1 && in2 ? dyz(a, i, j, k) : in2 ? dz(a, i, j, k) : a[id];
    if (!ex) return v;
    if (!shear) {
      if (i == s.n[0] - 1) v += dyz(a, -1, j, k);
      if (i == 0) v += dyz(a, s.n[0], j, k);
      return v;
    }
    const int n1 = s.n[1];
    const bool is_energy = fo.boost_energy && ch == nc;
    const TS* dy = fl.dep[B.ndim > 1 ? 1 : 0];
    auto row = [&](int side, int jr) {   // ghost row, energy frame-shifted
      jr = ((jr % n1) + n1) % n1;
      const int ig = side ? s.n[0] : -1;
      double g = double(dyz(a, ig, jr, k));
      if (is_energy) {
        const double du = sh.u * double(dyz(dy, ig, jr, k));
        g = side ? g + du : g - du;
      }
      return g;
    };
    if (i == 0) {
      // right ghost row j lands on floor(j + s) (1 - sf) and floor(j + s) + 1 (sf)
      double add0 = (1.0 - sh.sf) * row(1, j - sh.si);
      if (sh.sf > 0) add0 += sh.sf * row(1, j - sh.si - 1);
      v += TS(add0);
    }
    if (i == s.n[0] - 1) {
      // left ghost row j lands on floor(j - s) and floor(j - s) + 1
      double addn;
      if (sh.sf > 0) {
        const int c = sh.si + 1;  // ceil(s)
        addn = sh.sf * row(0, j + c) + (1.0 - sh.sf) * row(0, j + c - 1);
      } else {
        addn = row(0, j + sh.si);
      }
      v += TS(addn);
    }
    return v;
  };
  const TS v = folded(ch);
  fl.dep[ch][id] = v;   // (read by this thread only)
  if (FEED && ch < nc && i >= 0 && i < s.n[0] && in1 && in2) {
    const double D[3] = {double(v), double(v), double(v)};
    feedback(B, fl, ch, ch + 1, i, j, id, D);
  }
}

// Step start time.
__global__ void k_set_time(double* t, double v) { t[0] = v; }

void launch_set_time(double* tdev, double v, hipStream_t st) {
  hipLaunchKernelGGL(k_set_time, dim3(1), dim3(1), 0, st, tdev, v);
}

template <typename TS> __global__ void k_fill_value(TS* a, int64_t n, TS v) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) a[i] = v;
}

// FP64 sums of dV D over every stored cell of the boxes: a grid-stride loop
// over each box's blocks, a block reduction into the block's slot of
// `part`, then one workgroup adds the slots in a fixed order (no contended
// atomics, deterministic).  Before the boxes' blocks: the end of the step's
// fused launch (fe), whose one workgroup of partials then runs beside the
// others (128^3: 15 us of its own after a tile kernel of 8192 workgroups).
template <typename TS>
__global__ void __launch_bounds__(256) k_grid_sums(const Box* boxes, BoxGrid bg, FView<TS> fl,
                                                   double* __restrict__ part, FusedEnd<TS> fe) {
  if (blockIdx.x < bg.blk0[0]) {
    fused_end_block<TS, 256>(fe, blockIdx.x);
    return;
  }
  __shared__ double red[4][4];
  const int ge = grid_entry(bg);
  const Box& B = boxes[bg.box[ge]];
  const int nc = B.geom == GEOM_CART ? B.ndim : 3;
  const double inv_g0 = 1.0 / B.g0, inv_g1 = 1.0 / B.g1;
  double s[4] = {0, 0, 0, 0};
  const int64_t stride = (int64_t)(bg.blk0[ge + 1] - bg.blk0[ge]) * blockDim.x;
  for (int64_t t = grid_thread(bg, ge); t < B.nstore; t += stride) {
    int i, j, k;
    if (B.nstore < 0x7fffffffLL) {
      int r = div_small((int)t, B.g0, inv_g0);
      i = (int)t - r * B.g0;
      int q = div_small(r, B.g1, inv_g1);
      j = r - q * B.g1;
      k = q;
    } else {
      i = (int)(t % B.g0);
      j = (int)((t / B.g0) % B.g1);
      k = (int)(t / ((int64_t)B.g0 * B.g1));
    }
    double dv = 1.0 / inv_volume(B, i - 1, j - 1, k - B.k_off);
    int64_t id = B.store_base + t;
    for (int c = 0; c <= nc; ++c) s[c] += dv * double(fl.dep[c][id]);
  }
  for (int c = 0; c < 4; ++c) s[c] = wave_sum(s[c]);
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0)
    for (int c = 0; c < 4; ++c) red[wave][c] = s[c];
  __syncthreads();
  if (threadIdx.x < 4) {
    const int c = threadIdx.x;
    part[(size_t)(blockIdx.x - bg.blk0[0]) * 4 + c] = red[0][c] + red[1][c] + red[2][c] + red[3][c];
  }
}

// part[0 .. n) added to dg by one workgroup, in a fixed order.
__device__ void reduce_grid_partials(const double* __restrict__ part, int n, int nc, DiagDev* dg) {
  __shared__ double red[256][4];
  double acc[4] = {0, 0, 0, 0};
#pragma unroll 4
  for (int b = threadIdx.x; b < n; b += 256)
    for (int c = 0; c < 4; ++c) acc[c] += part[(size_t)b * 4 + c];
  for (int c = 0; c < 4; ++c) red[threadIdx.x][c] = acc[c];
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if (threadIdx.x < h)
      for (int c = 0; c < 4; ++c) red[threadIdx.x][c] += red[threadIdx.x + h][c];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    for (int c = 0; c < nc; ++c) dg->p_grid[c] += red[0][c];
    dg->e_grid += red[0][nc];
  }
}

__global__ void __launch_bounds__(256)
    k_reduce_grid_partials(const double* __restrict__ part, int n, int nc, DiagDev* dg) {
  reduce_grid_partials(part, n, nc, dg);
}

// After the fold, in one launch: the folded ghost deposits cleared and, in a
// workgroup past the boxes' (with end), what a step ends with: its grid sums
// added to the diagnostics, its time advanced, its step counted.
template <typename TS>
__global__ void __launch_bounds__(256) k_finish(const Box* boxes, BoxGrid bg, Arr4<TS> dep, int nch, StepEnd end) {
  if (blockIdx.x >= bg.blk0[bg.n]) {
    if (end.nparts > 0) reduce_grid_partials(end.part, end.nparts, nch - 1, end.dg);
    if (threadIdx.x == 0) {
      *end.tdev += end.dt;
      if (end.dg) end.dg->steps += 1;
    }
    return;
  }
  const int e = grid_entry(bg);
  const Box& B = boxes[bg.box[e]];
  const GhostSet s = ghost_set(B);
  const int64_t t = grid_thread(bg, e);
  if (t >= s.cx + s.cy + s.cz) return;
  int i, j, k;
  ghost_cell(s, t, i, j, k);
  const int64_t id = stored_index(B, i, j, k);
  for (int c = 0; c < nch; ++c) dep.a[c][id] = TS(0);
}

// ---------------------------------------------------------------- launchers

static inline unsigned blocks_for(int64_t n, int bs = 256) {
  return (unsigned)((n + bs - 1) / bs);
}

template <typename TS, typename A>
void launch_drift(const PView<TS>& p, const Box* boxes, int nbox, int geom, int ndim, int unif,
                  const Forces& f, double h, const double* tdev, double toff, int first,
                  DiagDev* dg, hipStream_t st) {
  if (p.n == 0) return;
  DUST_GEOM_SWITCH(geom, ndim, unif,
                   hipLaunchKernelGGL((k_drift<TS, A, G_, D_, U_>), dim3(blocks_for(p.n)), dim3(256), 0,
                                      st, p, boxes, nbox, f, A(h), tdev, toff, first, dg));
}

template <typename TS, typename A, typename TW>
void launch_gather(const PView<TS>& p, const Box* boxes, int nbox, int geom, int ndim, int unif,
                   const FView<TS>& fl, const double* xg, TW* rho_p, TW* const vg[3], DiagDev* dg,
                   hipStream_t st) {
  if (p.n == 0) return;
  DUST_GEOM_SWITCH(geom, ndim, unif,
                   hipLaunchKernelGGL((k_gather<TS, A, TW, G_, D_, U_>), dim3(blocks_for(p.n)), dim3(256),
                                      0, st, p, boxes, nbox, fl, xg, rho_p, vg[0], vg[1], vg[2], dg));
}

template <typename TS, typename A, typename TW>
void launch_kick(const PView<TS>& p, const Box* boxes, int nbox, int geom, int ndim, int unif,
                 const Forces& f, const Species* sp, int drag_mode, double dt, const TW* rho_p,
                 const TW* const vg[3], TW* const imp[4], DiagDev* dg, double* part, hipStream_t st) {
  if (p.n == 0) return;
  if (!dg) part = nullptr;
  const unsigned nb = std::min<unsigned>(blocks_for(p.n), KICK_BLOCKS);
  DUST_GEOM_SWITCH(geom, ndim, unif,
                   hipLaunchKernelGGL((k_kick<TS, A, TW, G_, D_, U_>), dim3(nb), dim3(256),
                                      0, st, p, boxes, nbox, f, sp, drag_mode, A(dt), rho_p, vg[0], vg[1],
                                      vg[2], imp[0], imp[1], imp[2], imp[3], dg, part));
  if (part)
    hipLaunchKernelGGL(k_reduce_kick_partials, dim3(1), dim3(256), 0, st, (const double*)part,
                       (int64_t)nb, dg);
}

int64_t kick_partial_words(int64_t n) {
  return 5 * (int64_t)std::min<unsigned>(blocks_for(std::max<int64_t>(n, 1)), KICK_BLOCKS);
}

template <typename TS, typename A, typename TW>
void launch_deposit(const PView<TS>& p, const Box* boxes, int nbox, int geom, int ndim, int unif,
                    const FView<TS>& fl, const TW* const imp[4], DiagDev* dg, hipStream_t st) {
  if (p.n == 0) return;
  DUST_GEOM_SWITCH(geom, ndim, unif,
                   hipLaunchKernelGGL((k_deposit<TS, A, TW, G_, D_, U_>), dim3(blocks_for(p.n)), dim3(256),
                                      0, st, p, boxes, nbox, fl, imp[0], imp[1], imp[2], imp[3], dg));
}

template <typename TS, typename A, typename TW>
void launch_deposit_pull(const PView<TS>& p, const Box& B, int geom, int ndim, int unif, const FView<TS>& fl,
                         int nch, double sgn, const TW* const imp[4], const uint32_t* perm,
                         const int64_t* bin_start, hipStream_t st) {
  if (B.nstore == 0) return;
  DUST_GEOM_SWITCH(geom, ndim, unif,
                   hipLaunchKernelGGL((k_deposit_pull<TS, A, TW, G_, D_, U_>), dim3(blocks_for(B.nstore)),
                                      dim3(256), 0, st, p, B, fl, nch, sgn, imp[0], imp[1], imp[2], imp[3],
                                      perm, bin_start));
}

template <typename TS, typename A>
void launch_source_coeffs(const PView<TS>& p, const Box* boxes, int nbox, int geom, int ndim, int unif,
                          const FView<TS>& fl, const Forces& f, const Species* sp, int drag_mode, double dt,
                          bool mass, A* const q[3], DiagDev* dg, hipStream_t st) {
  if (p.n == 0) return;
  if (mass)
    DUST_GEOM_SWITCH(geom, ndim, unif,
                     hipLaunchKernelGGL((k_source_coeffs<TS, A, G_, D_, U_, true>), dim3(blocks_for(p.n)),
                                        dim3(256), 0, st, p, boxes, nbox, fl, f, sp, drag_mode, A(1.0 / dt),
                                        q[0], q[1], q[2], dg));
  else
    DUST_GEOM_SWITCH(geom, ndim, unif,
                     hipLaunchKernelGGL((k_source_coeffs<TS, A, G_, D_, U_, false>), dim3(blocks_for(p.n)),
                                        dim3(256), 0, st, p, boxes, nbox, fl, f, sp, drag_mode, A(1.0 / dt),
                                        q[0], q[1], q[2], dg));
}

template <typename TS, typename A>
void launch_drag_source(const PView<TS>& p, const Box* boxes, int nbox, int geom, int ndim, int unif,
                        const FView<TS>& fl, const Forces& f, const Species* sp, int drag_mode,
                        double dt, DiagDev* dg, hipStream_t st) {
  if (p.n == 0) return;
  if (drag_mode == DRAG_EPSTEIN)
    DUST_GEOM_SWITCH(geom, ndim, unif,
                     hipLaunchKernelGGL((k_drag_source<TS, A, G_, D_, U_, true>),
                                        dim3(blocks_for(p.n, 256 * DS_PPT)), dim3(256), 0, st, p, boxes,
                                        nbox, fl, f, sp, drag_mode, A(1.0 / dt), dg));
  else
    DUST_GEOM_SWITCH(geom, ndim, unif,
                     hipLaunchKernelGGL((k_drag_source<TS, A, G_, D_, U_, false>),
                                        dim3(blocks_for(p.n, 256 * DS_PPT)), dim3(256), 0, st, p, boxes,
                                        nbox, fl, f, sp, drag_mode, A(1.0 / dt), dg));
}

template <typename TS, typename A>
void launch_mass_density(const PView<TS>& p, const Box* boxes, int nbox, int geom, int ndim, int unif,
                         TS* rho_d, const Species* sp, DiagDev* dg, hipStream_t st) {
  if (p.n == 0) return;
  FView<TS> fl{};
  fl.dep[0] = rho_d;
  DUST_GEOM_SWITCH(geom, ndim, unif,
                   hipLaunchKernelGGL((k_mass_density<TS, A, G_, D_, U_>), dim3(blocks_for(p.n, 256 * DS_PPT)),
                                      dim3(256), 0, st, p, boxes, nbox, fl, sp, dg));
}

// Launches `launch(grid, blocks)` over the boxes b with want(b), each with
// blocks(b) blocks, MB_BOXES boxes per launch.
template <typename Want, typename Blocks, typename Launch>
static void for_box_grids(const Box* hb, int nbox, Want want, Blocks blocks, Launch launch) {
  BoxGrid g{};
  uint32_t nb = 0;
  auto flush = [&]() {
    if (g.n) {
      g.blk0[g.n] = nb;
      launch(g, nb);
    }
    g = BoxGrid{};
    nb = 0;
  };
  for (int b = 0; b < nbox; ++b) {
    if (!want(hb[b])) continue;
    const uint32_t k = blocks(hb[b]);
    if (k == 0) continue;
    g.box[g.n] = b;
    g.blk0[g.n] = nb;
    nb += k;
    if (++g.n == MB_BOXES) flush();
  }
  flush();
}

static inline int box_nc(const Box& B) { return B.geom == GEOM_CART ? B.ndim : 3; }
static inline int64_t box_n(const Box& B, int d) { return d < B.ndim ? B.ax[d].n : 1; }

template <typename TS>
void launch_prepare(const Box* hb, int nbox, const Box* boxes_d, const Forces& f, const double* tdev, double toff,
                    const FView<TS>& fl, bool fill, double* xg, int nch, int64_t n_stored, hipStream_t st) {
  if (nbox <= 0) return;
  const int nc = box_nc(hb[0]);
  Prepare<TS> pr{};
  pr.gas = {{fl.rho, fl.vel[0], fl.vel[1], fl.vel[2]}};
  pr.na = fill ? nc + 1 : 0;
  pr.xg = xg;
  pr.qOmega = f.q * f.Omega;
  pr.toff = toff;
  pr.tdev = tdev;
  // the v_y ghosts across a shear face carry the boost -/+ q Omega L_x,
  // except for the residual velocities of orbital advection
  pr.boost = f.kind == FORCE_SHEARBOX;
  pr.dep = {{fl.dep[0], fl.dep[1], fl.dep[2], fl.dep[3]}};
  pr.n = n_stored;
  bool clear = nch > 0 && n_stored > 0;   // with the first launch
  auto run = [&](const BoxGrid& g, uint32_t nb) {
    pr.nch = clear ? nch : 0;
    if (clear) nb += (uint32_t)nch * blocks256((n_stored + CLEAR_PER - 1) / CLEAR_PER);
    clear = false;
    hipLaunchKernelGGL((k_prepare<TS>), dim3(nb), dim3(256), 0, st, boxes_d, g, pr);
  };
  if (fill)
    for_box_grids(hb, nbox, [](const Box&) { return true; },
                  [&](const Box& B) {
                    return (uint32_t)(nc + 1) * blocks256(fill_cells(B)) +
                           (xg ? (uint32_t)nc * blocks256(xghost_cells(B)) : 0u);
                  },
                  run);
  if (clear) run(BoxGrid{}, 0);
}

template <typename TS>
void launch_fold(const Box* hb, int nbox, const Box* boxes_d, const Forces& f, const double* tdev, double toff,
                 const FView<TS>& fl, bool feedback, hipStream_t st) {
  if (nbox <= 0) return;
  // the energy term of the boost: standard shearing box only
  const Fold<TS> fo{f.q * f.Omega, toff, tdev, f.kind == FORCE_SHEARBOX};
  for_box_grids(hb, nbox, [](const Box&) { return true; },
                [&](const Box& B) {
                  const FoldSet s = fold_set(B);
                  return (uint32_t)(box_nc(B) + 1) * blocks256(s.c[0] + s.c[1] + s.c[2]) +
                         (feedback ? blocks256(B.ncell) : 0u);
                },
                [&](const BoxGrid& g, uint32_t nb) {
                  if (feedback)
                    hipLaunchKernelGGL((k_fold<TS, true, true>), dim3(nb), dim3(256), 0, st, boxes_d, g, fl, fo);
                  else
                    hipLaunchKernelGGL((k_fold<TS, true, false>), dim3(nb), dim3(256), 0, st, boxes_d, g, fl, fo);
                });
}

template <typename TS>
void launch_finish(const Box* hb, int nbox, const Box* boxes_d, const FView<TS>& fl, const StepEnd* end,
                   hipStream_t st) {
  if (nbox <= 0) return;
  const int nch = box_nc(hb[0]) + 1;
  const Arr4<TS> deps{{fl.dep[0], fl.dep[1], fl.dep[2], fl.dep[3]}};
  bool pend = end != nullptr;   // with the first launch (nothing in the others reads what it writes)
  auto run = [&](const BoxGrid& g, uint32_t nb) {
    hipLaunchKernelGGL((k_finish<TS>), dim3(nb + (pend ? 1 : 0)), dim3(256), 0, st, boxes_d, g, deps, nch,
                       end ? *end : StepEnd{});
    pend = false;
  };
  for_box_grids(hb, nbox, [](const Box&) { return true; }, [](const Box& B) { return blocks256(fill_cells(B)); }, run);
  if (pend) run(BoxGrid{}, 0);
}

template <typename TS>
void launch_feedback(const Box* hb, int nbox, const Box* boxes_d, const FView<TS>& fl, hipStream_t st) {
  for_box_grids(hb, nbox, [](const Box&) { return true; }, [](const Box& B) { return blocks256(B.ncell); },
                [&](const BoxGrid& g, uint32_t nb) {
                  hipLaunchKernelGGL((k_fold<TS, false, true>), dim3(nb), dim3(256), 0, st, boxes_d, g, fl,
                                     Fold<TS>{});
                });
}

template <typename TS>
int launch_grid_sums(const Box* hb, int nbox, const Box* boxes_d, const FView<TS>& fl, DiagDev* dg, double* part,
                     const FusedEnd<TS>& fe, hipStream_t st) {
  if (nbox <= 0) return 0;
  const int nc = box_nc(hb[0]);
  int pend = 0;
  uint32_t end = (uint32_t)fe.blocks();   // with the first launch
  // blocks shared out in proportion to the stored cells of each launch's
  // boxes (at most GRID_SUM_BLOCKS + MB_BOXES in all)
  for (int b0 = 0; b0 < nbox; b0 += MB_BOXES) {
    const int b1 = std::min(nbox, b0 + MB_BOXES);
    int64_t tot = 0;
    for (int b = b0; b < b1; ++b) tot += hb[b].nstore;
    if (tot == 0) continue;
    for_box_grids(hb + b0, b1 - b0, [](const Box& B) { return B.nstore > 0; },
                  [&](const Box& B) {
                    const int64_t share = (int64_t)GRID_SUM_BLOCKS * B.nstore / tot;
                    return (uint32_t)std::max<int64_t>(1, std::min<int64_t>(blocks256(B.nstore), share));
                  },
                  [&](BoxGrid g, uint32_t nb) {
                    for (int e = 0; e < g.n; ++e) g.box[e] += b0;
                    for (int e = 0; e <= g.n; ++e) g.blk0[e] += end;
                    if (pend)   // (the slots are free again after this)
                      hipLaunchKernelGGL(k_reduce_grid_partials, dim3(1), dim3(256), 0, st, (const double*)part, pend,
                                         nc, dg);
                    hipLaunchKernelGGL((k_grid_sums<TS>), dim3(nb + end), dim3(256), 0, st, boxes_d, g, fl, part, fe);
                    end = 0;
                    pend = (int)nb;
                  });
  }
  return pend;
}

template <typename TS> void launch_fill_value(TS* a, int64_t n, TS v, hipStream_t st) {
  if (n <= 0) return;
  hipLaunchKernelGGL((k_fill_value<TS>), dim3(blocks_for(n)), dim3(256), 0, st, a, n, v);
}

#define DUST_INST(TS, A, TW)                                                                      \
  template void launch_gather<TS, A, TW>(const PView<TS>&, const Box*, int, int, int, int,             \
                                         const FView<TS>&, const double*, TW*, TW* const[3],       \
                                         DiagDev*,                                                \
                                         hipStream_t);                                            \
  template void launch_kick<TS, A, TW>(const PView<TS>&, const Box*, int, int, int, int, const Forces&, \
                                       const Species*, int, double, const TW*, const TW* const[3], \
                                       TW* const[4], DiagDev*, double*, hipStream_t);             \
  template void launch_deposit<TS, A, TW>(const PView<TS>&, const Box*, int, int, int, int,            \
                                          const FView<TS>&, const TW* const[4], DiagDev*,         \
                                          hipStream_t);                                           \
  template void launch_deposit_pull<TS, A, TW>(const PView<TS>&, const Box&, int, int, int, const FView<TS>&, \
                                               int, double, const TW* const[4], const uint32_t*,       \
                                               const int64_t*, hipStream_t);

#define DUST_INST_DRIFT(TS, A)                                                                    \
  template void launch_drift<TS, A>(const PView<TS>&, const Box*, int, int, int, int, const Forces&,   \
                                    double, const double*, double, int, DiagDev*, hipStream_t);         \
  template void launch_drag_source<TS, A>(const PView<TS>&, const Box*, int, int, int, int,        \
                                          const FView<TS>&, const Forces&, const Species*, int,     \
                                          double, DiagDev*, hipStream_t);                          \
  template void launch_mass_density<TS, A>(const PView<TS>&, const Box*, int, int, int, int, TS*,  \
                                           const Species*, DiagDev*, hipStream_t);                \
  template void launch_source_coeffs<TS, A>(const PView<TS>&, const Box*, int, int, int, int,      \
                                            const FView<TS>&, const Forces&, const Species*, int,  \
                                            double, bool, A* const[3], DiagDev*, hipStream_t);

DUST_INST_DRIFT(float, double)
DUST_INST_DRIFT(float, float)
DUST_INST_DRIFT(double, double)
DUST_INST(float, double, float)
DUST_INST(float, double, double)
DUST_INST(float, float, float)
DUST_INST(double, double, double)

#define DUST_INST_GRID(TS)                                                                        \
  template void launch_prepare<TS>(const Box*, int, const Box*, const Forces&, const double*, double, \
                                   const FView<TS>&, bool, double*, int, int64_t, hipStream_t);   \
  template void launch_fold<TS>(const Box*, int, const Box*, const Forces&, const double*, double,   \
                                const FView<TS>&, bool, hipStream_t);                             \
  template void launch_finish<TS>(const Box*, int, const Box*, const FView<TS>&, const StepEnd*,  \
                                  hipStream_t);                                                   \
  template void launch_feedback<TS>(const Box*, int, const Box*, const FView<TS>&, hipStream_t);     \
  template int launch_grid_sums<TS>(const Box*, int, const Box*, const FView<TS>&, DiagDev*, double*, \
                                    const FusedEnd<TS>&, hipStream_t);                            \
  template void launch_fill_value<TS>(TS*, int64_t, TS, hipStream_t);

DUST_INST_GRID(float)
DUST_INST_GRID(double)

}  // namespace dust
