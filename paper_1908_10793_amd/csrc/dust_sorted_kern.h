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
//    and walks them tile by tile with an FP64 LDS window over the tile and
//    one cell around it;
//  * one lane per particle loads it, forms its weights and its channels'
//    values and puts them in LDS; then half a wave (a quarter in 2-D) takes
//    the particles one after the other, one lane per cell of the stencil,
//    and sums in registers until the host cell changes.  A lane holds one
//    cell's channels (4 registers where a thread per host cell needs 108),
//    so FP64 sums cost no occupancy, and lanes never wait for the fullest
//    cell of a wave;
//  * a run of one host cell is then added to the window (27 lanes, 27
//    words: no two lanes on one word), and the window to HBM once per tile.
#pragma once

#include "dust_device.h"
#include "dust_launch.h"
#include "dust_particle.h"
#include "dust_sorted.h"

namespace dust {

static constexpr int SORTED_THREADS = 256;   // also the particles of a chunk

template <typename A> struct GasCell { A v[4]; };   // three velocity components, density

// Compile-time layout of a kernel.
template <typename A, int GEOM, int NDIM, int MODE> struct SortedShape {
  static constexpr int NC = GEOM == GEOM_CART ? NDIM : 3;
  static constexpr int NCH = MODE == SORTED_MASS ? 1 : MODE == SORTED_SOURCE ? NC : NC + 1;
  static constexpr bool GAS = MODE == SORTED_SOURCE || MODE == SORTED_STEP;
  // the tile (FP64 with a gas window: half as long in x, so that three
  // workgroups fit a CU's LDS)
  static constexpr int T0 = sorted_tile_extent(sizeof(A) == 8, NDIM, 0);
  static constexpr int T1 = sorted_tile_extent(sizeof(A) == 8, NDIM, 1);
  static constexpr int T2 = sorted_tile_extent(sizeof(A) == 8, NDIM, 2);
  static constexpr int RX = T0 + 2, RY = T1 + 2, RZ = NDIM > 2 ? T2 + 2 : 1;
  static constexpr int WC = RX * RY * RZ;
  static constexpr int NT = NDIM > 2 ? 27 : 9;    // cells of a stencil
  static constexpr int G = NDIM > 2 ? 32 : 16;    // lanes (and particles of a chunk) of a group
  // one particle's words: FP32 q[4], w0[3], w1 w2 products[9] at 20 words
  // (consecutive lanes' 16-byte writes on distinct banks); FP64 q[4], w0[3],
  // w1[3], w2[3] at 14 (the same, with less LDS)
  static constexpr int RS = sizeof(A) == 4 ? 20 : 14;
  // the groups of a wave read at the same time: shifted by half (a quarter)
  // of the 64 banks
  static constexpr int GP = (NDIM > 2 ? 32 : 16) / (int)(sizeof(A) / 4);
  static constexpr int GS = G * RS + GP;
};

template <typename TS, typename A, typename TW, int GEOM, int NDIM, bool U, int MODE>
__global__ void __launch_bounds__(SORTED_THREADS)
    k_sorted(PView<TS> p, const Box* __restrict__ boxes, int nbox, FView<TS> fl, SortedIn<TW> in,
             const double* __restrict__ xg, Forces f, const Species* __restrict__ sp, int drag_mode, A dt,
             const uint32_t* __restrict__ key, const uint32_t* __restrict__ perm, uint32_t nbins, int ppb,
             DiagDev* dg, int sums) {
  using S = SortedShape<A, GEOM, NDIM, MODE>;
  constexpr int NC = S::NC, NCH = S::NCH, NT = S::NT, G = S::G, RX = S::RX, RY = S::RY, WC = S::WC;
  constexpr int c2 = NDIM > 2 ? 1 : 0;
  constexpr bool F32 = sizeof(A) == 4;
  __shared__ double win[NCH * WC];
  __shared__ __align__(16) A rec[(SORTED_THREADS / G) * S::GS];
  __shared__ int s_r[SORTED_THREADS];
  __shared__ GasCell<A> gas[S::GAS ? WC : 1];
  const int tid = threadIdx.x;
  const int64_t s0 = (int64_t)blockIdx.x * ppb;
  const int64_t s1 = s0 + ppb < p.n ? s0 + ppb : p.n;
  uint32_t flags = 0;
  double sum[5] = {0, 0, 0, 0, 0}, cells = 0.0;   // SORTED_STEP: the kick's diagnostics
  // this lane's cell of the stencil, relative to the host cell
  const int grp = tid / G, s = tid % G, sc_ = s < NT ? s : 0;
  const int sa = sc_ % 3, sb = (sc_ / 3) % 3, scc = NDIM > 2 ? sc_ / 9 : 0;
  const int soff = (sa - 1) + RX * ((sb - 1) + RY * (scc - c2));

  int64_t cur = s0;
  while (cur < s1) {
    const uint32_t k0 = key[cur];
    if (k0 >= nbins) {
      // sorted last: particles without a cell, and cell ids out of range
      for (int64_t e = cur + tid; e < s1; e += SORTED_THREADS)
        if (p.cell[perm[e]] >= 0) flags |= DUST_FLAG_BAD_CELL;
      break;
    }
    // the tile of this key (its cells are consecutive keys)
    const int ub = __builtin_amdgcn_readfirstlane(nbox == 1 ? 0 : find_box(boxes, nbox, k0));
    const Box& B = boxes[ub];
    const int n0 = B.ax[0].n, n1 = B.ax[1].n, n2 = NDIM > 2 ? B.ax[2].n : 1;
    int ti, tj, tk, e0, e1, e2;
    uint32_t kend;
    {
      uint32_t r = k0 - (uint32_t)B.cell_base;
      const uint32_t layer = (uint32_t)n0 * (uint32_t)n1 * (uint32_t)min(S::T2, n2);   // (at most the box)
      tk = NDIM > 2 ? (int)(r / layer) : 0;
      r -= (uint32_t)tk * layer;
      e2 = min(S::T2, n2 - tk * S::T2);
      const uint32_t row = (uint32_t)n0 * (uint32_t)min(S::T1, n1) * (uint32_t)e2;
      tj = (int)(r / row);
      r -= (uint32_t)tj * row;
      e1 = min(S::T1, n1 - tj * S::T1);
      const uint32_t col = (uint32_t)S::T0 * (uint32_t)(e1 * e2);
      ti = (int)(r / col);
      r -= (uint32_t)ti * col;
      e0 = min(S::T0, n0 - ti * S::T0);
      kend = k0 - r + (uint32_t)(e0 * e1 * e2);
    }
    const int o0 = ti * S::T0 - 1, o1 = tj * S::T1 - 1, o2 = tk * S::T2 - c2;   // window origin
    for (int r = tid; r < WC; r += SORTED_THREADS) {
#pragma unroll
      for (int m = 0; m < NCH; ++m) win[m * WC + r] = 0.0;
      if constexpr (S::GAS) {
        const int a = r % RX, b = (r / RX) % RY, c = r / (RX * RY);
        GasCell<A> g{};
        if (a < e0 + 2 && b < e1 + 2 && (NDIM < 3 || c < e2 + 2)) {
#pragma unroll
          for (int m = 0; m < NC; ++m) g.v[m] = A(gas_comp(B, fl, xg, m, o0 + a, o1 + b, o2 + c));
          if (drag_mode == DRAG_EPSTEIN) g.v[3] = A(fl.rho[stored_index(B, o0 + a, o1 + b, o2 + c)]);
        }
        gas[r] = g;
      }
    }
    // chunks of 256 slots while they stay in the tile
    for (;;) {
      const int64_t e = cur + tid;
      const bool has = e < s1 && key[e < s1 ? e : s1 - 1] < kend;
      const int cnt = __syncthreads_count(has);   // (sorted: the first cnt threads)
      if (cnt == 0) break;
      int r0 = -1;
      if (has) {
        const int64_t i = perm[e];
        const int64_t c = p.cell[i];
        int idx[3];
        A off[3], mom[3] = {A(0), A(0), A(0)};
        unravel(B, c - B.cell_base, idx);
        bool bad = false, nonfinite = false;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          off[d] = d < NDIM ? A(p.off[d][i]) : A(0);
          bad |= !(off[d] >= A(-0.5) && off[d] < A(0.5));
          if (MODE != SORTED_MASS && d < NC && (S::GAS || p.mom[d])) mom[d] = A(p.mom[d][i]);
          nonfinite |= !isfinite(double(mom[d]));
        }
        flags |= bad ? (uint32_t)DUST_FLAG_OFFSET_RANGE : 0u;
        flags |= nonfinite ? (uint32_t)DUST_FLAG_NONFINITE : 0u;
        r0 = (idx[0] - o0) + RX * ((idx[1] - o1) + RY * (idx[2] - o2));
        Stencil<A> st;
        stencil_weights<A, GEOM, NDIM, U>(B, idx, off, st);
        A q[4] = {A(0), A(0), A(0), A(0)};
        if constexpr (MODE == SORTED_DEPOSIT) {
#pragma unroll
          for (int m = 0; m < NCH; ++m) q[m] = -A(in.q[m][i]);
        } else {
          int spc = p.species ? p.species[i] : 0;
          if (spc >= sp->n) {
            flags |= DUST_FLAG_BAD_CELL;
            spc = 0;
          }
          const A m = p.mass ? A(p.mass[i]) : A(sp->mass[spc]);
          if constexpr (MODE == SORTED_MASS) {
            q[0] = m;
          } else {
            const A dval = drag_mode == DRAG_SPECIES ? A(1) : A(p.drag[i]);
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
                  const GasCell<A> g = gas[r0 + a + RX * (bb + RY * cc)];
                  if (drag_mode == DRAG_EPSTEIN) rg += wt * g.v[3];
#pragma unroll
                  for (int d = 0; d < NC; ++d) {
                    if constexpr (MODE == SORTED_SOURCE) v[d] += wt * (g.v[d] * w.sc[d] - mom[d]);
                    else v[d] += wt * g.v[d];
                  }
                }
              }
            }
            const A it = drag_mode == DRAG_EPSTEIN
                             ? rg / dval
                             : inverse_tau<A, GEOM>(f, drag_mode, dval, A(sp->inv_tau[spc]), w);
            if constexpr (MODE == SORTED_SOURCE) {
              const A k = m * (it < dt ? it : dt);   // dt: the reciprocal of the step here
#pragma unroll
              for (int d = 0; d < NC; ++d) q[d] = -(k * v[d]);
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
                p.mom[d][i] = TS(mom[d]);
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
        A* rw = rec + grp * S::GS + s * S::RS;
#pragma unroll
        for (int m = 0; m < 4; ++m) rw[m] = q[m];
#pragma unroll
        for (int a = 0; a < 3; ++a) rw[4 + a] = st.w[0][a];
        if constexpr (F32) {
#pragma unroll
          for (int a = 0; a < 9; ++a) rw[7 + a] = st.w[1][a % 3] * st.w[2][NDIM > 2 ? a / 3 : 1];
        } else {
#pragma unroll
          for (int a = 0; a < 3; ++a) {
            rw[7 + a] = st.w[1][a];
            rw[10 + a] = st.w[2][a];
          }
        }
      }
      s_r[tid] = r0;
      __syncthreads();
      // a group's particles one after the other, a lane per stencil cell
      {
        const A* rr = rec + grp * S::GS;
        const int* rc = s_r + grp * G;
        const int nw = min(G, cnt - (tid / 64) * 64);   // the wave's first group has the most
        A acc[NCH];
#pragma unroll
        for (int m = 0; m < NCH; ++m) acc[m] = A(0);
        int host = -1;
        auto flush = [&]() {
          if (host >= 0 && s < NT) {
#pragma unroll
            for (int m = 0; m < NCH; ++m) atomicAdd(&win[m * WC + host + soff], double(acc[m]));
          }
        };
        for (int j = 0; j < nw; ++j) {
          const int r = rc[j];
          if (r < 0) continue;
          if (r != host) {
            flush();
            host = r;
#pragma unroll
            for (int m = 0; m < NCH; ++m) acc[m] = A(0);
          }
          const A* w = rr + j * S::RS;
          A wt;
          if constexpr (F32) wt = w[4 + sa] * w[7 + sb + 3 * scc];
          else wt = w[4 + sa] * (w[7 + sb] * w[10 + (NDIM > 2 ? scc : 1)]);
#pragma unroll
          for (int m = 0; m < NCH; ++m) acc[m] += wt * w[m];
        }
        flush();
      }
      cur += cnt;
      if (cnt < SORTED_THREADS) break;   // (uniform) the tile's or the block's last slots
    }
    __syncthreads();
    // the window to the grid
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
    __syncthreads();
  }
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

template <typename TS, typename A, typename TW, int MODE>
void launch_sorted(const PView<TS>& p, const Box* boxes, int nbox, int geom, int ndim, int unif,
                   const FView<TS>& fl, const SortedIn<TW>& in, const double* xg, const Forces& f,
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
      const PView<TS>&, const Box*, int, int, int, int, const FView<TS>&, const SortedIn<TW>&, const double*, \
      const Forces&, const Species*, int, double, const uint32_t*, const uint32_t*, int64_t, DiagDev*, bool, \
      hipStream_t);

}  // namespace dust
