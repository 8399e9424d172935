// The fused step right after a rebinning, for few particles per cell (gfx950):
// the same step as the tile kernel of dust_fused_kern.h, a particle per lane.
//
// The tile kernel gives a thread one cell and its particles one after the
// other.  At four particles per cell a wave's fullest cell has more than
// twice the mean (2.3 lane-slots per particle), and the 108 register sums of
// a thread's stencil leave 2 waves per SIMD, which wait 57 % of their cycles
// (the cylindrical disk of 2^25 particles: 7.5 ms, its VALU busy for 2.8).
// Right after a rebinning the particles are sorted by the cell they kick in,
// so here a workgroup walks its tile's particles in that order, 256 at a time,
// one per lane, and sums their deposits by runs of one cell (dust_runsum.h):
// every lane has a particle, and the registers are half.  Each particle is
// written to the slot that the tile kernel's layout gives it (slot_of): at
// few particles per cell the lanes of a wave still write whole stretches of
// each level, at many (a wave within one cell) they would write as many lines
// as lanes, and the tile kernel's lanes are busy anyway: it stays for those.
//
// Every particle is in the cell of its sort key at x^{n+1/2}, so the window
// is the tile and one cell around it; one that is not (a shear-periodic
// crossing, a rounding of the key's drift) is stored unstepped in its slot and
// left to the deferred-particle kernel, in place.
#pragma once

#include "dust_fused_kern.h"
#include "dust_runsum.h"

namespace dust {

template <typename TS, typename A, int GEOM, int NDIM, bool U, bool FG>
__global__ void __launch_bounds__(RUN_THREADS) __attribute__((amdgpu_waves_per_eu(2)))
    k_cells(const TileDesc* __restrict__ tiles, int split, int TX, int TY, int TZ, PView<TS> p, ShadowView<TS> sh,
            int clear_removed, const Box* __restrict__ boxes, FView<TS> fl, Forces f,
            const Species* __restrict__ sp, int drag_mode, A dt, const double* __restrict__ tdev,
            const int64_t* __restrict__ bin_start, const double* __restrict__ xg, DiagDev* dg,
            double* __restrict__ part, int sums, uint32_t* __restrict__ defer_list,
            uint32_t* __restrict__ defer_count, const uint32_t* __restrict__ perm,
            const uint32_t* __restrict__ slot_of) {
  constexpr int nc = GEOM == GEOM_CART ? NDIM : 3;
  constexpr int c2 = NDIM > 2 ? 1 : 0;
  const int RX = TX + 2, RY = TY + 2, RZ = c2 ? TZ + 2 : 1;
  const int WC = RX * RY * RZ;
  using G4 = typename Vec4<TS>::type;
  extern __shared__ double smem[];
  double* dep = smem;                                                   // (nc+1) * WC
  G4* gas = reinterpret_cast<G4*>(smem + ((WC * (nc + 1) + 3) & ~3));    // WC
  __shared__ __align__(16) A rec[RunSums<A, NDIM>::WORDS];
  // per-species drag propagator and mass (as the tile kernel)
  __shared__ A sp_c[DUST_MAX_SPECIES], sp_psi[DUST_MAX_SPECIES], sp_m[DUST_MAX_SPECIES];
  const int tid = threadIdx.x;
  const TileDesc td = tiles[blockIdx.x / (unsigned)split];
  const Box& B = boxes[td.box];
  const int ox = td.i0 - 1, oy = td.j0 - 1, oz = td.k0 - c2;   // window origin
  int64_t s0 = bin_start[td.key0], s1 = bin_start[td.key0 + (int64_t)td.ex * td.ey * td.ez];
  if (split > 1) tile_piece(s0, s1, split);
  double s_j[3] = {0, 0, 0}, s_e = 0, s_abs = 0;
  A a_cells = A(0);
  uint32_t flags_acc = 0;
  if (s0 < s1) {
    if (tid < sp->n) {
      A c, psi;
      propagator<A>(dt * A(sp->inv_tau[tid]), c, psi);
      sp_c[tid] = c;
      sp_psi[tid] = psi;
      sp_m[tid] = A(sp->mass[tid]);
    }
    run_sums_init<A, NDIM>(rec);
    const double t0 = *tdev;
    const A h = A(0.5) * dt;
    const int n0 = B.ax[0].n, n1 = B.ax[1].n, n2 = NDIM > 2 ? B.ax[2].n : 1;
    const bool per0 = axis_periodic(B.ax[0]), per1 = axis_periodic(B.ax[1]);
    const bool per2 = NDIM > 2 && axis_periodic(B.ax[2]);
    // the first particles are on their way while the window is staged; then
    // each chunk's are loaded one chunk ahead, their places two (past the
    // last: the last one again, not used)
    auto place = [&](int64_t e) { return e < s1 ? e : s1 - 1; };
    uint32_t far = perm[place(s0 + RUN_THREADS + tid)];
    uint32_t slot_n = slot_of[place(s0 + tid)];
    Raw<TS> nxt;
    load_raw<TS, NDIM, nc>(sh, perm[place(s0 + tid)], nxt);
    // stage the gas window (periodic images beyond the box), clear the deposit window
    for (int r = tid; r < WC; r += RUN_THREADS) {
      const int a = r % RX, bq = (r / RX) % RY, cq = r / (RX * RY);
      int i = ox + a, j = oy + bq, k = oz + cq;
      if (per0) i = wrap_index(i, n0);
      if (per1) j = wrap_index(j, n1);
      if (per2) k = wrap_index(k, n2);
      const bool in = i >= -1 && i <= n0 && j >= -1 && j <= n1 && (NDIM < 3 || (k >= -1 && k <= n2));
      const int64_t id = in ? stored_index(B, i, j, k) : 0;
      TS gv[3] = {TS(0), TS(0), TS(0)};
      TS lo = TS(0);
      if (in && xg && B.xg_base >= 0 && (i < 0 || i >= n0)) {
        // x ghost of a shear-periodic box: the FP64 ghost value, its y
        // component (which carries the shear boost) as a sum of two words
#pragma unroll
        for (int m = 0; m < nc; ++m) {
          const double v = gas_comp(B, fl, xg, m, i, j, k);
          gv[m] = TS(v);
          if (m == 1) lo = TS(v - double(gv[m]));
        }
      } else if (in) {
#pragma unroll
        for (int m = 0; m < nc; ++m) gv[m] = fl.vel[m][id];
      }
      gas[r] = Vec4<TS>::make(gv[0], gv[1], gv[2], lo);
#pragma unroll
      for (int m = 0; m <= nc; ++m) dep[m * WC + r] = 0.0;
    }
    __syncthreads();
    for (int64_t cb = s0; cb < s1; cb += RUN_THREADS) {
      const bool has = cb + tid < s1;
      const Raw<TS> cur = nxt;
      const uint32_t i = slot_n;
      slot_n = slot_of[place(cb + RUN_THREADS + tid)];
      load_raw<TS, NDIM, nc>(sh, far, nxt);
      far = perm[place(cb + 2 * RUN_THREADS + tid)];
      const int32_t cid = cur.cell;
      bool live = has && cid >= B.cell_base && cid < B.cell_base + B.ncell;
      bool removed = false, deferred = false;
      flags_acc |= has && cid >= 0 && !live ? (uint32_t)DUST_FLAG_BAD_CELL : 0u;
      int idx[3] = {td.i0, td.j0, td.k0};
      A off[3], mom[3];
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        off[d] = A(cur.off[d]);
        mom[d] = A(cur.mom[d]);
      }
      if (live) {
        unravel(B, cid - B.cell_base, idx);
        bool bad = false;
#pragma unroll
        for (int d = 0; d < 3; ++d) bad |= !(off[d] >= A(-0.5) && off[d] < A(0.5));
        flags_acc |= bad ? (uint32_t)DUST_FLAG_OFFSET_RANGE : 0u;
        // half drift to x^{n+1/2}
        if (!drift<A, GEOM, NDIM, U, FG>(B, f, true, h, t0 + double(h), idx, off, mom)) {
          store_particle<TS, A, GEOM, NDIM, FG>(p, B, f, t0 + double(h), i, false, idx, off, mom, dg);
          live = false;
          removed = true;
        }
      }
      const int la = win_coord(idx[0], ox, n0, RX, per0), lb = win_coord(idx[1], oy, n1, RY, per1);
      const int lc = c2 ? win_coord(idx[2], oz, n2, RZ, per2) : 0;
      deferred = live & !((la >= 1) & (la <= RX - 2) & (lb >= 1) & (lb <= RY - 2) &
                          ((c2 == 0) | ((lc >= 1) & (lc <= RZ - 2))));
      {
        const uint64_t dm = __ballot(deferred);
        if (dm) {
          const int leader = __ffsll((unsigned long long)dm) - 1;
          uint32_t base = 0;
          if ((tid & 63) == leader) base = atomicAdd(defer_count, (uint32_t)__popcll(dm));
          base = __shfl(base, leader, 64);
          if (deferred) defer_list[base + lanes_below(dm)] = i;
        }
      }
      live = live && !deferred;
      const int r0 = live ? la + RX * (lb + RY * lc) : -1;
      A q[4] = {A(0), A(0), A(0), A(0)};
      Stencil<A> s;
#pragma unroll
      for (int d = 0; d < 3; ++d)
#pragma unroll
        for (int a = 0; a < 3; ++a) s.w[d][a] = A(0);
      if (live) {
        // weights at x^{n+1/2}; gather (Eq. Delta_vp) in slip form (see the
        // tile kernel)
        stencil_weights<A, GEOM, NDIM, U>(B, idx, off, s);
        constexpr bool AZ = az_gather<A, GEOM>();
        constexpr int PHI = az_comp<GEOM>();
        double wr[3] = {0.0, 0.0, 0.0};
        if constexpr (AZ) radial_weights64<A, GEOM, U>(B, idx[0], off[0], s, wr);
        Where<A> wh;
        where<A, GEOM, NDIM, U>(B, idx, off, wh);
        SlipScale<A> ss;
        slip_scale<A, GEOM, NDIM, U>(B, idx, off, mom, wh, ss);
        const A* up = ss.up;
        A v[3] = {A(0), A(0), A(0)};
        double vaz = 0.0;   // azimuthal component in FP64 (AZ)
        // (one plane of the stencil per iteration: straight-line code would
        // issue every read first, and hold its registers)
#pragma unroll 1
        for (int c = -c2; c <= c2; ++c) {
          const A wz = NDIM < 3 ? s.w[2][1] : c < 0 ? s.w[2][0] : c == 0 ? s.w[2][1] : s.w[2][2];
#pragma unroll
          for (int bb = -1; bb <= 1; ++bb) {
            const int rr = r0 + RX * (bb + RY * c);
            A u[3] = {A(0), A(0), A(0)};
            double uaz = 0.0;
#pragma unroll
            for (int a = -1; a <= 1; ++a) {
              const G4 g = gas[rr + a];
              const TS gv[3] = {g.x, g.y, g.z};
#pragma unroll
              for (int m = 0; m < nc; ++m) u[m] += s.w[0][a + 1] * (A(gv[m]) - up[m]);
              if (nc > 1) u[1] += s.w[0][a + 1] * A(g.w);   // low word (shear x ghosts only)
              if constexpr (AZ) uaz += wr[a + 1] * (double(gv[PHI]) - double(up[PHI]));
            }
            const A wbc = s.w[1][bb + 1] * wz;
#pragma unroll
            for (int m = 0; m < nc; ++m) v[m] += wbc * u[m];
            if constexpr (AZ) vaz += (double(s.w[1][bb + 1]) * double(wz)) * uaz;
          }
        }
        if constexpr (AZ) v[PHI] = A(vaz);   // (the FP32 sum of that component is dropped)
        // kick
        A sl[3];
#pragma unroll
        for (int m = 0; m < 3; ++m) sl[m] = m < nc ? slip_canonical<A, GEOM>(ss, m, v[m]) : A(0);
        int spc = cur.species;
        flags_acc |= spc >= sp->n ? (uint32_t)DUST_FLAG_BAD_CELL : 0u;
        spc = spc >= sp->n ? 0 : spc;
        const A m = p.mass ? A(cur.mass) : sp_m[spc];
        A c, psi;
        if (drag_mode == DRAG_SPECIES) {
          c = sp_c[spc];
          psi = sp_psi[spc];
        } else {
          const A it = inverse_tau<A, GEOM>(f, drag_mode, A(cur.drag), A(0), wh);
          propagator<A>(dt * it, c, psi);
        }
        KickOut<A> o;
        kick<A, GEOM, NDIM, FG>(B, f, dt, c, psi, wh, mom, sl, o);
#pragma unroll
        for (int k = 0; k < nc; ++k) {
          q[k] = -m * o.j[k];   // deposits carry the minus sign of Eq. dust_feedback_final
          if (sums) {
            A cps;
            if constexpr (GEOM == GEOM_CART && U) {
              cps = fabs((mom[k] + A(0.5) * o.dp[k]) * dt * A(B.ax[k].inv_d));
            } else {
              const A vbar = (mom[k] + A(0.5) * o.dp[k]) / wh.sc[k];
              const A dl = cell_width<A, U>(B.ax[k], idx[k]) * (GEOM == GEOM_CART || k == 0 ? A(1) : wh.sc[k]);
              cps = fabs(vbar * dt / dl);
            }
            a_cells = cps > a_cells ? cps : a_cells;
          }
          mom[k] += o.dp[k];
        }
        q[nc] = -m * o.e;
        if (sums) {
#pragma unroll
          for (int k = 0; k < nc; ++k) {
            s_j[k] -= double(q[k]);
            s_abs += fabs(double(q[k]));
          }
          s_e -= double(q[nc]);
        }
      }
      run_sums<A, NDIM, nc + 1>(dep, RX, RY, WC, rec, r0, live, q, s);
      // second half drift to x^{n+1}
      if (live) {
        const bool alive = drift<A, GEOM, NDIM, U, FG>(B, f, false, h, t0 + double(dt), idx, off, mom);
        store_particle<TS, A, GEOM, NDIM, FG>(p, B, f, t0 + double(dt), i, alive, idx, off, mom, dg);
        if (!alive && clear_removed) {
#pragma unroll
          for (int d = 0; d < 3; ++d) {
            if (d < NDIM) p.off[d][i] = TS(0);
            if (d < nc) p.mom[d][i] = TS(0);
          }
        }
      }
      if (has) {
        if (!live) {
          // removed or cell-less particles keep their last offsets and momenta;
          // a deferred one is stored as it came
          if (!removed) p.cell[i] = cid;
#pragma unroll
          for (int d = 0; d < 3; ++d) {
            if (d < NDIM) p.off[d][i] = cur.off[d];
            if (d < nc) p.mom[d][i] = cur.mom[d];
          }
        }
        if (p.drag) p.drag[i] = cur.drag;
        if (p.mass) p.mass[i] = cur.mass;
        if (p.species) p.species[i] = (uint8_t)cur.species;
        if (p.id) p.id[i] = cur.id;
      }
    }
    __syncthreads();
    // add the deposit window to the grid (periodic images to their cells)
    for (int r = tid; r < WC; r += RUN_THREADS) {
      const int a = r % RX, bq = (r / RX) % RY, cq = r / (RX * RY);
      int i = ox + a, j = oy + bq, k = oz + cq;
      if (per0) i = wrap_index(i, n0);
      if (per1) j = wrap_index(j, n1);
      if (per2) k = wrap_index(k, n2);
      const bool in = i >= -1 && i <= n0 && j >= -1 && j <= n1 && (NDIM < 3 || (k >= -1 && k <= n2));
      if (!in) continue;
      const int64_t id = stored_index(B, i, j, k);
      const double iv = inv_volume(B, i, j, k);
#pragma unroll
      for (int m = 0; m <= nc; ++m) {
        const double x = dep[m * WC + r];
        if (x != 0.0) unsafeAtomicAdd(&fl.dep[m][id], TS(x * iv));
      }
    }
  }
  if (dg && flags_acc) atomicOr(&dg->flags, (unsigned)flags_acc);
  // diagnostics: the workgroup's FP64 sums to its own slot of `part`
  if (dg) {
    // (in the records' place: three workgroups of the 4x16x4 tiles just fit)
    double (*red)[PART_WORDS] = reinterpret_cast<double (*)[PART_WORDS]>(rec);
    __syncthreads();
    double s[PART_WORDS] = {s_j[0], s_j[1], s_j[2], s_e, s_abs, double(a_cells), 0.0, 0.0};
    if (sums) {
#pragma unroll
      for (int k = 0; k < 5; ++k) s[k] = wave_sum(s[k]);
      s[5] = wave_max(s[5]);
    }
    if ((tid & 63) == 0) {
#pragma unroll
      for (int k = 0; k < PART_WORDS; ++k) red[tid >> 6][k] = s[k];
    }
    __syncthreads();
    if (tid < PART_WORDS) {
      double v = red[0][tid];
      for (int w = 1; w < RUN_THREADS / 64; ++w) v = tid == 5 ? fmax(v, red[w][tid]) : v + red[w][tid];
      part[(size_t)blockIdx.x * PART_WORDS + tid] = sums || tid >= 6 ? v : 0.0;
    }
  }
}

// LDS of the windows of a workgroup.
template <typename TS, int GEOM, int NDIM> size_t cells_lds_bytes(const TileShape& t) {
  constexpr int nc = GEOM == GEOM_CART ? NDIM : 3;
  const size_t wc = (size_t)(t.t[0] + 2) * (t.t[1] + 2) * (NDIM > 2 ? t.t[2] + 2 : 1);
  return ((wc * (nc + 1) + 3) & ~(size_t)3) * sizeof(double) + wc * 4 * sizeof(TS);
}

template <typename TS, typename A, int GEOM, int NDIM, bool U>
void launch_cells_g(const FusedPlan& plan, const PView<TS>& p, const FusedMove<TS>& mv, const Box* boxes_d,
                    const FView<TS>& fl, const Forces& f, const Species* sp, int drag_mode, double dt,
                    const double* tdev, const int64_t* bin_start, const double* xg, DiagDev* dg, bool sums,
                    hipStream_t st) {
  const size_t lds = cells_lds_bytes<TS, GEOM, NDIM>(plan.tile);
  auto run = [&](auto kern) {
    const int split = cells_split(plan.ntiles, p.n, sizeof(A) == 8);
    hipLaunchKernelGGL(kern, dim3(plan.ntiles * split), dim3(RUN_THREADS), lds, st, plan.tiles_d, split, plan.tile.t[0],
                       plan.tile.t[1], NDIM > 2 ? plan.tile.t[2] : 1, p, mv.sh, mv.clear_removed, boxes_d, fl, f, sp,
                       drag_mode, A(dt), tdev, bin_start, xg, dg, plan.part_d, (int)sums, plan.defer_list,
                       plan.defer_count, mv.perm, mv.slot_of);
  };
  if constexpr (GEOM == GEOM_CART && NDIM == 3) {
    if (f.kind == FORCE_FARGO) {
      run(k_cells<TS, A, GEOM, NDIM, U, true>);
      return;
    }
  }
  run(k_cells<TS, A, GEOM, NDIM, U, false>);
}

#define DUST_CELLS_DECL(PREFIX, TS, A, G, D, UU)                                                              \
  PREFIX template void launch_cells_g<TS, A, G, D, UU>(                                                      \
      const FusedPlan&, const PView<TS>&, const FusedMove<TS>&, const Box*, const FView<TS>&, const Forces&, \
      const Species*, int, double, const double*, const int64_t*, const double*, DiagDev*, bool, hipStream_t);
#define DUST_CELLS_ALL(PREFIX, TS, A)                  \
  DUST_CELLS_DECL(PREFIX, TS, A, GEOM_CART, 2, true)   \
  DUST_CELLS_DECL(PREFIX, TS, A, GEOM_CART, 2, false)  \
  DUST_CELLS_DECL(PREFIX, TS, A, GEOM_CART, 3, true)   \
  DUST_CELLS_DECL(PREFIX, TS, A, GEOM_CART, 3, false)  \
  DUST_CELLS_DECL(PREFIX, TS, A, GEOM_CYL, 3, false)   \
  DUST_CELLS_DECL(PREFIX, TS, A, GEOM_SPH, 3, false)

}  // namespace dust
