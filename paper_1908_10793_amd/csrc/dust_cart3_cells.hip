// The fused step right after a rebinning, for few particles per cell, on the
// FP32 uniform-Cartesian path (gfx950): a particle per lane, as
// dust_cells_kern.h does for the other geometries, with this path's
// arithmetic (dust_cart3_kern.h, same expressions) and layout.
//
// The workgroup walks its tile's particles cell by cell in the order in which
// the layout hands the cells to lanes (order_src, order_slot of
// k_c3_level_perm), so that the lanes of a wave write stretches of a level.
// 128^3 shearing box, 8 particles per cell: 734 us, its VALU busy for 460 (1070
// instructions per 64 particles) and its LDS for 480 (the gather's reads 330,
// the sums by runs most of the rest); with the tile kernel of dust_cart3_kern.h
// the whole step takes 1529 us instead of 1472.
#include "dust_cart3_kern.h"
#include "dust_runsum.h"

namespace dust {

template <bool SB, int BOXES>
__global__ void __launch_bounds__(RUN_THREADS)
    k_c3_cells(const TileDesc* __restrict__ tiles, int split, int TX, int TY, int TZ, PView<float> p, ShadowView<float> sh,
               const Box* __restrict__ boxes, FView<float> fl, Forces f, const Species* __restrict__ sp, float dt,
               const double* __restrict__ tdev, const int64_t* __restrict__ bin_start,
               const double* __restrict__ xg, DiagDev* dg, double* __restrict__ part, int sums,
               uint32_t* __restrict__ defer_list, uint32_t* __restrict__ defer_count,
               const uint32_t* __restrict__ order_src, const uint32_t* __restrict__ order_slot) {
  const int RX = TX + 2, RY = TY + 2, RZ = TZ + 2;
  const int WC = RX * RY * RZ;
  extern __shared__ double smem[];
  double* dep = smem;                                        // 4 * WC
  float4* gas = reinterpret_cast<float4*>(smem + 4 * WC);    // WC
  float2* xres = reinterpret_cast<float2*>(gas + WC);        // SB: q Omega x_c of the window's columns, hi + lo
  __shared__ __align__(16) float rec[RunSums<float, 3>::WORDS];
  // per species: mass, c, h1, dt psi (as the tile kernel); SB: W, 1 / (1 + W^2)
  __shared__ float4 sp_k[DUST_MAX_SPECIES];
  __shared__ float2 sp_w[DUST_MAX_SPECIES];
  const int tid = threadIdx.x;
  const TileDesc td = tiles[blockIdx.x / (unsigned)split];
  const Box& B = boxes[td.box];
  const C3Box cb = c3_box(B, dt);
  const int ox = td.i0 - 1, oy = td.j0 - 1, oz = td.k0 - 1;
  uint32_t s0 = (uint32_t)bin_start[td.key0], s1 = (uint32_t)bin_start[td.key0 + (int64_t)td.ex * td.ey * td.ez];
  if (split > 1) tile_piece(s0, s1, split);
  float s_j0 = 0.0f, s_j1 = 0.0f, s_j2 = 0.0f, s_e = 0.0f, s_abs = 0.0f, s_cells = 0.0f;
  uint32_t flags_acc = 0, n_rem = 0;
  if (s0 < s1) {
    if (tid < sp->n) {
      float c, psi;
      propagator<float>(dt * float(sp->inv_tau[tid]), c, psi);
      const float h1 = dt + dt * psi;
      sp_k[tid] = make_float4(float(sp->mass[tid]), c, h1, dt * psi);
      if (SB) {
        const float W = float(f.Omega) * h1;
        sp_w[tid] = make_float2(W, 1.0f / (1.0f + W * W));
      }
    }
    run_sums_init<float, 3>(rec);
    const double qO = SB ? f.q * f.Omega : 0.0;
    const double x_lo = B.ax[0].lo, dx0 = B.ax[0].d;
    if (SB && tid < RX) {
      const double v = qO * (x_lo + (double(ox + tid) + 0.5) * dx0);
      const float hi = float(v);
      xres[tid] = make_float2(hi, float(v - double(hi)));
    }
    const double t0 = *tdev;
    const int n0 = cb.n[0], n1 = cb.n[1], n2 = cb.n[2];
    const bool small = BOXES >= C3_SMALL || cb.ncell < (1 << 24);
    // the first particles are on their way while the window is staged; then
    // each chunk's are loaded one chunk ahead, their places two (past the
    // last: the last one again, not used)
    auto place = [&](uint32_t e) { return e < s1 ? e : s1 - 1; };
    uint32_t far = at32(order_src, place(s0 + RUN_THREADS + tid));
    uint32_t slot_n = at32(order_slot, place(s0 + tid));
    C3Raw nxt;
    c3_load(sh, at32(order_src, place(s0 + tid)), nxt);
    for (int r = tid; r < WC; r += RUN_THREADS) {
      const int a = r % RX, bq = (r / RX) % RY, cq = r / (RX * RY);
      int i = ox + a, j = oy + bq, k = oz + cq;
      if (cb.per[0]) i = wrap_index(i, n0);
      if (cb.per[1]) j = wrap_index(j, n1);
      if (cb.per[2]) k = wrap_index(k, n2);
      const bool in = i >= -1 && i <= n0 && j >= -1 && j <= n1 && k >= -1 && k <= n2;
      float gv[3] = {0.0f, 0.0f, 0.0f};
      if (in) {
        if (SB) {
          // velocity relative to the background shear, formed in FP64
          const double xc = x_lo + (double(i) + 0.5) * dx0;
#pragma unroll
          for (int m = 0; m < 3; ++m) {
            const double v = gas_comp(B, fl, xg, m, i, j, k);
            gv[m] = float(m == 1 ? v + qO * xc : v);
          }
        } else {
          const int64_t id = stored_index(B, i, j, k);
#pragma unroll
          for (int m = 0; m < 3; ++m) gv[m] = fl.vel[m][id];
        }
      }
      gas[r] = make_float4(gv[0], gv[1], gv[2], 0.0f);
#pragma unroll
      for (int m = 0; m < 4; ++m) dep[m * WC + r] = 0.0;
    }
    const float Om = float(f.Omega);
    const float qOdx = float(qO * dx0);
    const float g0c = float(f.g[0]), g1c = float(f.g[1]), g2c = float(f.g[2]);
    const bool cg = !SB && f.kind == FORCE_CONST;
    const float gz_c = SB && f.vertical_gravity ? -Om * Om : 0.0f;
    const float z_lo = float(B.ax[2].lo), dz = float(B.ax[2].d);
    __syncthreads();
    for (uint32_t cb0 = s0; cb0 < s1; cb0 += RUN_THREADS) {
      const bool has = cb0 + tid < s1;
      const C3Raw cur = nxt;
      const uint32_t i = slot_n;
      slot_n = at32(order_slot, place(cb0 + RUN_THREADS + tid));
      c3_load(sh, far, nxt);
      far = at32(order_src, place(cb0 + 2 * RUN_THREADS + tid));
      const int32_t cid = has ? cur.cell : -1;
      bool live = cid >= cb.cell_base && cid < cb.cell_base + cb.ncell;
      bool deferred = false, removed = false;
      if (cid >= 0 && !live) flags_acc |= DUST_FLAG_BAD_CELL;
      int idx[3] = {td.i0, td.j0, td.k0};
      float off[3] = {cur.off[0], cur.off[1], cur.off[2]}, mom[3] = {cur.mom[0], cur.mom[1], cur.mom[2]};
      if (live) {
        bool bad = false;
#pragma unroll
        for (int d = 0; d < 3; ++d) bad |= !(off[d] >= -0.5f && off[d] < 0.5f);
        if (bad) flags_acc |= DUST_FLAG_OFFSET_RANGE;
        c3_unravel(cid - cb.cell_base, n0, n1, B.ax[0].inv_n, B.ax[1].inv_n, idx, small);
        // half drift to x^{n+1/2} (periodic images, open faces remove, a
        // shear-periodic x face defers)
#pragma unroll
        for (int d = 0; d < 3; ++d) idx[d] = c3_move(idx[d], off[d], mom[d], cb.hinv[d]);
        if ((unsigned)idx[0] >= (unsigned)n0 || (unsigned)idx[1] >= (unsigned)n1 || (unsigned)idx[2] >= (unsigned)n2) {
#pragma unroll
          for (int d = 0; d < 3; ++d)
            if (idx[d] < 0 || idx[d] >= cb.n[d]) {
              if (cb.per[d]) idx[d] = c3_wrap(idx[d], cb.n[d]);
              else if (d == 0 && cb.shear) deferred = true;
              else removed = true;
            }
        }
      }
      const int la = win_coord(idx[0], ox, n0, RX, cb.per[0]), lb = win_coord(idx[1], oy, n1, RY, cb.per[1]),
                lcz = win_coord(idx[2], oz, n2, RZ, cb.per[2]);
      live = live && !removed;
      deferred = live & (deferred | !((la >= 1) & (la <= RX - 2) & (lb >= 1) & (lb <= RY - 2) & (lcz >= 1) &
                                      (lcz <= RZ - 2)));
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
      const int r0 = live ? la + RX * (lb + RY * lcz) : -1;
      float q[4] = {0.0f, 0.0f, 0.0f, 0.0f};
      Stencil<float> st;
#pragma unroll
      for (int d = 0; d < 3; ++d)
#pragma unroll
        for (int a = 0; a < 3; ++a) st.w[d][a] = 0.0f;
      int32_t ncell = -1;
      if (live) {
#pragma unroll
        for (int d = 0; d < 3; ++d) c3_weights<BOXES == C3_TSC>(cb.tsc[d], off[d], st.w[d]);
        // gather (Eq. Delta_vp), one z-plane of the stencil at a time
        float v[3] = {0.0f, 0.0f, 0.0f};
        int rr = r0 - RX * RY - RX;
#pragma unroll 1
        for (int c = 0; c < 3; ++c, rr += RX * RY) {
          const float wz = c == 0 ? st.w[2][0] : c == 1 ? st.w[2][1] : st.w[2][2];
          float4 g[9];
#pragma unroll
          for (int q9 = 0; q9 < 9; ++q9) g[q9] = gas[rr + RX * (q9 / 3) + (q9 % 3) - 1];
#pragma unroll
          for (int bb = 0; bb < 3; ++bb) {
            const float4 g0 = g[3 * bb], g1 = g[3 * bb + 1], g2 = g[3 * bb + 2];
            const float ux = st.w[0][0] * g0.x + st.w[0][1] * g1.x + st.w[0][2] * g2.x;
            const float uy = st.w[0][0] * g0.y + st.w[0][1] * g1.y + st.w[0][2] * g2.y;
            const float uz = st.w[0][0] * g0.z + st.w[0][1] * g1.z + st.w[0][2] * g2.z;
            const float wbc = st.w[1][bb] * wz;
            v[0] += wbc * ux;
            v[1] += wbc * uy;
            v[2] += wbc * uz;
          }
        }
        // kick (Eq. exp_midpoint; App. B.1 Eq. standard_SB_exp_midpoint)
        int spc = p.species ? cur.species : 0;
        flags_acc |= spc >= sp->n ? (uint32_t)DUST_FLAG_BAD_CELL : 0u;
        spc = spc >= sp->n ? 0 : spc;
        const float4 kc = sp_k[spc];
        const float m = kc.x, c = kc.y, h1 = kc.z, dtp = kc.w;
        float dp[3], jj[3];
        if constexpr (SB) {
          // y relative to the background shear: v_y + q Omega x at x^{n+1/2}
          const float2 xr = xres[la];
          const float uy = (mom[1] + xr.x) + fmaf(qOdx, off[0], xr.y);
          const float s0_ = v[0] - mom[0], s1_ = v[1] - uy, s2_ = v[2] - mom[2];
          const float gz = gz_c * (z_lo + (float(idx[2]) + 0.5f + off[2]) * dz);
          const float an0 = 2.0f * Om * uy, an1 = -2.0f * Om * mom[0];
          const float r0_ = c * s0_ + h1 * an0, r1_ = c * s1_ + h1 * an1;
          const float2 wk = sp_w[spc];
          const float W = wk.x, den = wk.y;
          dp[0] = (r0_ + W * r1_) * den;
          dp[1] = (r1_ - W * r0_) * den;
          dp[2] = c * s2_ + h1 * gz;
          const float a0 = an0 + Om * dp[1], a1 = an1 - Om * dp[0];
          jj[0] = c * s0_ + dtp * a0;
          jj[1] = c * s1_ + dtp * a1;
          jj[2] = c * s2_ + dtp * gz;
        } else {
          const float gk[3] = {cg ? g0c : 0.0f, cg ? g1c : 0.0f, cg ? g2c : 0.0f};
#pragma unroll
          for (int k = 0; k < 3; ++k) {
            const float sk = v[k] - mom[k];
            dp[k] = c * sk + h1 * gk[k];
            jj[k] = c * sk + dtp * gk[k];
          }
        }
        float e = 0.0f, cells = 0.0f;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          const float vbar = mom[k] + 0.5f * dp[k];
          e += vbar * jj[k];
          q[k] = -m * jj[k];   // deposits carry the minus sign of Eq. dust_feedback_final
          cells = fmaxf(cells, fabsf(vbar) * cb.dtinv[k]);
          mom[k] += dp[k];
        }
        q[3] = -m * e;
        s_cells = fmaxf(s_cells, cells);
        s_j0 -= q[0];
        s_j1 -= q[1];
        s_j2 -= q[2];
        s_e -= q[3];
        s_abs += fabsf(q[0]) + fabsf(q[1]) + fabsf(q[2]);
      }
      run_sums<float, 3, 4>(dep, RX, RY, WC, rec, r0, live, q, st);
      if (live) {
        // second half drift to x^{n+1}
        bool alive = true;
#pragma unroll
        for (int d = 0; d < 3; ++d) idx[d] = c3_move(idx[d], off[d], mom[d], cb.hinv[d]);
        if ((unsigned)idx[0] >= (unsigned)n0 || (unsigned)idx[1] >= (unsigned)n1 || (unsigned)idx[2] >= (unsigned)n2) {
          if (cb.shear && (idx[0] < 0 || idx[0] >= n0)) shear_image<float, false>(B, f, t0 + double(dt), idx, off, mom);
#pragma unroll
          for (int d = 0; d < 3; ++d)
            if (idx[d] < 0 || idx[d] >= cb.n[d]) {
              if (cb.per[d] || (d == 0 && cb.shear)) idx[d] = c3_wrap(idx[d], cb.n[d]);
              else alive = false;
            }
        }
        ncell = alive ? c3_cell_id(cb, idx[0], idx[1], idx[2], small) : -1;
        removed = !alive;
      } else if (deferred || (!removed && has)) {
        // stored as it came: for the deferred-particle kernel, or a cell id of
        // no box
        ncell = cid;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          off[d] = cur.off[d];
          mom[d] = cur.mom[d];
        }
      }
      // (a particle removed in the first half drift keeps the offsets and
      // momenta it had when it left)
      n_rem += removed ? 1u : 0u;
      if (has) {
        at32(p.cell, i) = ncell;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          at32(p.off[d], i) = off[d];
          at32(p.mom[d], i) = mom[d];
        }
        if (p.species) at32(p.species, i) = (uint8_t)cur.species;
        if (p.id) at32(p.id, i) = cur.id;
      }
    }
    __syncthreads();
    // the deposit window to the grid (periodic images to their cells; uniform
    // cell volume)
    const double iv = inv_volume(B, 0, 0, 0);
    for (int r = tid; r < WC; r += RUN_THREADS) {
      const int a = r % RX, bq = (r / RX) % RY, cq = r / (RX * RY);
      int i = ox + a, j = oy + bq, k = oz + cq;
      if (cb.per[0]) i = wrap_index(i, n0);
      if (cb.per[1]) j = wrap_index(j, n1);
      if (cb.per[2]) k = wrap_index(k, n2);
      const bool in = i >= -1 && i <= n0 && j >= -1 && j <= n1 && k >= -1 && k <= n2;
      if (!in) continue;
      const int64_t id = stored_index(B, i, j, k);
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const double x = dep[m * WC + r];
        if (x != 0.0) unsafeAtomicAdd(&fl.dep[m][id], float(x * iv));
      }
    }
  }
  if (dg) {
    if (n_rem) {
      atomicAdd(&dg->n_removed, (unsigned long long)n_rem);
      flags_acc |= DUST_FLAG_LEFT_OPEN;
    }
    if (flags_acc) atomicOr(&dg->flags, (unsigned)flags_acc);
    // diagnostics: the workgroup's FP64 sums to its own slot of `part` (in the
    // records' place)
    double (*red)[PART_WORDS] = reinterpret_cast<double (*)[PART_WORDS]>(rec);
    __syncthreads();
    double s[PART_WORDS] = {double(s_j0), double(s_j1), double(s_j2), double(s_e), double(s_abs), double(s_cells),
                            0.0, 0.0};
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

void launch_c3_cells(const FusedPlan& plan, const PView<float>& p, const FusedMove<float>& mv, const Box* boxes_d,
                     const FView<float>& fl, const Forces& f, const Species* sp, double dt, const double* tdev,
                     const int64_t* bin_start, const double* xg, DiagDev* dg, bool sums, hipStream_t st) {
  const TileShape& t = plan.tile;
  const size_t wc = (size_t)(t.t[0] + 2) * (t.t[1] + 2) * (t.t[2] + 2);
  const size_t lds = wc * (4 * sizeof(double) + sizeof(float4)) + (size_t)(t.t[0] + 2) * sizeof(float2);
  auto run = [&](auto kern) {
    const int split = cells_split(plan.ntiles, p.n, false);
    hipLaunchKernelGGL(kern, dim3(plan.ntiles * split), dim3(RUN_THREADS), lds, st, plan.tiles_d, split, t.t[0], t.t[1], t.t[2], p,
                       mv.sh, boxes_d, fl, f, sp, float(dt), tdev, bin_start, xg, dg, plan.part_d, (int)sums,
                       plan.defer_list, plan.defer_count, mv.order_src, mv.slot_of);
  };
  const bool sb = f.kind == FORCE_SHEARBOX;
  if (plan.small && plan.tsc) {
    if (sb) run(k_c3_cells<true, C3_TSC>);
    else run(k_c3_cells<false, C3_TSC>);
  } else if (plan.small) {
    if (sb) run(k_c3_cells<true, C3_SMALL>);
    else run(k_c3_cells<false, C3_SMALL>);
  } else {
    if (sb) run(k_c3_cells<true, C3_ANY>);
    else run(k_c3_cells<false, C3_ANY>);
  }
}

}  // namespace dust
