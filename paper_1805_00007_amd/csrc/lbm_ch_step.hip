// gfx950 time-step kernels of the lattice Boltzmann Cahn-Hilliard solver
// (Zhang, Guo & Liang, arXiv:1805.00007).  The public contract, the method and the
// boundary rules are stated in include/lbm_ch.h; this file holds the fused phase-field
// step (single lattice and batched); the coupled Navier-Stokes step is in lbm_ch_ns.hip.
//
// The hot kernel, k_phi_step, is one fused pull-scheme update of all nine
// phase-field populations.  A block owns a strip of TX columns and marches down TY
// rows of it.  Per row it keeps three rolling rings in LDS:
//   stage 1, row y+2: pull g_i(x) = g_i*(x - c_i), phi = sum g_i, q = phi u   (Eq. macroscopicg)
//   stage 2, row y+1: mu = f'(phi) - kappa lap(phi), D = div q                 (Eqs. mu, mark3)
//   stage 3, row y  : grad mu, grad D (and grad p), F = F1 + F2, g^eq, S, BGK,
//                     store g*                                                 (Eqs. t0-phiu, mark3, geq, liangFi, LB)
// so every value is computed once per node and the only HBM traffic is the nine
// populations in and out (72 bytes per node update in float32).  The pops of a row
// are pulled two iterations before they are collided and stay in registers; the
// pull for the next row is issued before the barriers so that its latency overlaps
// the stencil work.  Four lanes of the block also compute phi (and mu, D) of the
// two halo columns on each side.  A row strip of the domain is handed to blocks in
// an order that keeps a band of neighbouring strips on one XCD (one L2), so the
// halo rows a block re-reads are L2 hits.
#include "lbm_ch_device.h"
#include "lbm_ch_stencil.h"

namespace lbmch {
namespace {

// ---------------------------------------------------------------------------------
// Fused phase-field step.
//   VMODE VEL_SEP: u = tf ax[x] ay[y]; VEL_FIELD: u = tf ux[y][x];
//   VEL_NSFIELD: u, p from the NS step, F1 = (phi/rho)(F_s + F_b - grad p).
// One row record of the register pipeline: the pulled populations (plus velocity and
// pressure in the field modes) and the order parameter and velocity of the row.
struct RowRec {
  float g[9];
  float lu, lv, lp;       // loaded velocity / pressure (field modes)
  float phi, lo, u, v;    // stage-1 results (u, v in the field modes)
  float fy_u, fy_v;       // separable mode: ay[y], by[y] as loaded, then times tf
  float xpx, xpy;         // model 3: X of the previous step at this node
};

#ifndef WPE_PHI
#define WPE_PHI 4
#endif
// One tile of the step: strip (L % nstrips) of TX columns, row chunk L / nstrips.
// MODEL 1: F = F1; 2: F = F1 + K grad(div(phi u)) (Eq. mark3); 3: Eq. F2-1 with the
// time derivatives as one-step differences of X = cA F1 + cB grad mu, stored per node.
// REC: also store phi of every marched row (the source state's order parameter) to
// a.phi_rec.
template <int TX, bool WALLS, int VMODE, int MODEL, int ST, bool REC = false>
__device__ __forceinline__ void phi_tile(const StepArgs& a, const int L) {
  constexpr bool MODEL2 = MODEL >= 2;
  constexpr bool HIST = MODEL == 3;
  constexpr bool NSC = VMODE == VEL_NSFIELD;
  constexpr bool VFIELD = VMODE != VEL_SEP;
  constexpr int LW = TX + 4;
  constexpr int QR = MODEL2 ? 4 : 1;
  constexpr int PR = NSC ? 8 : 1;
  __shared__ float s_phi[4][LW];
  __shared__ float s_mu[4][LW];
  __shared__ float s_qx[QR][LW];
  __shared__ float s_qy[QR][LW];
  __shared__ float s_d[QR][LW];
  __shared__ float s_p[PR][LW];

  const Coef& c = a.c;
  const int nx = a.nx, ny = a.ny;
  const uint32_t nodes = (uint32_t)nx * ny;
  const uint32_t pitch = a.pitch;
  const uint32_t rb = (uint32_t)nx * 4u;
  const rsrc_t rsrc = make_rsrc(a.src, pop_bytes(ST, pitch, ny));
  const rsrc_t rdst = make_rsrc(a.dst, pop_bytes(ST, pitch, ny));
  rsrc_t ru, rv, rp;
  if (VFIELD) {
    ru = make_rsrc(a.ux, nodes * 4u);
    rv = make_rsrc(a.uy, nodes * 4u);
  }
  if (NSC) rp = make_rsrc(a.pf, nodes * 4u);
  rsrc_t rxh;
  if (HIST) rxh = make_rsrc(a.xh, 2u * nodes * 4u);
  rsrc_t rrec;
  if (REC) rrec = make_rsrc(a.phi_rec, nodes * 4u);

  const int t = threadIdx.x;
  const int x0 = (L % a.nstrips) * TX;
  const int chunk = L / a.nstrips;
  const int rows = min(a.ty, ny - chunk * a.ty);
  // Vertically adjacent chunks march in opposite directions, so the two blocks that
  // share a chunk boundary pass it at the same moment (both at their start or both
  // at their end) and the halo rows one re-reads are still in L2.
  const int dir = (chunk & 1) ? -1 : 1;
  const int y0 = dir > 0 ? chunk * a.ty : chunk * a.ty + rows - 1;  // first row marched

  // Own column (wrapped) and its neighbours.
  const int xl = x0 + t;
  const bool active = xl < nx;
  const int xc = xl % nx;
  const uint32_t vc = xc;
  const uint32_t vm = xc == 0 ? nx - 1 : xc - 1;
  const uint32_t vp = xc == nx - 1 ? 0 : xc + 1;
  // Halo lanes t < 4: logical columns x0-2, x0-1, x0+TX, x0+TX+1 -> LDS 0, 1, TX+2, TX+3.
  // They sit in wave 0; the other waves skip the halo pull (a scalar branch).
  const bool hl = t < 4;
  const bool hwave = __builtin_amdgcn_readfirstlane(t) < 64;
  const int hlog = t < 2 ? x0 - 2 + t : x0 + TX - 2 + t;
  const int hc = ((hlog % nx) + nx) % nx;
  // Every lane of wave 0 issues the halo pull (a wave-uniform branch, so the wait for
  // the halo row is the only wait inside it); lanes other than the four halo lanes use
  // an offset beyond the buffer, for which a raw buffer load returns 0 without
  // accessing memory.
  constexpr uint32_t OOB = 0x3FFFFFC0u;  // column index whose byte offset exceeds any buffer
  const uint32_t hvc = hl ? hc : OOB;
  const uint32_t hvm = hl ? (hc == 0 ? nx - 1 : hc - 1) : OOB;
  const uint32_t hvp = hl ? (hc == nx - 1 ? 0 : hc + 1) : OOB;
  const int hj = t < 2 ? t : TX + t;
  const int j = t + 2;
  const int j2 = t == 0 ? 1 : TX + 2;  // stage-2 halo column of lanes 0 and 1

  float axc = 0.f, bxc = 0.f, axh = 0.f, bxh = 0.f;
  if (VMODE == VEL_SEP) {
    axc = a.ax[xc];
    bxc = a.bx[xc];
    if (hl) {
      axh = a.ax[hc];
      bxh = a.bx[hc];
    }
  }

  // Issue the pull of logical row r at one column (plus velocity and pressure in the
  // field modes) so that one wait covers all of it.
  auto issue = [&](int r, uint32_t cc, uint32_t cm, uint32_t cp, RowRec& R, bool own = true) {
    float sg;
    const int sr = row_of<WALLS>(r, ny, sg);
    pull9<WALLS, ST>(rsrc, pitch, ny, sr, cc, cm, cp, R.g);
    if (HIST && own) {
      R.xpx = ldb(rxh, cc * 4u, (uint32_t)sr * rb);
      R.xpy = ldb(rxh, cc * 4u, nodes * 4u + (uint32_t)sr * rb);
    }
    if (VMODE == VEL_SEP) {
      // row factors of the separable velocity, fetched with the pull so that one wait
      // covers both (a later load would make the wait cover the whole prefetch)
      R.fy_u = a.ay[sr];
      R.fy_v = a.by[sr];
    }
    if (VFIELD) {
      R.lu = ldb(ru, cc * 4u, (uint32_t)sr * rb);
      R.lv = ldb(rv, cc * 4u, (uint32_t)sr * rb);
      if (NSC) R.lp = ldb(rp, cc * 4u, (uint32_t)sr * rb);
    }
  };
  // Stage 1 for logical row r: phi (and q = phi u, p) into the rings at column jj.
  auto stage1 = [&](int r, RowRec& R, int jj, float axv, float bxv, bool wr = true) {
    float sg;
    row_of<WALLS>(r, ny, sg);
    R.phi = sum9(R.g, R.lo);
    if (__builtin_expect(!__builtin_isfinite(R.phi), 0) && a.nonfinite) *a.nonfinite = 1;
    float u, v;
    if (VMODE == VEL_SEP) {
      R.fy_u *= a.tf * sg;
      R.fy_v *= a.tf * sg;
      u = axv * R.fy_u;
      v = bxv * R.fy_v;
    } else {
      u = R.u = a.tf * R.lu * sg;
      v = R.v = a.tf * R.lv * sg;
    }
    if (!wr) return;
    s_phi[r & 3][jj] = R.phi;
    if (MODEL2) {
      s_qx[r & 3][jj] = R.phi * u;
      s_qy[r & 3][jj] = R.phi * v;
    }
    if (NSC) s_p[r & 7][jj] = R.lp;
  };
  // Stage 2 for logical row r at LDS column jj: mu (Eq. mu) and D = div(phi u).
  auto stage2 = [&](int r, int jj) {
    const float* pm = s_phi[(r - 1) & 3];
    const float* p0 = s_phi[r & 3];
    const float* pp = s_phi[(r + 1) & 3];
    s_mu[r & 3][jj] = mu_bulk(c, p0[jj]) - c.kappa * lap9(pm, p0, pp, jj);
    if (MODEL2) {
      s_d[r & 3][jj] = ddx(s_qx[(r - 1) & 3], s_qx[r & 3], s_qx[(r + 1) & 3], jj) +
                       ddy(s_qy[(r - 1) & 3], s_qy[r & 3], s_qy[(r + 1) & 3], jj);
    }
  };
  // Stage 3 for lattice row y: F = F1 (+ F2), collision, store.
  auto stage3 = [&](int y, RowRec& R) {
    // Lanes past the right edge of a ragged last strip wrap to columns another strip
    // owns and compute the very same values from the very same inputs, so their stores
    // duplicate identical data; they need no branch (which would make the wait for the
    // next row's pull also wait for this row's stores).  Model 3 keeps the branch: a
    // duplicate lane could read a history value its owner has already replaced.
    if (HIST && !active) return;
    const float* mm = s_mu[(y - 1) & 3];
    const float* m0 = s_mu[y & 3];
    const float* mp = s_mu[(y + 1) & 3];
    const float mux = ddx(mm, m0, mp, j), muy = ddy(mm, m0, mp, j);
    const float rho = c.a * R.phi + c.b;
    float tx = -R.phi * mux, ty = -R.phi * muy;
    if (NSC) {
      const float* qm = s_p[(y - 1) & 7];
      const float* q0 = s_p[y & 7];
      const float* qp = s_p[(y + 1) & 7];
      tx += rho * c.accel_x - ddx(qm, q0, qp, j);
      ty += -(rho - c.rho_mean) * c.gravity - ddy(qm, q0, qp, j);
    }
    const float s1 = R.phi * rcp(rho);
    float fx = s1 * tx, fy = s1 * ty;
    if (HIST) {  // (2 tau - 1 + 3K) dF1/dt + 3 cs^2 eta K d(grad mu)/dt of Eq. F2-1
      const float xx = c.x_f1 * fx + c.x_mu * mux, xy = c.x_f1 * fy + c.x_mu * muy;
      stb_nt(rxh, xx, vc * 4u, (uint32_t)y * rb);
      stb_nt(rxh, xy, vc * 4u, nodes * 4u + (uint32_t)y * rb);
      if (!a.xfirst) {
        fx += xx - R.xpx;
        fy += xy - R.xpy;
      }
    }
    if (MODEL2) {
      const float* dm = s_d[(y - 1) & 3];
      const float* d0 = s_d[y & 3];
      const float* dp = s_d[(y + 1) & 3];
      fx += c.k2 * ddx(dm, d0, dp, j);
      fy += c.k2 * ddy(dm, d0, dp, j);
    }
    const float u = VMODE == VEL_SEP ? axc * R.fy_u : R.u;
    const float v = VMODE == VEL_SEP ? bxc * R.fy_v : R.v;
    if (REC) stb_nt(rrec, R.phi, vc * 4u, (uint32_t)y * rb);
    collide_g(c, R.phi, R.lo, m0[j], u, v, fx, fy, R.g);
    finish_store<ST>(rdst, pitch, vc, (uint32_t)y, (double)R.phi + (double)R.lo, R.g);
  };

  // Prologue: rows y0-2d .. y0+2d through stage 1, rows y0-d and y0 through stage 2.
  //
  // Register pipeline.  Iteration y issues the pull of row y+3d first, then runs stage
  // 2 of row y+d and stage 3 of row y while it is in flight, and consumes it (stage 1)
  // last, so no load is outstanding when the loop branches back (a record with a load
  // in flight is then never moved between registers, which would make the wave wait
  // for every outstanding load).  A, B, C hold rows y, y+d, y+2d; N receives y+3d.
  const int d = dir;
  RowRec A, B, C, N, H0;
  {
    // wave 0 pulls the first two halo rows with the own rows, so the prologue has two
    // dependent round trips to memory instead of three
    RowRec T0, T1, U0, U1;
    if (hwave) {
      issue(y0 - 2 * d, hvc, hvm, hvp, U0, false);
      issue(y0 - d, hvc, hvm, hvp, U1, false);
    }
    issue(y0 - 2 * d, vc, vm, vp, T0);
    issue(y0 - d, vc, vm, vp, T1);
    issue(y0, vc, vm, vp, A);
    issue(y0 + d, vc, vm, vp, B);
    if (hwave) {
      stage1(y0 - 2 * d, U0, hj, axh, bxh, hl);
      stage1(y0 - d, U1, hj, axh, bxh, hl);
      issue(y0, hvc, hvm, hvp, U0, false);
      issue(y0 + d, hvc, hvm, hvp, U1, false);
    }
    stage1(y0 - 2 * d, T0, j, axc, bxc);
    stage1(y0 - d, T1, j, axc, bxc);
    stage1(y0, A, j, axc, bxc);
    stage1(y0 + d, B, j, axc, bxc);
    if (hwave) {
      stage1(y0, U0, hj, axh, bxh, hl);
      stage1(y0 + d, U1, hj, axh, bxh, hl);
    }
  }
  if (hwave) issue(y0 + 2 * d, hvc, hvm, hvp, H0, false);
  issue(y0 + 2 * d, vc, vm, vp, C);
  __syncthreads();
  stage2(y0 - d, j);
  stage2(y0, j);
  if (t < 2) {
    stage2(y0 - d, j2);
    stage2(y0, j2);
  }
  __syncthreads();
  // row y0+2d shares its ring slot with y0-2d, which stage 2 no longer needs
  if (hwave) stage1(y0 + 2 * d, H0, hj, axh, bxh, hl);
  stage1(y0 + 2 * d, C, j, axc, bxc);

  // One marching row.  On a block's last row the pull of y+3d is not needed; it is
  // clamped to the last row the block does need (already in cache), so the pull has no
  // branch and fetches nothing extra, and its stage 1 is skipped (a scalar branch), so
  // the block does not wait for it.
  const int last_needed = y0 + (rows + 1) * d;
  // On tall tiles (bandwidth-bound marches) a wave raises its issue priority while it
  // puts its row's pull in flight, so waves about to load go before waves in their
  // compute stages (2048^2: 0.8 % faster with float32, ~6 % with 16-bit storage).  Short
  // tiles are latency-bound chains, where it costs a few per cent, and keep priority 0.
  const bool prio = a.ty >= 8;
#pragma unroll 1
  for (int k = 0; k < rows; ++k) {
    const int y = y0 + k * d;
    const int ynext = k + 1 < rows ? y + 3 * d : last_needed;
    __builtin_amdgcn_sched_barrier(0);
    if (prio) __builtin_amdgcn_s_setprio(2);
    if (hwave) issue(ynext, hvc, hvm, hvp, H0, false);
    __builtin_amdgcn_sched_barrier(0);
    issue(ynext, vc, vm, vp, N);
    __builtin_amdgcn_sched_barrier(0);
    if (prio) __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
    stage2(y + d, j);
    if (t < 2) stage2(y + d, j2);
    __syncthreads();
    stage3(y, A);
    __builtin_amdgcn_sched_barrier(0);
    // row y+3d takes the ring slot of row y-d, which no later stage reads
    if (k + 1 < rows) {
      if (hwave) stage1(y + 3 * d, H0, hj, axh, bxh, hl);
      stage1(y + 3 * d, N, j, axc, bxc);
    }
    A = B;
    B = C;
    C = N;
  }
}

// Model 3 carries two more values per row record; it gets the register budget of
// three waves per SIMD so that nothing spills.
template <int TX, bool WALLS, int VMODE, int MODEL, int ST, bool REC = false>
__global__ void __launch_bounds__(TX)
__attribute__((amdgpu_waves_per_eu(MODEL == 3 ? 3 : WPE_PHI, 8)))
k_phi_step(const StepArgs a) {
  int L = blockIdx.x;
  if (a.xcd_remap) {  // workgroup w runs on XCD w % 8: give each XCD a band of chunks
    const int per = gridDim.x >> 3;
    L = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  }
  phi_tile<TX, WALLS, VMODE, MODEL, ST, REC>(a, L);
}

// Batched step, one tile per workgroup: the tiles of many lattices (one instance table
// entry each) in one launch.  The tiles are numbered instance by instance; when the grid
// is a multiple of 8, XCD x (workgroups w with w % 8 == x) gets the contiguous range
// [x per, (x + 1) per), so vertically adjacent tiles of one lattice share an L2.  Same
// register budget as the single-lattice kernel.
template <int TX, int VMODE, bool MODEL2>
__global__ void __launch_bounds__(TX) __attribute__((amdgpu_waves_per_eu(WPE_PHI, 8)))
k_phi_batch(const BatchArgs b) {
  int v = blockIdx.x;
  if ((gridDim.x & 7) == 0) {
    const int per = gridDim.x >> 3;
    v = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  }
  if (v >= b.total) return;
  int lo_i = 0, hi_i = b.n;  // instance of tile v: start[inst] <= v < start[inst + 1]
  while (hi_i - lo_i > 1) {
    const int mid = (lo_i + hi_i) >> 1;
    if (b.start[mid] <= v) lo_i = mid; else hi_i = mid;
  }
  StepArgs a = b.args[lo_i];
  if (b.parity) {
    const void* t = a.src;
    a.src = a.dst;
    a.dst = const_cast<void*>(t);
  }
  phi_tile<TX, false, VMODE, MODEL2 ? 2 : 1, ST_F32>(a, v - b.start[lo_i]);
}

// Batched step, persistent: the tiles of many lattices (one instance table entry each)
// in one launch of a grid sized to the resident capacity.  The tiles are numbered instance by instance; XCD x (workgroups
// w with w % 8 == x) owns the contiguous range [x per, (x + 1) per) and its workgroups
// stride through it, so vertically adjacent tiles of one lattice share that XCD's L2.
// Every workgroup leaves the loop after at most ceil(per / slots) tiles.
#ifndef WPE_BATCH
#define WPE_BATCH 3
#endif
template <int TX, int VMODE, bool MODEL2>
__global__ void __launch_bounds__(TX) __attribute__((amdgpu_waves_per_eu(WPE_BATCH, 8)))
k_phi_batch_persistent(const BatchArgs b) {
  const int slots = gridDim.x >> 3;
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  const int per = (b.total + 7) >> 3;
  const int lo = xcd * per, hi = min(b.total, lo + per);
  int v = lo + slot;
  if (v >= hi) return;
  int lo_i = 0, hi_i = b.n;  // instance of tile v: start[inst] <= v < start[inst + 1]
  while (hi_i - lo_i > 1) {
    const int mid = (lo_i + hi_i) >> 1;
    if (b.start[mid] <= v) lo_i = mid; else hi_i = mid;
  }
  int inst = __builtin_amdgcn_readfirstlane(lo_i);
#pragma unroll 1
  for (; v < hi; v += slots) {
    // the table is read after the previous tile's stores: its values (the same in every
    // lane) are moved to scalar registers explicitly
    while (__builtin_amdgcn_readfirstlane(b.start[inst + 1]) <= v) ++inst;
    StepArgs a = wave_uniform(b.args[inst]);
    if (b.parity) {
      const void* t = a.src;
      a.src = a.dst;
      a.dst = const_cast<void*>(t);
    }
    phi_tile<TX, false, VMODE, MODEL2 ? 2 : 1, ST_F32>(
        a, v - __builtin_amdgcn_readfirstlane(b.start[inst]));
    __syncthreads();  // the LDS rings are reused by the next tile
  }
}

template <int TX, bool WALLS, int VMODE, int ST>
hipError_t phi_step_m(int model, const StepArgs& a, int nb, hipStream_t s) {
  if (model == 2)
    hipLaunchKernelGGL((k_phi_step<TX, WALLS, VMODE, 2, ST>), dim3(nb), dim3(TX), 0, s, a);
  else if (model == 1)
    hipLaunchKernelGGL((k_phi_step<TX, WALLS, VMODE, 1, ST>), dim3(nb), dim3(TX), 0, s, a);
  else if constexpr (ST == ST_F32)
    hipLaunchKernelGGL((k_phi_step<TX, WALLS, VMODE, 3, ST>), dim3(nb), dim3(TX), 0, s, a);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

template <int TX, bool PERSIST>
hipError_t phi_batch_t(int vmode, bool model2, const BatchArgs& b, int grid, hipStream_t s) {
#define LBM_BATCH_LAUNCH(V, M)                                                                 \
  if (PERSIST)                                                                                 \
    hipLaunchKernelGGL((k_phi_batch_persistent<TX, V, M>), dim3(grid), dim3(TX), 0, s, b); \
  else                                                                                         \
    hipLaunchKernelGGL((k_phi_batch<TX, V, M>), dim3(grid), dim3(TX), 0, s, b)
  if (vmode == VEL_SEP) {
    if (model2) { LBM_BATCH_LAUNCH(VEL_SEP, true); } else { LBM_BATCH_LAUNCH(VEL_SEP, false); }
  } else {
    if (model2) { LBM_BATCH_LAUNCH(VEL_FIELD, true); } else { LBM_BATCH_LAUNCH(VEL_FIELD, false); }
  }
#undef LBM_BATCH_LAUNCH
  return hipGetLastError();
}

template <int TX, bool WALLS, int ST>
hipError_t phi_step_v(int vmode, int model, const StepArgs& a, int nb, hipStream_t s) {
  switch (vmode) {
    case VEL_SEP: return phi_step_m<TX, WALLS, VEL_SEP, ST>(model, a, nb, s);
    case VEL_FIELD: return phi_step_m<TX, WALLS, VEL_FIELD, ST>(model, a, nb, s);
    default: return phi_step_m<TX, WALLS, VEL_NSFIELD, ST>(model, a, nb, s);
  }
}

template <int ST>
hipError_t phi_step_t(int tx, bool walls, int vmode, int model, const StepArgs& a,
                      int nb, hipStream_t s) {
  switch (tx) {
    case 64:
      return walls ? phi_step_v<64, true, ST>(vmode, model, a, nb, s)
                   : phi_step_v<64, false, ST>(vmode, model, a, nb, s);
    case 128:
      return walls ? phi_step_v<128, true, ST>(vmode, model, a, nb, s)
                   : phi_step_v<128, false, ST>(vmode, model, a, nb, s);
    case 256:
      return walls ? phi_step_v<256, true, ST>(vmode, model, a, nb, s)
                   : phi_step_v<256, false, ST>(vmode, model, a, nb, s);
    case 512:
      return walls ? phi_step_v<512, true, ST>(vmode, model, a, nb, s)
                   : phi_step_v<512, false, ST>(vmode, model, a, nb, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

#ifdef LBM_STEP_16BIT_TU
// The 16-bit storage instances of the step, in their own translation unit
// (lbm_ch_step16.hip, built with other code-generation options).
hipError_t launch_phi_step16(int tx, bool walls, int vmode, int model, int storage,
                             const StepArgs& a, int nblocks, hipStream_t s) {
  switch (storage) {
    case ST_F16: return phi_step_t<ST_F16>(tx, walls, vmode, model, a, nblocks, s);
    case ST_BF16: return phi_step_t<ST_BF16>(tx, walls, vmode, model, a, nblocks, s);
    default: return hipErrorInvalidValue;
  }
}
#else
bool phi_record_fused(bool walls, int vmode, int model, int storage) {
  return !walls && storage == ST_F32 && (vmode == VEL_SEP || vmode == VEL_FIELD) &&
         (model == 1 || model == 2);
}

template <int TX>
static hipError_t phi_record_t(int vmode, int model, const StepArgs& a, int nb, hipStream_t s) {
#define LBM_REC_LAUNCH(V, M) \
  hipLaunchKernelGGL((k_phi_step<TX, false, V, M, ST_F32, true>), dim3(nb), dim3(TX), 0, s, a)
  if (vmode == VEL_SEP) {
    if (model == 2) { LBM_REC_LAUNCH(VEL_SEP, 2); } else { LBM_REC_LAUNCH(VEL_SEP, 1); }
  } else {
    if (model == 2) { LBM_REC_LAUNCH(VEL_FIELD, 2); } else { LBM_REC_LAUNCH(VEL_FIELD, 1); }
  }
#undef LBM_REC_LAUNCH
  return hipGetLastError();
}

hipError_t launch_phi_record(int tx, int vmode, int model, const StepArgs& a, int nblocks,
                             hipStream_t s) {
  if (!phi_record_fused(false, vmode, model, ST_F32) || !a.phi_rec) return hipErrorInvalidValue;
  switch (tx) {
    case 64: return phi_record_t<64>(vmode, model, a, nblocks, s);
    case 128: return phi_record_t<128>(vmode, model, a, nblocks, s);
    case 256: return phi_record_t<256>(vmode, model, a, nblocks, s);
    case 512: return phi_record_t<512>(vmode, model, a, nblocks, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_phi_step(int tx, bool walls, int vmode, int model, int storage,
                           const StepArgs& a, int nblocks, hipStream_t s) {
  switch (storage) {
    case ST_F32: return phi_step_t<ST_F32>(tx, walls, vmode, model, a, nblocks, s);
    case ST_F16:
    case ST_BF16: return launch_phi_step16(tx, walls, vmode, model, storage, a, nblocks, s);
    default: return hipErrorInvalidValue;
  }
}

int phi_batch_blocks_per_cu(int tx, int vmode, bool model2) {
  int nb = 0;
  hipError_t e = hipErrorInvalidValue;
  const bool sep = vmode == VEL_SEP;
#define LBM_OCC(T)                                                                                                           \
  e = sep ? (model2 ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_phi_batch_persistent<T, VEL_SEP, true>, T, 0)     \
                    : hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_phi_batch_persistent<T, VEL_SEP, false>, T, 0))    \
          : (model2 ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_phi_batch_persistent<T, VEL_FIELD, true>, T, 0)   \
                    : hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_phi_batch_persistent<T, VEL_FIELD, false>, T, 0))
  switch (tx) {
    case 64: LBM_OCC(64); break;
    case 128: LBM_OCC(128); break;
    case 256: LBM_OCC(256); break;
    default: break;
  }
#undef LBM_OCC
  return e == hipSuccess && nb > 0 ? nb : 1;
}

template <bool PERSIST>
static hipError_t phi_batch_tx(int tx, int vmode, bool model2, const BatchArgs& b, int grid,
                               hipStream_t s) {
  switch (tx) {
    case 64: return phi_batch_t<64, PERSIST>(vmode, model2, b, grid, s);
    case 128: return phi_batch_t<128, PERSIST>(vmode, model2, b, grid, s);
    case 256: return phi_batch_t<256, PERSIST>(vmode, model2, b, grid, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_phi_batch(int tx, int vmode, bool model2, bool persistent, const BatchArgs& b,
                            int grid, hipStream_t s) {
  if (grid <= 0 || (grid & 7) != 0 || b.n <= 0) return hipErrorInvalidValue;
  return persistent ? phi_batch_tx<true>(tx, vmode, model2, b, grid, s)
                    : phi_batch_tx<false>(tx, vmode, model2, b, grid, s);
}
#endif  // LBM_STEP_16BIT_TU

}  // namespace lbmch
