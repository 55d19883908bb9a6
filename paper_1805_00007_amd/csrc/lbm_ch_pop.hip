// gfx950 kernel of the population step of the lattice Boltzmann Cahn-Hilliard solver
// (Zhang, Guo & Liang, arXiv:1805.00007) at any tau_g with a prescribed velocity, as a
// march in registers: for lattices whose two population buffers stay in the caches, where
// the tiles of lbm_ch_step.hip are bound by their barriers and halo rows.
#include "lbm_ch_device.h"
#include "lbm_ch_lanes.h"

#include <type_traits>

namespace lbmch {
namespace {

// The values of phi_tile (lbm_ch_step.hip), rounding by rounding: that kernel is compiled with
// implicit multiply-add contraction, which the compiler resolves alike in all its
// instances; here every fused multiply-add is written out where it stands there.
#pragma clang fp contract(off)

// The stencils of lbm_ch_device.h (ddx, ddy, lap9) at a lane, on the values of the rows y-1
// (m), y (0) and y+1 (p) in its column; the derivatives times 12.
__device__ __forceinline__ float lane_dx(float m, float o, float p) {
  return fmaf(4.0f, east(o) - west(o), ((east(p) + east(m)) - west(p)) - west(m));
}
__device__ __forceinline__ float lane_dy(float m, float p) {
  return fmaf(4.0f, p - m, ((east(p) + west(p)) - east(m)) - west(m));
}
__device__ __forceinline__ float lane_lap(float m, float o, float p) {
  const float axis = ((east(o) + west(o)) + p) + m;
  const float diag = ((east(p) + west(p)) + east(m)) + west(m);
  return fmaf(-20.0f, o, fmaf(4.0f, axis, diag)) * (1.0f / 6.0f);
}
constexpr float R12 = 1.0f / 12.0f;

// Collision of Eq. LB (collide_g) with F = (fx, fy).  The diagonal directions take u = au bu
// (separable velocity) and, for Model-I, fx = s1 tx as products.
template <int MODEL, bool SEP>
__device__ __forceinline__ void lane_collide(const Coef& c, float phi, float mu, float u, float v,
                                             float au, float bu, float fx, float fy, float s1,
                                             float tx, float g[9]) {
  const float A = fmaf(c.eta, mu, -(phi * (1.5f * fmaf(v, v, u * u))));
  const float om1 = 1.0f - c.omega;
  auto dir = [&](int i, float cu, float cf) {
    const float eq = fmaf(phi * cu, fmaf(4.5f, cu, 3.0f), A);
    g[i] = fmaf(om1, g[i], WT[i] * fmaf(c.omega, eq, c.srcg * cf));
  };
  dir(1, u, fx);
  dir(2, v, fy);
  dir(3, -u, -fx);
  dir(4, -v, -fy);
  auto sum_u = [&](float w) { return SEP ? fmaf(au, bu, w) : u + w; };
  auto sub_u = [&](float w) { return SEP ? fmaf(-au, bu, w) : w - u; };
  auto sum_f = [&](float w) { return MODEL == 1 ? fmaf(s1, tx, w) : fx + w; };
  auto sub_f = [&](float w) { return MODEL == 1 ? fmaf(-s1, tx, w) : w - fx; };
  dir(5, sum_u(v), sum_f(fy));
  dir(6, sub_u(v), sub_f(fy));
  dir(7, sub_u(-v), sub_f(-fy));
  dir(8, sum_u(-v), sum_f(-fy));
}

// One wave marches up the rows of a strip of 64 lanes, one lane per column, as march_tile in
// lbm_ch_march.hip does, with the nine populations of a row carried from its pull (issued
// three rows ahead) to its collision two rows later: stages and arithmetic of phi_tile
// (lbm_ch_step.hip), no LDS and no barrier.  A strip yields 60 columns.  Bound by the
// caches' bandwidth and, below 1000^2, by latency: 768^2 float32 11.8 us a step (3.6 TB/s)
// against the tile's 17.1, 1500 x 1003 21.8 (5.0 TB/s) against 32.8.
template <bool WALLS, int VMODE, int MODEL, int ST>
__global__ void __launch_bounds__(256) k_pop_march(const StepArgs a, const int total) {
  constexpr bool VFIELD = VMODE == VEL_FIELD, MODEL2 = MODEL >= 2, HIST = MODEL == 3;
  constexpr int M = 2, OUT = POP_MARCH_OUT;
  static_assert(OUT == 64 - 2 * M, "a strip and its margins are one wave");
  const int per = gridDim.x >> 3;  // one band of strips and chunks per XCD
  const int L = ((blockIdx.x & 7) * per + (blockIdx.x >> 3)) * 4 +
                __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (L >= total) return;
  const Coef& c = a.c;
  const int nx = a.nx, ny = a.ny;
  const uint32_t nodes = (uint32_t)nx * ny, pitch = a.pitch;
  const uint32_t rb = (uint32_t)nx * 4u;
  const rsrc_t rsrc = make_rsrc(a.src, pop_bytes(ST, pitch, ny));
  const rsrc_t rdst = make_rsrc(a.dst, pop_bytes(ST, pitch, ny));
  rsrc_t ru, rv, rxh;
  if (VFIELD) {
    ru = make_rsrc(a.ux, nodes * 4u);
    rv = make_rsrc(a.uy, nodes * 4u);
  }
  if (HIST) rxh = make_rsrc(a.xh, 2u * nodes * 4u);

  const int lane = threadIdx.x & 63;
  const int x0 = (L % a.mstrips) * OUT;
  const int y0 = (L / a.mstrips) * a.mty;
  const int rows = min(a.mty, ny - y0);
  const int xl = x0 - M + lane;
  const int x = ((xl % nx) + nx) % nx;
  const uint32_t xm = x == 0 ? nx - 1 : x - 1, xp = x == nx - 1 ? 0 : x + 1;
  const bool own = lane >= M && lane < M + OUT && xl < nx;
  constexpr uint32_t OOB = 0x3FFFFFC0u;  // as in march_tile
  const uint32_t cst = own ? (uint32_t)x : OOB;
  float axc = 0.f, bxc = 0.f;
  if (!VFIELD) {
    axc = a.ax[x];
    bxc = a.bx[x];
  }

  struct In {
    float g[9], a, b, sg, hx, hy;
  };
  In in[3];
  int row = y0 - M;               // logical row that is pulled next
  const int end = y0 + rows + M;  // one past the last needed (repeated beyond: in cache)
  auto fetch = [&](In& I) {
    const int sr = row_of<WALLS>(row, ny, I.sg);
    pull9<WALLS, ST>(rsrc, pitch, ny, sr, (uint32_t)x, xm, xp, I.g);
    if (VFIELD) {
      I.a = ldb(ru, (uint32_t)x * 4u, (uint32_t)sr * rb);
      I.b = ldb(rv, (uint32_t)x * 4u, (uint32_t)sr * rb);
    } else {
      I.a = ld_uniform(a.ay, sr);
      I.b = ld_uniform(a.by, sr);
    }
    if (HIST) {  // used in own rows only, which no other wave writes
      I.hx = ldb(rxh, (uint32_t)x * 4u, (uint32_t)sr * rb);
      I.hy = ldb(rxh, (uint32_t)x * 4u, nodes * 4u + (uint32_t)sr * rb);
    }
    if (row + 1 < end) ++row;
  };

  float g[3][9], ph[3], lo[3], u[3], v[3], qx[3], qy[3], mu[3], dv[3], hx[3], hy[3];
  // Row K enters slot K % 3: stage 0, its sums; 1, mu and D of the row before; 2, collision
  // and store of row y0 + i, the one before that.
  auto push = [&](auto K, auto STAGE, int i) {
    constexpr int j = decltype(K)::value % 3, j1 = (j + 2) % 3, j2 = (j + 1) % 3;
    constexpr int stage = decltype(STAGE)::value;
    In& I = in[j];
#pragma unroll
    for (int q = 0; q < 9; ++q) g[j][q] = I.g[q];
    ph[j] = sum9(g[j], lo[j]);
    if (__builtin_expect(!__builtin_isfinite(ph[j]), 0) && a.nonfinite) *a.nonfinite = 1;
    // the velocity (field) or its row factors (separable)
    u[j] = VFIELD ? a.tf * I.a * I.sg : I.a * (a.tf * I.sg);
    v[j] = VFIELD ? a.tf * I.b * I.sg : I.b * (a.tf * I.sg);
    if (HIST) {
      hx[j] = I.hx;
      hy[j] = I.hy;
    }
    fetch(I);
    if (MODEL2) {
      qx[j] = ph[j] * (VFIELD ? u[j] : axc * u[j]);
      qy[j] = ph[j] * (VFIELD ? v[j] : bxc * v[j]);
    }
    if (stage < 1) return;
    mu[j1] = fmaf(c.beta2 * (ph[j1] - c.phia) * (ph[j1] - c.phib), fmaf(2.0f, ph[j1], -c.phia) - c.phib,
                  -(c.kappa * lane_lap(ph[j2], ph[j1], ph[j])));
    if (MODEL2) dv[j1] = fmaf(lane_dx(qx[j2], qx[j1], qx[j]), R12, lane_dy(qy[j2], qy[j]) * R12);
    if (stage < 2) return;
    // rows y - 1, y, y + 1 of mu and D are in slots j, j2, j1
    const float phi = ph[j2];
    const float mux = lane_dx(mu[j], mu[j2], mu[j1]) * R12, muy = lane_dy(mu[j], mu[j1]) * R12;
    const float rho = fmaf(c.a, phi, c.b);
    const float tx = -phi * mux, ty = -phi * muy;
    const float s1 = phi * rcp(rho);
    float fx = s1 * tx, fy = s1 * ty;
    const uint32_t y = (uint32_t)(y0 + i);
    if (HIST) {  // (2 tau - 1 + 3K) dF1/dt + 3 cs^2 eta K d(grad mu)/dt of Eq. F2-1
      const float xx = fmaf(c.x_mu, mux, c.x_f1 * fx), xy = fmaf(c.x_mu, muy, c.x_f1 * fy);
      stb(rxh, xx, cst * 4u, y * rb);
      // the second plane ends at the buffer's end: an own lane's offset stays in range, the
      // others' lies beyond it whatever the plane
      stb(rxh, xy, cst * 4u, nodes * 4u + y * rb);
      if (!a.xfirst) {
        fx = fmaf(s1, tx, xx - hx[j2]);
        fy = fmaf(s1, ty, xy - hy[j2]);
      }
    }
    if (MODEL2) {
      fx = fmaf(c.k2, lane_dx(dv[j], dv[j2], dv[j1]) * R12, fx);
      fy = fmaf(c.k2, lane_dy(dv[j], dv[j1]) * R12, fy);
    }
    const float uu = VFIELD ? u[j2] : axc * u[j2], vv = VFIELD ? v[j2] : bxc * v[j2];
    lane_collide<MODEL, !VFIELD>(c, phi, mu[j2], uu, vv, axc, u[j2], fx, fy, s1, tx, g[j2]);
    finish_store<ST, false>(rdst, pitch, cst, y, (double)phi + (double)lo[j2], g[j2]);
  };

  fetch(in[0]);
  fetch(in[1]);
  fetch(in[2]);
  push(ic<0>{}, ic<0>{}, 0);
  push(ic<1>{}, ic<0>{}, 0);
  push(ic<2>{}, ic<1>{}, 0);
  push(ic<3>{}, ic<1>{}, 0);
#pragma unroll 1
  for (int i = 0; i < rows; i += 3) {
    push(ic<4>{}, ic<2>{}, i);
    if (i + 1 >= rows) break;
    push(ic<5>{}, ic<2>{}, i + 1);
    if (i + 2 >= rows) break;
    push(ic<6>{}, ic<2>{}, i + 2);
  }
}

#pragma clang fp contract(fast)

template <bool WALLS, int VMODE, int ST>
hipError_t pop_march_m(int model, const StepArgs& a, hipStream_t s) {
  const int total = a.mstrips * ((a.ny + a.mty - 1) / a.mty);
  const dim3 grid(((total + 3) / 4 + 7) / 8 * 8), block(256);
  switch (model) {
    case 1: hipLaunchKernelGGL((k_pop_march<WALLS, VMODE, 1, ST>), grid, block, 0, s, a, total); break;
    case 2: hipLaunchKernelGGL((k_pop_march<WALLS, VMODE, 2, ST>), grid, block, 0, s, a, total); break;
    case 3:
      if constexpr (ST == ST_F32) {
        hipLaunchKernelGGL((k_pop_march<WALLS, VMODE, 3, ST>), grid, block, 0, s, a, total);
        break;
      }
      return hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int ST>
hipError_t pop_march_t(bool walls, int vmode, int model, const StepArgs& a, hipStream_t s) {
  if (vmode == VEL_SEP)
    return walls ? pop_march_m<true, VEL_SEP, ST>(model, a, s) : pop_march_m<false, VEL_SEP, ST>(model, a, s);
  return walls ? pop_march_m<true, VEL_FIELD, ST>(model, a, s) : pop_march_m<false, VEL_FIELD, ST>(model, a, s);
}

}  // namespace

hipError_t launch_pop_march(bool walls, int vmode, int model, int storage, const StepArgs& a,
                            hipStream_t s) {
  if ((vmode != VEL_SEP && vmode != VEL_FIELD) || a.mty < 1 || a.mstrips != pop_march_strips(a.nx))
    return hipErrorInvalidValue;
  switch (storage) {
    case ST_F32: return pop_march_t<ST_F32>(walls, vmode, model, a, s);
    case ST_F16: return pop_march_t<ST_F16>(walls, vmode, model, a, s);
    case ST_BF16: return pop_march_t<ST_BF16>(walls, vmode, model, a, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace lbmch
