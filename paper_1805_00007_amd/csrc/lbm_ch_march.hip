// gfx950 kernels of several consecutive tau_g = 1 steps of the lattice Boltzmann
// Cahn-Hilliard solver (Zhang, Guo & Liang, arXiv:1805.00007), in the order-parameter
// form of the state.
//
// At tau_g = 1 the collision of Eq. LB keeps nothing of the pulled populations (g* =
// g^eq + S/2), so between two steps the state is the field m(x) = sum_i g_i alone: one
// FP64 value per node instead of nine populations.  Such a state is kept in both forms: m
// passes from step to step (16 bytes per node update instead of 72), and the last step of
// a call writes the populations as well.  Every step still forms the nine
// populations of a node exactly as the population kernels store them (collide_t1,
// stored_values: the float32 values with their mass closure, or the decoded 16-bit
// codes) and sums the pulled ones in the same order (sum9d), so the result is bitwise
// that of single steps.
#include "lbm_ch_device.h"
#include "lbm_ch_lanes.h"
#include "lbm_ch_stencil.h"

#include <type_traits>

namespace lbmch {
namespace {

#pragma clang fp contract(off)

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ double ldb64(rsrc_t r, uint32_t voff, uint32_t soff) {
  return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
}
__device__ __forceinline__ void stb64(rsrc_t r, double v, uint32_t voff, uint32_t soff) {
  __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, voff, soff, 0);
}
// One wave marches up TY rows of a strip of 64 lanes, one lane per column, with every
// rolling row in registers and the x neighbours from the adjacent lanes (DPP shifts): no
// LDS and no barrier, so waves never wait for each other.  Row r enters (pulled or
// loaded three rows ahead), then
//   row r    : phi, u, q = phi u, and the E - W, E + W of each                 (Eq. macroscopicg)
//   row r - 1: mu, D = div q, and theirs                                        (Eqs. mu, mark3)
//   row r - 2: F = F1 + F2, the nine populations as storage ST keeps them       (Eqs. t0-phiu, geq, liangFi, LB)
//   row r - 3: the sum of the populations pulled from rows r - 4 .. r - 2       (streaming)
// Across walls the stencils see mirrored rows (velocity odd) and populations that leave
// come back at their own node.  The outer lanes of a strip lose one column of validity per stage, M = 2 or (sums) 3 on
// each side, so a strip yields 58 columns.  A chunk of TY
// rows marches through 2M more.
//
// VALU-bound: about 150 vector instructions per wave and row (FP64 ones and lane shifts
// take 4.3-5 cycles, float32 ones 2.9); at 2048^2, two waves a SIMD, the VALU is busy 72 %
// of the launch, and HBM carries 73 MB of the 67 MB a step needs.  2048^2 float32: 26 us a
// step against 61.5 us for the population step's 302 MB; 4096^2 80 us against 216; half
// storage 2048^2 30 us against 44.  The step that writes the populations too takes 40 us at
// 2048^2 (5.1 TB/s); those stores keep the default cache policy, because a strip's rows are
// parts of lines that the neighbouring strip completes in L2.  A row holds no branch: phi
// that is NaN or Inf is reported after the march (a test in every row cost 2-3 % at 2048^2,
// 10 % of a batch).
//
// NT = 1 (writing float32 populations of lattices beyond the caches): strips of 48 columns,
// whose rows start and end at multiples of 64 bytes, and non-temporal stores.  Streamed past
// the caches in whole requests the populations leave the 256 MB cache to the sums: a call of
// one step at 2560^2 took 115 us, now 58; 4096^2 273 -> 146 (HBM 604 MB, 4.1 TB/s).  58 columns
// non-temporal 105 and 271 (parts of requests), 48 without 113 and 265.  NT = 2: stored
// velocities and recorded phi pass the caches too, where with them the sums would not fit
// (4096^2 stored velocity 277 -> 245, recorded 273 -> 179; where they fit it costs: 2500 x 2700
// 85 -> 114 and 66 -> 78).
template <bool WALLS, int VMODE, bool MODEL2, int ST, bool TO_G, bool REC, int NT = 0>
__device__ __forceinline__ void march_tile(const StepArgs& a, const int L) {
  constexpr bool VFIELD = VMODE == VEL_FIELD;
  constexpr int M = 3;
  static_assert(MARCH_OUT == 64 - 2 * M, "a strip and its margins are one wave");
  const int out = TO_G ? a.mout : MARCH_OUT;
  const Coef& c = a.c;
  const int nx = a.nx, ny = a.ny;
  const uint32_t nodes = (uint32_t)nx * ny, pitch = a.pitch;
  const uint32_t rb = (uint32_t)nx * 4u;
  const rsrc_t rdst = make_rsrc(a.mdst, nodes * 8u);
  const rsrc_t rsrc = make_rsrc(a.msrc, nodes * 8u);
  rsrc_t rgd, ru, rv, rrec;
  if (TO_G) rgd = make_rsrc(a.dst, pop_bytes(ST, pitch, ny));
  if (VFIELD) {
    ru = make_rsrc(a.ux, nodes * 4u);
    rv = make_rsrc(a.uy, nodes * 4u);
  }
  if (REC) rrec = make_rsrc(a.phi_rec, nodes * 4u);

  const int lane = threadIdx.x & 63;
  const int chunk = (int)((uint32_t)L / (uint32_t)a.mstrips);
  const int x0 = (L - chunk * a.mstrips) * out;
  const int y0 = chunk * a.mty;
  const int rows = min(a.mty, ny - y0);
  const int xl = x0 - M + lane;
  // by comparison (more than one on lattices narrower than a strip only): the two divisions of
  // a remainder before the first load were a good part of a short launch
  int x = xl < 0 ? xl + nx : xl;
  while (x >= nx) x -= nx;
  // columns this strip stores; the other lanes store at an offset beyond any buffer for
  // each element size (8, 4 and 2 bytes: 0xFFFFFE00, 0xFFFFFF00 and, against at most 1.2e9
  // bytes of 16-bit state, 0x7FFFFF80), which drops the store
  const bool own = lane >= M && lane < M + out && xl < nx;
  constexpr uint32_t OOB = 0x3FFFFFC0u;
  const uint32_t cst = own ? (uint32_t)x : OOB;
  constexpr int K0 = 2 * M;  // rows that enter before the first row is stored

  float axc = 0.f, bxc = 0.f;
  if (!VFIELD) {
    axc = a.ax[x];
    bxc = a.bx[x];
  }

  struct In {
    double m;
    float a, b, f;  // f: time factor of the row's velocity, odd across a wall
  };
  In in[3];
  // rows enter in order from y0 - M; past the last needed row the load repeats it (in cache)
  int lrow = WALLS || y0 >= M ? y0 - M : y0 - M + ny;
  int left = rows + 2 * M;
  auto fetch = [&](In& I) {
    int row = lrow;
    I.f = a.tf;
    if (WALLS) {
      float sg;
      row = row_of<true>(lrow, ny, sg);
      I.f = a.tf * sg;
    }
    I.m = ldb64(rsrc, (uint32_t)x * 8u, (uint32_t)row * 2u * rb);
    if (VFIELD) {
      auto ld = [&](rsrc_t r) {
        return NT == 2 ? ldb_nt(r, (uint32_t)x * 4u, (uint32_t)row * rb) : ldb(r, (uint32_t)x * 4u, (uint32_t)row * rb);
      };
      I.a = ld(ru);
      I.b = ld(rv);
    } else {
      I.a = ld_uniform(a.ay, row);
      I.b = ld_uniform(a.by, row);
    }
    if (--left > 0) lrow = !WALLS && lrow + 1 == ny ? 0 : lrow + 1;
  };

  double m[3];
  float ph[3], hph[3], u[3], v[3], qx[3], xqx[3], qy[3], hqy[3];
  float mu[3], xmu[3], hmu[3], dv[3], xd[3], hd[3];
  bool bad = false;  // a phi that is NaN or Inf (reported at the end: no branch in a row)
  double ac = 0.0, aw = 0.0, ae = 0.0, sc = 0.0, sw = 0.0, se = 0.0;

  auto row_x = [](float q) { return east(q) - west(q); };
  auto ddx = [&](float qm, float qp, float X0) { return row_dx(X0, row_x(qp + qm)); };

  // Row K enters slot K % 3; stage: the last of the four above that this row runs.  The sum
  // of row y0 + i is stored, and with TO_G the populations of the row after it.
  auto push = [&](auto K, auto STAGE, int i) {
    constexpr int j = decltype(K)::value % 3, j1 = (j + 2) % 3, j2 = (j + 1) % 3;
    constexpr int stage = decltype(STAGE)::value;
    In& I = in[j];
    const float phi_out = ph[j];  // phi of row r - 3
    // --- row r
    m[j] = I.m;
    ph[j] = (float)m[j];
    bad |= !__builtin_isfinite(ph[j]);
    if (VFIELD) {
      u[j] = I.f * I.a;
      v[j] = I.f * I.b;
    } else {
      u[j] = axc * (I.a * I.f);
      v[j] = bxc * (I.b * I.f);
    }
    fetch(I);
    hph[j] = east(ph[j]) + west(ph[j]);
    if (MODEL2) {
      qx[j] = ph[j] * u[j];
      qy[j] = ph[j] * v[j];
      xqx[j] = row_x(qx[j]);
      hqy[j] = east(qy[j]) + west(qy[j]);
    }
    if (stage < 1) return;
    // --- row r - 1
    mu[j1] = t1_mu(c, ph[j1], row_lap(ph[j2], ph[j1], ph[j], hph[j2], hph[j1], hph[j]));
    xmu[j1] = row_x(mu[j1]);
    hmu[j1] = east(mu[j1]) + west(mu[j1]);
    if (MODEL2) {
      dv[j1] = ddx(qx[j2], qx[j], xqx[j1]) + row_dy(qy[j2], qy[j], hqy[j2], hqy[j]);
      xd[j1] = row_x(dv[j1]);
      hd[j1] = east(dv[j1]) + west(dv[j1]);
    }
    if (stage < 2) return;
    // --- row r - 2: mu and D of rows r - 3, r - 2, r - 1 in slots j, j2, j1
    float fx, fy, dx = 0.f, dy = 0.f, g[9];
    if (MODEL2) {
      dx = ddx(dv[j], dv[j1], xd[j2]);
      dy = row_dy(dv[j], dv[j1], hd[j], hd[j1]);
    }
    t1_force<MODEL2>(c, ph[j2], ddx(mu[j], mu[j1], xmu[j2]), row_dy(mu[j], mu[j1], hmu[j], hmu[j1]), dx, dy, fx, fy);
    collide_t1(c, ph[j2], mu[j2], u[j2], v[j2], fx, fy, g);
    uint32_t h[9];
    if (TO_G && (stage == 3 || K == K0 - 1)) {
      const bool in = stage < 3 || i + 1 < rows;
      finish_store<ST, NT != 0>(rgd, pitch, in ? cst : OOB, (uint32_t)(in ? y0 + i + 1 : y0), m[j2], g);
    } else {
      stored_values<ST>(m[j2], g, h);
    }
    // --- row r - 3: the groups of sum9d, each summed at its source column
    double i4 = g[4], i8 = g[8], i7 = g[7];  // what row r - 3 receives from this row
    if (WALLS && y0 + i + 1 == ny) {  // half-way bounce-back: g_2, g_6, g_5 of row r - 3 itself
      i4 = sc;
      i8 = east(se);
      i7 = west(sw);
    }
    const double oc = ac + i4, ow = aw + i8, oe = ae + i7;
    if (WALLS && y0 + i + 1 == 0) {  // g_4, g_7, g_8 of this row in place of the row below
      sc = (double)g[4];
      sw = east((double)g[7]);
      se = west((double)g[8]);
    }
    ac = (double)g[0] + sc;
    aw = (double)g[1] + sw;
    ae = (double)g[3] + se;
    sc = (double)g[2];
    sw = (double)g[5];
    se = (double)g[6];
    if (stage < 3) return;
    if (REC && NT == 2) stb_nt(rrec, phi_out, cst * 4u, (uint32_t)(y0 + i) * rb);
    else if (REC) stb(rrec, phi_out, cst * 4u, (uint32_t)(y0 + i) * rb);
    stb64(rdst, oc + (west(ow) + east(oe)), cst * 8u, (uint32_t)(y0 + i) * 2u * rb);
  };

  fetch(in[0]);
  fetch(in[1]);
  fetch(in[2]);
  push(ic<0>{}, ic<0>{}, 0);
  push(ic<1>{}, ic<0>{}, 0);
  push(ic<2>{}, ic<1>{}, 0);
  push(ic<3>{}, ic<1>{}, 0);
  push(ic<4>{}, ic<2>{}, -2);
  push(ic<K0 - 1>{}, ic<2>{}, -1);
#pragma unroll 1
  for (int i = 0; i < rows; i += 3) {
    push(ic<K0>{}, ic<3>{}, i);
    if (i + 1 >= rows) break;
    push(ic<K0 + 1>{}, ic<3>{}, i + 1);
    if (i + 2 >= rows) break;
    push(ic<K0 + 2>{}, ic<3>{}, i + 2);
  }
  if (bad && a.nonfinite) *a.nonfinite = 1;
}

constexpr int MARCH_WAVES = 4;  // waves per workgroup (independent of each other)

template <bool WALLS, int VMODE, bool MODEL2, int ST, bool TO_G, bool REC, int NT>
__global__ void __launch_bounds__(64 * MARCH_WAVES) k_phi_march(const StepArgs a, const int total) {
  // workgroup w runs on XCD w % 8: give each XCD a band of neighbouring strips and chunks
  const int per = gridDim.x >> 3;
  const int w = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  const int L = w * MARCH_WAVES + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (L >= total) return;
  march_tile<WALLS, VMODE, MODEL2, ST, TO_G, REC, NT>(a, L);
}

// The marches of many lattices in one launch: wave L belongs to the instance whose range of
// waves holds it, found by every lane testing one start each; its arguments are read
// through the scalar cache (the tables are written before the launch).
template <int VMODE, bool MODEL2, bool TO_G>
__global__ void __launch_bounds__(64 * MARCH_WAVES) k_march_batch(const BatchArgs b) {
  const int per = gridDim.x >> 3;
  const int w = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  const int L = w * MARCH_WAVES + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (L >= b.total) return;
  int inst = -1;
  for (int i = 0; i < b.n; i += 64) {
    const int k = i + (int)(threadIdx.x & 63);
    inst += __popcll(__ballot(k < b.n && b.start[k] <= L));
  }
  typedef const __attribute__((address_space(4))) uint32_t* scalar_words;
  StepArgs a;
  static_assert(sizeof(StepArgs) % 4 == 0, "whole words");
  uint32_t words[sizeof(StepArgs) / 4];
  const scalar_words src = (scalar_words)(uintptr_t)(b.args + inst);
#pragma unroll
  for (int i = 0; i < (int)(sizeof(StepArgs) / 4); ++i) words[i] = src[i];
  __builtin_memcpy(&a, words, sizeof(StepArgs));
  if (b.parity) {
    a.dst = const_cast<void*>(a.src);
    const double* t = a.msrc;
    a.msrc = a.mdst;
    a.mdst = const_cast<double*>(t);
  }
  const int first = ((const __attribute__((address_space(4))) int*)(uintptr_t)b.start)[inst];
  march_tile<false, VMODE, MODEL2, ST_F32, TO_G, false>(a, L - first);
}

// Periodic index of i in -72 < i < n + 72.
__device__ __forceinline__ int wrap_near(int i, int n) {
  if (n >= 72) return i < 0 ? i + n : i >= n ? i - n : i;  // the same way for a whole wave
  return ((i % n) + n) % n;
}

// Several steps of one launch, for lattices too small to fill the chip with marches, where
// a step is a launch and a trip to memory: a workgroup of 16 waves loads m on a region of
// 64 columns x 16 K rows (a lane per column, K rows per wave) and takes T steps on it,
// the valid part shrinking by 3 nodes on every side in each; it yields 64 - 6 T columns
// x 16 K - 6 T rows.  x neighbours come from the adjacent lanes, y neighbours through LDS
// in four stages a step (those of march_tile), a barrier after each of the first three.
// Every value is formed as in march_tile, so results are bitwise the same.
template <int K, int VMODE, bool MODEL2, int ST, bool TO_G, bool REC>
__global__ void __launch_bounds__(1024) k_phi_block(const StepArgs a, const BlockSteps b) {
  constexpr bool VFIELD = VMODE == VEL_FIELD;
  constexpr int RR = 16 * K;
  __shared__ float s_ph[RR][64], s_hp[RR][64], s_qx[RR][64], s_qy[RR][64], s_hq[RR][64];
  __shared__ float s_mu[RR][64], s_hm[RR][64], s_d[RR][64], s_hd[RR][64];
  __shared__ float s_g[6][RR][64];  // g_2, g_5, g_6 and g_4, g_7, g_8
  const Coef& c = a.c;
  const int nx = a.nx, ny = a.ny, T = b.steps;
  const uint32_t nodes = (uint32_t)nx * ny, pitch = a.pitch;
  const uint32_t rb = (uint32_t)nx * 4u;
  const int outc = 64 - 6 * T, outr = RR - 6 * T;
  const int strips = (nx + outc - 1) / outc;
  const int chunk = (int)(blockIdx.x / (uint32_t)strips);
  const int x0 = ((int)blockIdx.x - chunk * strips) * outc, y0 = chunk * outr;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int xl = x0 - 3 * T + lane;
  const int x = wrap_near(xl, nx);
  const bool own = lane >= 3 * T && lane < 3 * T + outc && xl < nx;
  constexpr uint32_t OOB = 0x3FFFFFC0u;  // as in march_tile
  const uint32_t cst = own ? (uint32_t)x : OOB;
  const rsrc_t rsrc = make_rsrc(a.msrc, nodes * 8u), rdst = make_rsrc(a.mdst, nodes * 8u);
  const rsrc_t rgd = make_rsrc(a.dst, TO_G ? pop_bytes(ST, pitch, ny) : 0u);

  float axc = 0.f, bxc = 0.f, va[K], vb[K];
  double m[K];
  int yw[K];      // lattice row
  bool ownr[K];   // a row this workgroup stores
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int r = w * K + k, y = y0 - 3 * T + r;
    yw[k] = wrap_near(y, ny);
    ownr[k] = r >= 3 * T && r < 3 * T + outr && y < ny;
    m[k] = ldb64(rsrc, (uint32_t)x * 8u, (uint32_t)yw[k] * 2u * rb);
    if (VFIELD) {
      va[k] = a.ux[(uint32_t)yw[k] * nx + x];
      vb[k] = a.uy[(uint32_t)yw[k] * nx + x];
    } else {
      va[k] = ld_uniform(a.ay, yw[k]);
      vb[k] = ld_uniform(a.by, yw[k]);
    }
  }
  if (!VFIELD) {
    axc = a.ax[x];
    bxc = a.bx[x];
  }
  auto row_x = [](float q) { return east(q) - west(q); };
  auto ddx = [&](float qm, float q0, float qp) { return row_dx(row_x(q0), row_x(qp + qm)); };

#pragma unroll 1
  for (int s = 0; s < T; ++s) {
    const float tf = b.tf[s];
    const bool last = s == T - 1;
    float ph[K], u[K], v[K], hp[K], qx[K], mu[K], dv[K], g[K][9];
    // rows that stage q of step s still has to form
    auto active = [&](int r, int q) { return r >= 3 * s + q && r < RR - 3 * s - q; };
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int r = w * K + k;
      if (!active(r, 0)) continue;
      ph[k] = (float)m[k];
      if (__builtin_expect(!__builtin_isfinite(ph[k]), 0) && own && ownr[k] && a.nonfinite)
        *a.nonfinite = 1;
      u[k] = VFIELD ? tf * va[k] : axc * (va[k] * tf);
      v[k] = VFIELD ? tf * vb[k] : bxc * (vb[k] * tf);
      hp[k] = east(ph[k]) + west(ph[k]);
      s_ph[r][lane] = ph[k];
      s_hp[r][lane] = hp[k];
      if (MODEL2) {
        qx[k] = ph[k] * u[k];
        const float qy = ph[k] * v[k];
        s_qx[r][lane] = qx[k];
        s_qy[r][lane] = qy;
        s_hq[r][lane] = east(qy) + west(qy);
      }
      if (REC && ownr[k]) {
        const rsrc_t rrec = make_rsrc(a.phi_rec + (size_t)s * nodes, nodes * 4u);
        stb(rrec, ph[k], cst * 4u, (uint32_t)yw[k] * rb);
      }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int r = w * K + k;
      if (!active(r, 1)) continue;
      mu[k] = t1_mu(c, ph[k], row_lap(s_ph[r - 1][lane], ph[k], s_ph[r + 1][lane], s_hp[r - 1][lane],
                                      hp[k], s_hp[r + 1][lane]));
      s_mu[r][lane] = mu[k];
      s_hm[r][lane] = east(mu[k]) + west(mu[k]);
      if (MODEL2) {
        dv[k] = ddx(s_qx[r - 1][lane], qx[k], s_qx[r + 1][lane]) +
                row_dy(s_qy[r - 1][lane], s_qy[r + 1][lane], s_hq[r - 1][lane], s_hq[r + 1][lane]);
        s_d[r][lane] = dv[k];
        s_hd[r][lane] = east(dv[k]) + west(dv[k]);
      }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int r = w * K + k;
      if (!active(r, 2)) continue;
      float dx = 0.f, dy = 0.f, fx, fy;
      const float mm = s_mu[r - 1][lane], mp = s_mu[r + 1][lane];
      if (MODEL2) {
        const float dm = s_d[r - 1][lane], dp = s_d[r + 1][lane];
        dx = ddx(dm, dv[k], dp);
        dy = row_dy(dm, dp, s_hd[r - 1][lane], s_hd[r + 1][lane]);
      }
      t1_force<MODEL2>(c, ph[k], ddx(mm, mu[k], mp), row_dy(mm, mp, s_hm[r - 1][lane], s_hm[r + 1][lane]),
                       dx, dy, fx, fy);
      collide_t1(c, ph[k], mu[k], u[k], v[k], fx, fy, g[k]);
      if (TO_G && last && ownr[k]) {
        finish_store<ST, false>(rgd, pitch, cst, (uint32_t)yw[k], m[k], g[k]);
      } else {
        uint32_t h[9];
        stored_values<ST>(m[k], g[k], h);
      }
      s_g[0][r][lane] = g[k][2];
      s_g[1][r][lane] = g[k][5];
      s_g[2][r][lane] = g[k][6];
      s_g[3][r][lane] = g[k][4];
      s_g[4][r][lane] = g[k][7];
      s_g[5][r][lane] = g[k][8];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int r = w * K + k;
      if (!active(r, 3)) continue;
      const double oc = ((double)g[k][0] + (double)s_g[0][r - 1][lane]) + (double)s_g[3][r + 1][lane];
      const double ow = ((double)g[k][1] + (double)s_g[1][r - 1][lane]) + (double)s_g[5][r + 1][lane];
      const double oe = ((double)g[k][3] + (double)s_g[2][r - 1][lane]) + (double)s_g[4][r + 1][lane];
      m[k] = oc + (west(ow) + east(oe));
    }
  }
#pragma unroll
  for (int k = 0; k < K; ++k)
    if (ownr[k]) stb64(rdst, m[k], cst * 8u, (uint32_t)yw[k] * 2u * rb);
}
// One step, populations written too, of a lattice whose tiles are one round of the CUs: a
// workgroup of 16 waves takes a tile of 64 columns x 16 rows, a wave its row.  Margin nodes
// (phi on 3 around the tile, mu and D on 2, populations on 1) are a second, partial pass of
// each stage, all neighbours are in LDS, with a barrier after each stage.  At these sizes a step
// is bound by the latency of a launch and by vector instructions: the tile forms 1.16
// populations per node where a march of 5 rows forms 1.55, 512^2 7.0 -> 6.2 us, half storage
// 7.0 -> 5.9.  Every value is formed as in march_tile, so results are bitwise the same.
template <int VMODE, bool MODEL2, int ST, bool REC>
__global__ void __launch_bounds__(1024) k_phi_single(const StepArgs a) {
  constexpr bool VFIELD = VMODE == VEL_FIELD;
  constexpr int TW = 64, TH = 16;
  struct Fields {
    float ph[TH + 6][TW + 6], qx[TH + 6][TW + 6], qy[TH + 6][TW + 6];
    float u[TH + 2][TW + 2], v[TH + 2][TW + 2];
    double m[TH + 2][TW + 2];
    float mu[TH + 4][TW + 4], d[TH + 4][TW + 4];
  };
  union Shared {
    Fields f;
    float g[8][TH + 2][TW + 2];  // g_1 .. g_8, once the fields are read
  };
  __shared__ Shared s;
  Fields& F = s.f;
  const Coef& c = a.c;
  const int nx = a.nx, ny = a.ny;
  const uint32_t nodes = (uint32_t)nx * ny;
  const uint32_t rb = (uint32_t)nx * 4u;
  const int strips = (nx + TW - 1) / TW;
  // one band of tiles per XCD (the grid is a multiple of 8; the last tiles may be none)
  const int L = (int)((blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3));
  const int chunk = (int)((uint32_t)L / (uint32_t)strips);
  const int x0 = (L - chunk * strips) * TW, y0 = chunk * TH;
  if (y0 >= ny) return;
  const int t = threadIdx.x, lane = t & 63;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const rsrc_t rsrc = make_rsrc(a.msrc, nodes * 8u), rdst = make_rsrc(a.mdst, nodes * 8u);
  const rsrc_t rgd = make_rsrc(a.dst, pop_bytes(ST, a.pitch, ny));
  const int x = wrap_near(x0 + lane, nx), y = wrap_near(y0 + w, ny);
  const bool own = x0 + lane < nx && y0 + w < ny;
  constexpr uint32_t OOB = 0x3FFFFFC0u;  // as in march_tile
  const uint32_t cst = own ? (uint32_t)x : OOB;

  // Margin node e of a region with margin M around the tile: its row and column in it.
  auto margin = [&](auto MM, int e, int& r, int& q) {
    constexpr int M = decltype(MM)::value, RW = TW + 2 * M, ROWS = M * RW;
    if (e < 2 * ROWS) {
      const int k = e < ROWS ? e : e - ROWS;
      r = k / RW + (e < ROWS ? 0 : M + TH);
      q = k % RW;
    } else {
      const int k = e - 2 * ROWS;
      r = M + k / (2 * M);
      q = k % (2 * M);
      q += q < M ? 0 : TW;
    }
  };
  constexpr int N3 = 2 * 3 * (TW + 6) + 6 * TH, N2 = 2 * 2 * (TW + 4) + 4 * TH, N1 = 2 * (TW + 2) + 2 * TH;

  // loads of the tile's node and of a margin node
  double m = ldb64(rsrc, (uint32_t)x * 8u, (uint32_t)y * 2u * rb), mm = 0.0;
  float ua, va, ub = 0.f, vb = 0.f, ax = 0.f, bx = 0.f, axm = 0.f, bxm = 0.f;
  int r3 = 0, q3 = 0;
  if (VFIELD) {
    ua = a.ux[(uint32_t)y * nx + x];
    va = a.uy[(uint32_t)y * nx + x];
  } else {
    ua = ld_uniform(a.ay, y);
    va = ld_uniform(a.by, y);
    ax = a.ax[x];
    bx = a.bx[x];
  }
  if (t < N3) {
    margin(ic<3>{}, t, r3, q3);
    const uint32_t xm = wrap_near(x0 - 3 + q3, nx), ym = wrap_near(y0 - 3 + r3, ny);
    mm = ldb64(rsrc, (ym * nx + xm) * 8u, 0);
    if (VFIELD) {
      ub = a.ux[ym * nx + xm];
      vb = a.uy[ym * nx + xm];
    } else {
      ub = a.ay[ym];
      vb = a.by[ym];
      axm = a.ax[xm];
      bxm = a.bx[xm];
    }
  }

  // phi, u and q = phi u on the tile and 3 nodes around it
  auto fields = [&](int r, int q, double mi, float ui, float vi) {
    const float ph = (float)mi;
    F.ph[r][q] = ph;
    if (MODEL2) {
      F.qx[r][q] = ph * ui;
      F.qy[r][q] = ph * vi;
    }
  };
  const float u = VFIELD ? a.tf * ua : ax * (ua * a.tf), v = VFIELD ? a.tf * va : bx * (va * a.tf);
  const float ph = (float)m;
  if (__builtin_expect(!__builtin_isfinite(ph), 0) && own && a.nonfinite) *a.nonfinite = 1;
  fields(w + 3, lane + 3, m, u, v);
  if (t < N3) {
    const float um = VFIELD ? a.tf * ub : axm * (ub * a.tf), vm = VFIELD ? a.tf * vb : bxm * (vb * a.tf);
    fields(r3, q3, mm, um, vm);
    if (r3 >= 2 && r3 < TH + 4 && q3 >= 2 && q3 < TW + 4) {  // for the populations there
      F.u[r3 - 2][q3 - 2] = um;
      F.v[r3 - 2][q3 - 2] = vm;
      F.m[r3 - 2][q3 - 2] = mm;
    }
  }
  if (REC) stb(make_rsrc(a.phi_rec, nodes * 4u), ph, cst * 4u, (uint32_t)y * rb);
  __syncthreads();

  // mu and D = div q on 2 nodes around it; r, q in the region of phi
  auto potential = [&](int r, int q, float p) {
    const float mu = t1_mu(c, p, t1_lap(F.ph[r - 1], F.ph[r], F.ph[r + 1], q));
    F.mu[r - 1][q - 1] = mu;
    if (MODEL2)
      F.d[r - 1][q - 1] = t1_dx(F.qx[r - 1], F.qx[r], F.qx[r + 1], q) + t1_dy(F.qy[r - 1], F.qy[r], F.qy[r + 1], q);
    return mu;
  };
  const float mu = potential(w + 3, lane + 3, ph);
  if (t < N2) {
    int r, q;
    margin(ic<2>{}, t, r, q);
    potential(r + 1, q + 1, F.ph[r + 1][q + 1]);
  }
  __syncthreads();

  // the populations on one node around it; r, q in the region of mu
  auto collide = [&](int r, int q, float p, float mui, float ui, float vi, float g[9]) {
    float fx, fy, dx = 0.f, dy = 0.f;
    if (MODEL2) {
      dx = t1_dx(F.d[r - 1], F.d[r], F.d[r + 1], q);
      dy = t1_dy(F.d[r - 1], F.d[r], F.d[r + 1], q);
    }
    t1_force<MODEL2>(c, p, t1_dx(F.mu[r - 1], F.mu[r], F.mu[r + 1], q),
                     t1_dy(F.mu[r - 1], F.mu[r], F.mu[r + 1], q), dx, dy, fx, fy);
    collide_t1(c, p, mui, ui, vi, fx, fy, g);
  };
  float g[9], gm[9];
  collide(w + 2, lane + 2, ph, mu, u, v, g);
  finish_store<ST, false>(rgd, a.pitch, cst, (uint32_t)y, m, g);
  int r1 = 0, q1 = 0;
  if (t < N1) {
    margin(ic<1>{}, t, r1, q1);
    uint32_t h[9];
    collide(r1 + 1, q1 + 1, F.ph[r1 + 2][q1 + 2], F.mu[r1 + 1][q1 + 1], F.u[r1][q1], F.v[r1][q1], gm);
    stored_values<ST>(F.m[r1][q1], gm, h);
  }
  __syncthreads();  // the fields are read: their place takes the populations
#pragma unroll
  for (int i = 1; i < 9; ++i) s.g[i - 1][w + 1][lane + 1] = g[i];
  if (t < N1) {
#pragma unroll
    for (int i = 1; i < 9; ++i) s.g[i - 1][r1][q1] = gm[i];
  }
  __syncthreads();

  // the sum of the populations pulled to the tile's node (sum9d)
  auto G = [&](int i, int dr, int dq) { return (double)s.g[i - 1][w + 1 + dr][lane + 1 + dq]; };
  const double oc = ((double)g[0] + G(2, -1, 0)) + G(4, 1, 0);
  const double ow = (G(1, 0, -1) + G(5, -1, -1)) + G(8, 1, -1);
  const double oe = (G(3, 0, 1) + G(6, -1, 1)) + G(7, 1, 1);
  stb64(rdst, oc + (ow + oe), cst * 8u, (uint32_t)y * 2u * rb);
}
#pragma clang fp contract(fast)

// Workgroups for `total` waves, a multiple of 8 (one band per XCD).
int march_grid(int total) { return ((total + MARCH_WAVES - 1) / MARCH_WAVES + 7) / 8 * 8; }

template <int ST, bool TO_G, int NT>
hipError_t march_f(bool walls, int vmode, bool model2, const StepArgs& a, hipStream_t s) {
  const int total = a.mstrips * ((a.ny + a.mty - 1) / a.mty);
  const dim3 grid(march_grid(total)), block(64 * MARCH_WAVES);
  const bool rec = a.phi_rec != nullptr;
  if (walls && rec) return hipErrorInvalidValue;
#define LBM_MARCH(W, V, M2, R) \
  hipLaunchKernelGGL((k_phi_march<W, V, M2, ST, TO_G, R, NT>), grid, block, 0, s, a, total)
#define LBM_MARCH_FORM(V, M2)                         \
  if (walls) LBM_MARCH(true, V, M2, false);           \
  else if (rec) LBM_MARCH(false, V, M2, true);        \
  else LBM_MARCH(false, V, M2, false)
  if (vmode == VEL_SEP) {
    if (model2) { LBM_MARCH_FORM(VEL_SEP, true); } else { LBM_MARCH_FORM(VEL_SEP, false); }
  } else {
    if (model2) { LBM_MARCH_FORM(VEL_FIELD, true); } else { LBM_MARCH_FORM(VEL_FIELD, false); }
  }
#undef LBM_MARCH_FORM
#undef LBM_MARCH
  return hipGetLastError();
}

template <int K, int ST, bool TO_G>
hipError_t block_f(int vmode, bool model2, const StepArgs& a, const BlockSteps& b, hipStream_t s) {
  const int outc = 64 - 6 * b.steps, outr = 16 * K - 6 * b.steps;
  if (b.steps < 1 || b.steps > BLOCK_STEPS || outr < 1) return hipErrorInvalidValue;
  const int grid = ((a.nx + outc - 1) / outc) * ((a.ny + outr - 1) / outr);
  const bool rec = a.phi_rec != nullptr;
#define LBM_BLOCK(V, M2, R) \
  hipLaunchKernelGGL((k_phi_block<K, V, M2, ST, TO_G, R>), dim3(grid), dim3(1024), 0, s, a, b)
  if (vmode == VEL_SEP) {
    if (model2) { if (rec) LBM_BLOCK(VEL_SEP, true, true); else LBM_BLOCK(VEL_SEP, true, false); }
    else { if (rec) LBM_BLOCK(VEL_SEP, false, true); else LBM_BLOCK(VEL_SEP, false, false); }
  } else {
    if (model2) { if (rec) LBM_BLOCK(VEL_FIELD, true, true); else LBM_BLOCK(VEL_FIELD, true, false); }
    else { if (rec) LBM_BLOCK(VEL_FIELD, false, true); else LBM_BLOCK(VEL_FIELD, false, false); }
  }
#undef LBM_BLOCK
  return hipGetLastError();
}

template <int K, int ST>
hipError_t block_t(int vmode, bool model2, bool to_g, const StepArgs& a, const BlockSteps& b,
                   hipStream_t s) {
  return to_g ? block_f<K, ST, true>(vmode, model2, a, b, s) : block_f<K, ST, false>(vmode, model2, a, b, s);
}

template <int ST>
hipError_t single_t(int vmode, bool model2, const StepArgs& a, hipStream_t s) {
  const dim3 grid((((a.nx + 63) / 64) * ((a.ny + 15) / 16) + 7) / 8 * 8), block(1024);
  const bool rec = a.phi_rec != nullptr;
#define LBM_SINGLE(V, M2)                                                                 \
  if (rec) hipLaunchKernelGGL((k_phi_single<V, M2, ST, true>), grid, block, 0, s, a);     \
  else hipLaunchKernelGGL((k_phi_single<V, M2, ST, false>), grid, block, 0, s, a)
  if (vmode == VEL_SEP) {
    if (model2) { LBM_SINGLE(VEL_SEP, true); } else { LBM_SINGLE(VEL_SEP, false); }
  } else {
    if (model2) { LBM_SINGLE(VEL_FIELD, true); } else { LBM_SINGLE(VEL_FIELD, false); }
  }
#undef LBM_SINGLE
  return hipGetLastError();
}

template <int ST>
hipError_t march_t(bool walls, int vmode, bool model2, bool to_g, const StepArgs& a, hipStream_t s) {
  return to_g ? march_f<ST, true, 0>(walls, vmode, model2, a, s)
              : march_f<ST, false, 0>(walls, vmode, model2, a, s);
}

}  // namespace

bool march_ok(int vmode, int model, bool t1) {
  return t1 && (vmode == VEL_SEP || vmode == VEL_FIELD) && (model == 1 || model == 2);
}

hipError_t launch_phi_march(bool walls, int vmode, int model, int storage, bool to_g, int nt,
                            const StepArgs& a, hipStream_t s) {
  if (!march_ok(vmode, model, true) || a.mty < 1 ||
      a.mout < 1 || a.mout > MARCH_OUT || a.mstrips != march_strips(a.nx, a.mout))
    return hipErrorInvalidValue;
  if (nt) {
    if (!to_g || storage != ST_F32) return hipErrorInvalidValue;
    return nt == 2 ? march_f<ST_F32, true, 2>(walls, vmode, model == 2, a, s)
                   : march_f<ST_F32, true, 1>(walls, vmode, model == 2, a, s);
  }
  switch (storage) {
    case ST_F32: return march_t<ST_F32>(walls, vmode, model == 2, to_g, a, s);
    case ST_F16: return march_t<ST_F16>(walls, vmode, model == 2, to_g, a, s);
    case ST_BF16: return march_t<ST_BF16>(walls, vmode, model == 2, to_g, a, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_phi_block(int rows, int vmode, int model, int storage, bool to_g,
                            const StepArgs& a, const BlockSteps& b, hipStream_t s) {
  if (!march_ok(vmode, model, true) || (rows != 16 && rows != 32)) return hipErrorInvalidValue;
#define LBM_BLOCK_ST(ST)                                                        \
  return rows == 16 ? block_t<1, ST>(vmode, model == 2, to_g, a, b, s)          \
                    : block_t<2, ST>(vmode, model == 2, to_g, a, b, s)
  switch (storage) {
    case ST_F32: LBM_BLOCK_ST(ST_F32);
    case ST_F16: LBM_BLOCK_ST(ST_F16);
    case ST_BF16: LBM_BLOCK_ST(ST_BF16);
    default: return hipErrorInvalidValue;
  }
#undef LBM_BLOCK_ST
}

hipError_t launch_phi_single(int vmode, int model, int storage, const StepArgs& a, hipStream_t s) {
  if (!march_ok(vmode, model, true)) return hipErrorInvalidValue;
  switch (storage) {
    case ST_F32: return single_t<ST_F32>(vmode, model == 2, a, s);
    case ST_F16: return single_t<ST_F16>(vmode, model == 2, a, s);
    case ST_BF16: return single_t<ST_BF16>(vmode, model == 2, a, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_march_batch(int vmode, bool model2, bool to_g, const BatchArgs& b, hipStream_t s) {
  if (b.n <= 0 || b.total <= 0) return hipErrorInvalidValue;
  const dim3 grid(march_grid(b.total)), block(64 * MARCH_WAVES);
#define LBM_MB(V, M2)                                                                \
  if (to_g) hipLaunchKernelGGL((k_march_batch<V, M2, true>), grid, block, 0, s, b);  \
  else hipLaunchKernelGGL((k_march_batch<V, M2, false>), grid, block, 0, s, b)
  if (vmode == VEL_SEP) {
    if (model2) { LBM_MB(VEL_SEP, true); } else { LBM_MB(VEL_SEP, false); }
  } else {
    if (model2) { LBM_MB(VEL_FIELD, true); } else { LBM_MB(VEL_FIELD, false); }
  }
#undef LBM_MB
  return hipGetLastError();
}

}  // namespace lbmch
