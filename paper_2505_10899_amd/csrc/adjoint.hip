// Discrete adjoint of the FP64 coupled D2Q9 step (hand-written reverse sweep).
//
// The objective J is a function of the phase field after the last step, linearised as
// J = sum over labels of s0 sum(phi) + s1 . sum(phi d) + s2 : sum(phi d d^T).  The adjoint
// state of the populations pulled at step t is kept in two parts:
//     dJ/dg_i(t)(x) = lg_i(x) + lphi(x),   dJ/df_i(t)(x) = lf_i(x),   dJ/dJprev(t)(x) = lJ(x)
// where lphi is the adjoint of phi(x) = sum_i g_i(x) (Eq. 35), shared by the nine g_i.
// One backward step t+1 -> t is one launch, k_adj_tile, a workgroup per tile of nodes:
//   - phi and psi of step t on the tile and its halo, pulled from the stored state into LDS;
//   - lphi of step t + 1 on the same nodes, by the transposed stencils (behind a wall, the
//     ghost row is the wetting ghost of the edge row: its slope joins the chain) and
//     dpsi/dphi from Eq. 37, from what step t + 1 left in `aux`: the adjoints of what its
//     nodes read through stencils, staged in LDS with a halo of two nodes;
//   - per node x: gather the adjoint of the node's post-collision populations (transpose
//     of the pull streaming with half-way bounce-back and the moving-wall term), recompute
//     the node's forward step, and run it in reverse.  Writes lg, lf, lJ and aux of step t
//     (own phi, the Laplacian and gradient of phi and the gradient of psi, Eqs. 39-40, and
//     phi itself).  Accumulates dJ/dsigma and dJ/dM per workgroup.
// As three kernels (phi and psi, the local reverse, the stencils) a step of 512 x 256 took
// 29 us and two more launches, a whole step with its recomputed forward one and the copies
// of J 43; as one 20 and 30.  Its bytes (376 read and 216 written a node) take 13 us at the
// copy rate; a 128 x 64 grid, whose bytes take under 1 and whose 64 workgroups leave most CUs
// idle, needs 12: the chain of a node's reverse, some 1500 FP64 operations.  On 512 x 256 that
// chain is hidden behind two waves per SIMD only, all that the grid has (registers allow 3).
// Away from the interface psi saturates and |grad psi| falls to rounding level; the
// derivative of the unit normal there has a gain of order lambda / |grad psi| per step
// and grows without bound, so the normal is differentiated only where
// |grad psi| >= normal_tau (psi is a signed distance, |grad psi| = 1, across the
// interface); normal_tau = 0 gives the exact derivative of the discrete map.
// The initial state (g = g_eq(phi0), f = f_eq(0, rho(phi0), u0), Jprev = phi0 u0) has its
// own reverse pair giving dJ/dphi0.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "adjoint.hpp"

namespace vclb {

namespace {

using R = double;
using DC = DevCase<D2Q9, StoreF64>;

__device__ __forceinline__ int xwrap(int x, int nx) { return x < 0 ? x + nx : (x >= nx ? x - nx : x); }

// row of the neighbour y + dy for the phi/psi stencils: wrap, or the edge row itself
// behind a wall (mirrored ghost)
__device__ __forceinline__ int stencil_row(int y, int dy, int ny, bool wall) {
  const int v = y + dy;
  if (v < 0) return wall ? 0 : v + ny;
  if (v >= ny) return wall ? ny - 1 : v - ny;
  return v;
}

// v = M^T y with the integer matrix of Eq. 24
__device__ __forceinline__ void moments_T(const R (&y)[9], R (&v)[9]) {
#pragma unroll
  for (int i = 0; i < 9; ++i) {
    R acc = R(0);
#pragma unroll
    for (int k = 0; k < 9; ++k) {
      const int m = D2Q9::M[k][i];
      if (m == 1) acc += y[k];
      else if (m == -1) acc -= y[k];
      else if (m != 0) acc += R(m) * y[k];
    }
    v[i] = acc;
  }
}

// d(mu)/d(sigma) at fixed phi: mu = 4 beta c(phi) - kappa lap, beta and kappa linear in sigma
__device__ __forceinline__ R dmu_dsigma(const AdjArgs& a, R cub, R lap) {
  return a.beta4_per_sigma * cub - a.kappa_per_sigma * lap;
}

// per-workgroup accumulation of (dJ/dsigma, dJ/dM) into this workgroup's own slot
__device__ __forceinline__ void add_params(const AdjArgs& a, int slot, double sig, double mob) {
  __shared__ double red[16 * 2];
  const double v[2] = {sig, mob};
  const double s = block_sum_fields<2>(v, 2, red);
  if (threadIdx.x < 2) a.param_part[threadIdx.x * a.part_slots + slot] += s;
}

// sum over the stencil readers m of node (x, y), m + c_i = (x, y): fn(i, m, side), with
// side 0 for a reader of the node itself and -1 / +1 for a reader of the ghost row behind
// the bottom / top wall, which holds the wetting ghost of this edge node (its mirror for
// a neutral wall)
template <class Fn>
__device__ __forceinline__ void stencil_readers(const DC& c, int x, int y, Fn&& fn) {
  const int nx = c.nx, ny = c.ny;
#pragma unroll
  for (int i = 1; i < 9; ++i) {
    const int xs = xwrap(x - D2Q9::cx[i], nx);
    const int ys = y - D2Q9::cy[i];
    if (ys >= 0 && ys < ny) fn(i, xs + long(nx) * ys, 0);
    else if (!c.wall) fn(i, xs + long(nx) * (ys < 0 ? ys + ny : ys - ny), 0);
    if (c.wall && y == 0 && D2Q9::cy[i] < 0) fn(i, xs + long(nx) * y, -1);
    if (c.wall && y == ny - 1 && D2Q9::cy[i] > 0) fn(i, xs + long(nx) * y, 1);
  }
}

// the wetting-ghost coefficient of the wall on this side: phi_g = phi_e + w phi_e (1 - phi_e)
__device__ __forceinline__ R wet_coef(const DC& c, int side) { return side < 0 ? c.np.wet_lo : c.np.wet_hi; }

// d(phi_g)/d(phi_e) of the wetting ghost
__device__ __forceinline__ R wet_slope(R w, R phi) { return R(1) + w * (R(1) - R(2) * phi); }

// dpsi/dphi of Eq. 37 on the clipped range (zero where the clip holds psi fixed)
__device__ __forceinline__ R dpsi_dphi(const DC& c, R phi) {
  if (!(phi >= R(0) && phi <= R(1))) return R(0);
  const R aa = phi + c.np.xi, bb = (R(1) - phi) + c.np.xi;
  return c.np.W4 * (R(1) / aa + R(1) / bb);
}

}  // namespace

// -------------------------------------------------------------------------- seed
// dJ/dphi(x) at the final step from the per-label moment weights; lg = lf = lJ = 0.
__global__ void __launch_bounds__(256) k_adj_seed(DC c, AdjArgs a) {
  const long n = blockIdx.x * long(blockDim.x) + threadIdx.x;
  if (n >= c.n) return;
  const int x = int(n % c.nx), y = int(n / c.nx);
  double d[kMaxLabels][2];
#pragma unroll
  for (int k = 0; k < kMaxLabels; ++k) {
    d[k][0] = min_image(double(x) - c.cen[k][0], c.nx, true);
    d[k][1] = min_image(double(y) - c.cen[k][1], c.ny, !c.wall);
  }
  int lab = 0;
  if (c.nl > 1 && d[1][0] * d[1][0] + d[1][1] * d[1][1] < d[0][0] * d[0][0] + d[0][1] * d[0][1]) lab = 1;
  const double* s = a.seed + lab * kSeedFields;
  const double dx = d[lab][0], dy = d[lab][1];
  // moments: sum, d (x, y, z), d d^T (xx, yy, zz, xy, xz, yz); z terms vanish in 2D
  a.lphi[n] = s[0] + s[1] * dx + s[2] * dy + s[4] * dx * dx + s[5] * dy * dy + s[7] * dx * dy;
#pragma unroll
  for (int i = 0; i < 9; ++i) {
    a.lg_out[long(i) * c.n + n] = 0.0;
    a.lf_out[long(i) * c.n + n] = 0.0;
  }
  a.lJ_out[n] = 0.0;
  a.lJ_out[c.n + n] = 0.0;
}

// -------------------------------------------------------------------------- local reverse
// Reverse of one node's step.  q, s: phi and psi at x + c_i; g, f, Jp: the stored state's
// pulled populations and previous phi u; lgs, lfs: adjoints of the node's post-collision
// populations; lJn: adjoint of this step's phi u as the next step's Jprev; lrho: the
// moving walls' share of the adjoint of rho.  Writes lg, lf, lJ and aux of node n.
__device__ __forceinline__ void adj_node(const DC& c, const AdjArgs& a, long n, const R (&q)[9], const R (&s)[9],
                                         const R (&g)[9], const R (&f)[9], const R (&Jp)[2], const R (&lgs)[9],
                                         const R (&lfs)[9], const R (&lJn)[2], R lrho, double& acc_sig,
                                         double& acc_mob) {
  const auto& p = c.np;
  const R phi = q[0];
  const R rho = p.rho_l + phi * p.drho;
  const bool inside = phi >= R(0) && phi <= R(1);
  const R pc = clamp01(phi);
  const R aa = pc + p.xi, bb = (R(1) - pc) + p.xi;
  const R An = p.An4 * aa * bb;                       // a + b = 1 + 2 xi
  const R dAn = inside ? p.An4 * (bb - aa) : R(0);
  const R gpx = R(1.0 / 3.0) * (q[1] - q[3]) + R(1.0 / 12.0) * ((q[5] - q[7]) + (q[8] - q[6]));
  const R gpy = R(1.0 / 3.0) * (q[2] - q[4]) + R(1.0 / 12.0) * ((q[5] - q[7]) + (q[6] - q[8]));
  const R lap = R(2.0 / 3.0) * (((q[1] + q[3]) + (q[2] + q[4])) - R(4) * q[0]) +
                R(1.0 / 6.0) * (((q[5] + q[7]) + (q[6] + q[8])) - R(4) * q[0]);
  const R gsx = R(1.0 / 3.0) * (s[1] - s[3]) + R(1.0 / 12.0) * ((s[5] - s[7]) + (s[8] - s[6]));
  const R gsy = R(1.0 / 3.0) * (s[2] - s[4]) + R(1.0 / 12.0) * ((s[5] - s[7]) + (s[6] - s[8]));
  const R cub = phi * (phi - R(1)) * (phi - R(0.5));
  const R mu = p.beta4 * cub - p.kappa * lap;
  const R Fx = mu * gpx, Fy = mu * gpy;
  const R grx = p.drho * gpx, gry = p.drho * gpy;
  R fm[9];
  d2q9_moments<R>(f, fm);
  const R irho = R(1) / rho;
  const R ux = (fm[3] + R(0.5) * Fx) * irho, uy = (fm[5] + R(0.5) * Fy) * irho;
  const R uu = ux * ux + uy * uy;
  const R Jx = phi * ux, Jy = phi * uy;
  const R ir = rsqrt_of(gsx * gsx + gsy * gsy + p.eps2);
  const R nxn = gsx * ir, nyn = gsy * ir;
  const R Vx = R(3) * (Jx - Jp[0]) + An * nxn, Vy = R(3) * (Jy - Jp[1]) + An * nyn;
  R gm[9];
  d2q9_moments<R>(g, gm);
  const R H = mu + p.lam * phi;
  const R geq[9] = {phi, R(-4) * phi + R(2) * H, R(4) * phi - R(3) * H, Jx, -Jx, Jy, -Jy, R(0), R(0)};
  const R Gx = Vx * R(1.0 / 3.0), Gy = Vy * R(1.0 / 3.0);
  const R gsrc[9] = {R(0), R(0), R(0), Gx, -Gx, Gy, -Gy, R(0), R(0)};

  // ---- f collision (Eq. 25) in reverse: f* = M^-1 [(1 - s) m + s m_eq + (1 - s/2) m_F],
  // M^-T = diag(1/|M_k|^2) M
  // With unequal viscosities the stress rows relax at the node's own rate
  // s = 1 / (1/2 + 3 mu / rho) (Eq. 27), mu = mu_l + phi dmu: their adjoint also reaches
  // phi and rho through s, with dm*_k/ds = m_eq,k - m_k - m_F,k / 2.
  const bool visc = c.visc != 0;
  const R s_st = visc ? stress_rate<D2Q9, R>(p, phi, irho) : R(0);
  const R meq_st[2] = {rho * (ux * ux - uy * uy), rho * ux * uy};
  const R mF_st[2] = {R(2.0 / 3.0) * (ux * grx - uy * gry), R(1.0 / 3.0) * (ux * gry + uy * grx)};
  R ls_st = R(0);   // adjoint of s
  R lmf[9];
  d2q9_moments<R>(lfs, lmf);
  R lfm[9], leqf[9], lsrcf[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    const R lms = lmf[k] * R(1.0 / double(row_norm<D2Q9>(k)));
    const bool st = visc && D2Q9::f_stress_row[k];
    const R sk = st ? s_st : p.sfr[k];
    lfm[k] = (R(1) - sk) * lms;
    leqf[k] = sk * lms;
    lsrcf[k] = (R(1) - R(0.5) * sk) * lms;
    if (st) ls_st += lms * (meq_st[k - 7] - fm[k] - R(0.5) * mF_st[k - 7]);
  }
  // s = 1 / (1/2 + 3 mu / rho): ds/dphi = -3 s^2 dmu / rho (through mu), ds/drho = 3 s^2 mu / rho^2
  const R lphi_st = visc ? ls_st * (R(-3) * s_st * s_st * p.dmu * irho) : R(0);
  if (visc) lrho += ls_st * (R(3) * s_st * s_st * (p.mu_l + phi * p.dmu) * irho * irho);
  // equilibrium moments (0, 6p + 3 rho uu, -9p - 3 rho uu, rho ux, -rho ux, rho uy, -rho uy,
  // rho (ux^2 - uy^2), rho ux uy)
  const R lpress = R(6) * leqf[1] - R(9) * leqf[2];
  const R l12 = leqf[1] - leqf[2];
  lrho += R(3) * uu * l12 + ux * (leqf[3] - leqf[4]) + uy * (leqf[5] - leqf[6]) +
          (ux * ux - uy * uy) * leqf[7] + ux * uy * leqf[8];
  R lux = R(6) * rho * ux * l12 + rho * (leqf[3] - leqf[4]) + R(2) * rho * ux * leqf[7] + rho * uy * leqf[8];
  R luy = R(6) * rho * uy * l12 + rho * (leqf[5] - leqf[6]) - R(2) * rho * uy * leqf[7] + rho * ux * leqf[8];
  // forcing moments (u.grad rho, 0, -u.grad rho, Fx, -Fx, Fy, -Fy, 2/3 (ux gx - uy gy), 1/3 (ux gy + uy gx))
  R lug = lsrcf[0] - lsrcf[2];
  R lFx = lsrcf[3] - lsrcf[4], lFy = lsrcf[5] - lsrcf[6];
  lux += R(2.0 / 3.0) * grx * lsrcf[7] + R(1.0 / 3.0) * gry * lsrcf[8];
  luy += R(-2.0 / 3.0) * gry * lsrcf[7] + R(1.0 / 3.0) * grx * lsrcf[8];
  R lgrx = R(2.0 / 3.0) * ux * lsrcf[7] + R(1.0 / 3.0) * uy * lsrcf[8];
  R lgry = R(-2.0 / 3.0) * uy * lsrcf[7] + R(1.0 / 3.0) * ux * lsrcf[8];

  // ---- g collision (Eq. 33) in reverse
  R lmg[9];
  d2q9_moments<R>(lgs, lmg);
  R lgm[9], leqg[9], lsrcg[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    const R lms = lmg[k] * R(1.0 / double(row_norm<D2Q9>(k)));
    const R sk = p.sgr[k];
    lgm[k] = (R(1) - sk) * lms;
    leqg[k] = sk * lms;
    lsrcg[k] = (R(1) - R(0.5) * sk) * lms;
    // rates set by the mobility: s = 1 / (1/2 + 3 M), ds/dM = -3 s^2
    if ((a.mobility_rows >> k) & 1) acc_mob += lms * (geq[k] - gm[k] - R(0.5) * gsrc[k]) * (R(-3) * sk * sk);
  }
  const R lH = R(2) * leqg[1] - R(3) * leqg[2];
  R lphi = leqg[0] - R(4) * leqg[1] + R(4) * leqg[2] + p.lam * lH + lphi_st;
  R lmu = lH;
  R lJx = leqg[3] - leqg[4], lJy = leqg[5] - leqg[6];
  const R lVx = (lsrcg[3] - lsrcg[4]) * R(1.0 / 3.0), lVy = (lsrcg[5] - lsrcg[6]) * R(1.0 / 3.0);

  // ---- V = 3 (J - Jprev) + An n (Eq. 32), n = grad psi / sqrt(|grad psi|^2 + eps^2);
  // this step's J is the next step's Jprev
  lJx += R(3) * lVx + lJn[0];
  lJy += R(3) * lVy + lJn[1];
  const R lAn = lVx * nxn + lVy * nyn;
  // where psi has saturated (|grad psi| below the cut) the normal is held fixed
  const bool n_live = !(gsx * gsx + gsy * gsy < a.normal_tau2);
  const R lgsx = n_live ? An * (lVx - nxn * lAn) * ir : R(0);
  const R lgsy = n_live ? An * (lVy - nyn * lAn) * ir : R(0);

  // ---- J = phi u
  lphi += lJx * ux + lJy * uy;
  lux += phi * lJx;
  luy += phi * lJy;

  // ---- pressure (Eq. 29): p = 3/5 (sum_{i>0} f_i + u.grad rho / 2 - 2/3 rho uu)
  const R lP = R(0.6) * lpress;
  lug += R(0.3) * lpress;
  lrho += R(-0.4) * uu * lpress;
  lux += R(-0.8) * rho * ux * lpress + grx * lug;
  luy += R(-0.8) * rho * uy * lpress + gry * lug;
  lgrx += ux * lug;
  lgry += uy * lug;

  // ---- velocity (Eq. 28): u = (j + F/2) / rho
  lfm[3] += lux * irho;
  lfm[5] += luy * irho;
  lFx += R(0.5) * lux * irho;
  lFy += R(0.5) * luy * irho;
  lrho -= (ux * lux + uy * luy) * irho;

  // ---- F = mu grad phi, grad rho = drho grad phi
  lmu += lFx * gpx + lFy * gpy;
  const R lgpx = mu * lFx + p.drho * lgrx, lgpy = mu * lFy + p.drho * lgry;

  // ---- chemical potential (Eq. 2), density, correction amplitude
  lphi += lmu * p.beta4 * (R(3) * phi * phi - R(3) * phi + R(0.5));
  acc_sig += lmu * dmu_dsigma(a, cub, lap);
  lphi += p.drho * lrho + dAn * lAn;

  // ---- the pulled populations through m = M pop, and P = m_0 - f_0
  lfm[0] += lP;
  R lgd[9], lfd[9];
  moments_T(lgm, lgd);
  moments_T(lfm, lfd);
  lfd[0] -= lP;
#pragma unroll
  for (int i = 0; i < 9; ++i) {
    a.lg_out[long(i) * c.n + n] = lgd[i];
    a.lf_out[long(i) * c.n + n] = lfd[i];
  }
  a.lJ_out[n] = R(-3) * lVx;
  a.lJ_out[c.n + n] = R(-3) * lVy;
  // adjoints of what the stencils read, and phi: [phi (own; with the centre weight of the
  // Laplacian, -sum_i 6 w_i = -6 (1 - w_0)), lap phi, d/dx phi, d/dy phi, d/dx psi, d/dy psi, phi]
  const R llap = -p.kappa * lmu;
  a.aux_out[n] = lphi + R(-6.0 * (1.0 - D2Q9::w[0])) * llap;
  a.aux_out[c.n + n] = llap;
  a.aux_out[2 * c.n + n] = lgpx;
  a.aux_out[3 * c.n + n] = lgpy;
  a.aux_out[4 * c.n + n] = lgsx;
  a.aux_out[5 * c.n + n] = lgsy;
  a.aux_out[6 * c.n + n] = phi;
}

// Contributions of the readers of a node's phi and psi in row y through the stencils of
// their own, at(j, dx, dy) = aux component j of the node at (x + dx, y + dy): lphi starts
// from aux 0.
template <class At>
__device__ __forceinline__ R stencil_transpose(const DC& c, int y, R lphi, R phi, At&& at) {
  const bool wall = c.wall;
  R lpsi = R(0);
  R gphi[2] = {R(0), R(0)}, gpsi[2] = {R(0), R(0)};   // through the ghost rows (bottom, top)
#pragma unroll
  for (int i = 1; i < 9; ++i) {
    const R wx = R(3.0 * D2Q9::w[i] * D2Q9::cx[i]), wy = R(3.0 * D2Q9::w[i] * D2Q9::cy[i]), wl = R(6.0 * D2Q9::w[i]);
    auto dphi = [&](int dy) {
      R v = wl * at(1, -D2Q9::cx[i], dy);
      if (D2Q9::cx[i] != 0) v += wx * at(2, -D2Q9::cx[i], dy);
      if (D2Q9::cy[i] != 0) v += wy * at(3, -D2Q9::cx[i], dy);
      return v;
    };
    auto dpsi = [&](int dy) {
      R v = R(0);
      if (D2Q9::cx[i] != 0) v += wx * at(4, -D2Q9::cx[i], dy);
      if (D2Q9::cy[i] != 0) v += wy * at(5, -D2Q9::cx[i], dy);
      return v;
    };
    const int ys = y - D2Q9::cy[i];
    if (!wall || (ys >= 0 && ys < c.ny)) {
      lphi += dphi(-D2Q9::cy[i]);
      lpsi += dpsi(-D2Q9::cy[i]);
    }
    // readers of the ghost row behind a wall, which holds the wetting ghost of this edge
    // node: nodes of this row
    if (wall && D2Q9::cy[i] < 0 && y == 0) {
      gphi[0] += dphi(0);
      gpsi[0] += dpsi(0);
    }
    if (wall && D2Q9::cy[i] > 0 && y == c.ny - 1) {
      gphi[1] += dphi(0);
      gpsi[1] += dpsi(0);
    }
  }
  lphi += lpsi * dpsi_dphi(c, phi);
  // the ghost value phi_g (and psi of it) depends on this edge node's phi
  for (int k = 0; k < 2; ++k) {
    if (gphi[k] == R(0) && gpsi[k] == R(0)) continue;
    const R w = wet_coef(c, k ? 1 : -1);
    const R phig = wet_ghost<R>(phi, w);
    lphi += wet_slope(w, phi) * (gphi[k] + gpsi[k] * dpsi_dphi(c, phig));
  }
  return lphi;
}

// One backward step.  FIRST: the last step of the run, whose lphi is the seed (a.lphi).
template <int LX, int LY, bool FIRST>
__global__ void __launch_bounds__(1 << (LX + LY), 3) k_adj_tile(DC c, AdjArgs a, int ntx, int ntiles) {
  constexpr int TX = 1 << LX, TY = 1 << LY, nodes = TX * TY;
  constexpr int PW = TX + 2, ring1 = PW * (TY + 2), AW = TX + 4, ring2 = AW * (TY + 4);
  struct alignas(16) PhiPsi {
    R phi, psi;
  };
  __shared__ PhiPsi ring[ring1];
  __shared__ R lph[ring1];
  __shared__ R ax[FIRST ? 1 : 5][FIRST ? 1 : ring2];
  const int tile = xcd_tile(blockIdx.x, ntiles);
  const int tyi = tile / ntx, txi = tile - tyi * ntx;
  const int nx = c.nx, ny = c.ny;
  const bool wall = c.wall;
  const int x0 = txi * TX, y0 = tyi * TY;
  const int tid = threadIdx.x, tx = tid % TX, ty = tid / TX;
  const int xg = x0 + tx, yg = y0 + ty;
  const bool active = xg < nx && yg < ny;
  // node of a position around the tile: the periodic image, or past a wall the edge row
  auto col_of = [&](int x) { return x >= 0 && x < nx ? x : (x % nx + nx) % nx; };
  auto row_of = [&](int y) {
    if (y >= 0 && y < ny) return y;
    if (wall) return y < 0 ? 0 : ny - 1;
    return (y % ny + ny) % ny;
  };
  const int x = col_of(xg), y = row_of(yg);
  const long n = x + long(nx) * y;
  // loads first: the node's populations, and the adjoints of its post-collision ones
  R g[9], f[9], Jp[2], lgs[9], lfs[9], lJn[2];
  pull<D2Q9, StoreF64>(c, c.pop[0][0], nullptr, x, y, 0, g, nullptr);
  if (active) {
    pull<D2Q9, StoreF64>(c, c.pop[1][0], nullptr, x, y, 0, f, nullptr);
    Jp[0] = ldg(c.J, n);
    Jp[1] = ldg(c.J, c.ns + n);
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      const int yd = y + D2Q9::cy[i];
      const bool back = wall && (yd < 0 || yd >= ny);   // bounced back: read by this node as the opposite direction
      const long dst = back ? n : col_of(x + D2Q9::cx[i]) + long(nx) * row_of(yd);
      const int di = back ? D2Q9::opp[i] : i;
      lgs[i] = ldg(a.lg_in, long(di) * c.n + dst);
      lfs[i] = ldg(a.lf_in, long(di) * c.n + dst);
    }
    lJn[0] = ldg(a.lJ_in, n);
    lJn[1] = ldg(a.lJ_in, c.n + n);
  }
  if constexpr (!FIRST) {
    for (int k = tid; k < ring2; k += nodes) {
      const int py = k / AW, px = k - py * AW;
      const long m = col_of(x0 - 2 + px) + long(nx) * row_of(y0 - 2 + py);
#pragma unroll
      for (int j = 0; j < 5; ++j) ax[j][k] = ldg(a.aux_in, (j + 1) * c.n + m);
    }
  }
  auto form = [&](const R (&v)[9], int yr, int at) {
    R ph = R(0);
#pragma unroll
    for (int i = 0; i < 9; ++i) ph += v[i];
    if (wall && yr < 0) ph = wet_ghost<R>(ph, c.np.wet_lo);
    else if (wall && yr >= ny) ph = wet_ghost<R>(ph, c.np.wet_hi);
    ring[at] = PhiPsi{ph, psi_of<R>(ph, c.np.W4, c.np.xi)};
  };
  // halo cells of phi and psi, one per lane
  constexpr int nring = 2 * PW + 2 * TY;
  static_assert(nring <= nodes, "a halo cell per lane");
  if (tid < nring) {
    int px, py;
    if (tid < 2 * PW) {
      py = tid < PW ? 0 : TY + 1;
      px = tid < PW ? tid : tid - PW;
    } else {
      const int k = tid - 2 * PW;
      py = 1 + (k >> 1);
      px = (k & 1) ? PW - 1 : 0;
    }
    R gh[9];
    pull<D2Q9, StoreF64>(c, c.pop[0][0], nullptr, col_of(x0 - 1 + px), row_of(y0 - 1 + py), 0, gh, nullptr);
    form(gh, y0 - 1 + py, py * PW + px);
  }
  const int own = (ty + 1) * PW + tx + 1;
  form(g, yg, own);
  __syncthreads();
  // lphi of the step before (in backward order) on the tile and its halo
  for (int k = tid; k < ring1; k += nodes) {
    const int py = k / PW, px = k - py * PW, yr = y0 - 1 + py;
    if (wall && (yr < 0 || yr >= ny)) continue;   // nothing streams to a row behind a wall
    const int yw = row_of(yr);
    const long m = col_of(x0 - 1 + px) + long(nx) * yw;
    if constexpr (FIRST) {
      lph[k] = ldg(a.lphi, m);
    } else {
      const int at0 = (py + 1) * AW + px + 1;
      lph[k] = stencil_transpose(c, yw, ldg(a.aux_in, m), ldg(a.aux_in, 6 * c.n + m),
                                 [&](int j, int dx, int dy) { return ax[j - 1][at0 + dy * AW + dx]; });
    }
  }
  __syncthreads();
  double acc_sig = 0.0, acc_mob = 0.0;
  if (active) {
    R q[9], s[9], lrho = R(0);
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      const int o = own + D2Q9::cy[i] * PW + D2Q9::cx[i];
      q[i] = ring[o].phi;
      s[i] = ring[o].psi;
      const int yd = y + D2Q9::cy[i];
      lgs[i] += lph[wall && (yd < 0 || yd >= ny) ? own : o];
      // moving-wall term added to the populations leaving through a wall
      if (wall && y == 0 && D2Q9::cy[i] < 0) lrho += c.np.wb[i] * lfs[i];
      if (wall && y == ny - 1 && D2Q9::cy[i] > 0) lrho += c.np.wt[i] * lfs[i];
    }
    adj_node(c, a, n, q, s, g, f, Jp, lgs, lfs, lJn, lrho, acc_sig, acc_mob);
  }
  add_params(a, tile, acc_sig, acc_mob);
}

// lphi of the first step of the run, for the initial state's reverse
__global__ void __launch_bounds__(256) k_adj_stencil(DC c, AdjArgs a) {
  const long n = blockIdx.x * long(blockDim.x) + threadIdx.x;
  if (n >= c.n) return;
  const int x = int(n % c.nx), y = int(n / c.nx);
  a.lphi[n] = stencil_transpose(c, y, a.aux_in[n], a.aux_in[6 * c.n + n], [&](int j, int dx, int dy) {
    const int yr = c.wall ? (y + dy < 0 ? 0 : (y + dy >= c.ny ? c.ny - 1 : y + dy)) : xwrap(y + dy, c.ny);
    return a.aux_in[j * c.n + xwrap(x + dx, c.nx) + long(c.nx) * yr];
  });
}

// -------------------------------------------------------------------------- initial state
// pass 1 at node x: dJ/d(phi0(x)) through g_eq, f_eq and Jprev at x, and the adjoint of
// lap phi0(x) (written to aux[1]); mu0 = 4 beta c(phi0) - kappa lap phi0
__global__ void __launch_bounds__(256) k_adj_init_local(DC c, AdjArgs a, const double* __restrict__ phi0,
                                                        const double* __restrict__ u0) {
  const long n = blockIdx.x * long(blockDim.x) + threadIdx.x;
  double acc_sig = 0.0;
  if (n < c.n) {
    const int nx = c.nx, ny = c.ny;
    const int x = int(n % nx), y = int(n / nx);
    const auto& p = c.np;
    R q[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      q[i] = phi0[xwrap(x + D2Q9::cx[i], nx) + long(nx) * stencil_row(y, D2Q9::cy[i], ny, c.wall)];
      const int yn = y + D2Q9::cy[i];
      if (c.wall && (yn < 0 || yn >= ny)) q[i] = wet_ghost<R>(q[i], wet_coef(c, yn < 0 ? -1 : 1));
    }
    const R phi = q[0];
    const R lap = R(2.0 / 3.0) * (((q[1] + q[3]) + (q[2] + q[4])) - R(4) * q[0]) +
                  R(1.0 / 6.0) * (((q[5] + q[7]) + (q[6] + q[8])) - R(4) * q[0]);
    const R cub = phi * (phi - R(1)) * (phi - R(0.5));
    const R ux = u0 ? u0[n] : R(0), uy = u0 ? u0[c.n + n] : R(0);
    const R uu = ux * ux + uy * uy;
    const R lph = a.lphi[n];
    R lH = R(0), lphi = R(0);
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      const R lg = a.lg_in[long(i) * c.n + n] + lph;
      const R lf = a.lf_in[long(i) * c.n + n];
      const R wi = R(D2Q9::w[i]);
      const R cu = R(D2Q9::cx[i]) * ux + R(D2Q9::cy[i]) * uy;
      // Eq. 31: g_0 = phi + (w_0 - 1) H, g_i = w_i H + 3 w_i c_i . (phi u)
      if (i == 0) {
        lH += R(D2Q9::w[0] - 1.0) * lg;
        lphi += lg;
      } else {
        lH += wi * lg;
        lphi += R(3) * wi * cu * lg;
      }
      // Eqs. 22-23 at p = 0: f_i = rho s_i(u)
      lphi += p.drho * wi * (R(3) * cu + R(4.5) * cu * cu - R(1.5) * uu) * lf;
    }
    lphi += ux * a.lJ_in[n] + uy * a.lJ_in[c.n + n];
    lphi += p.lam * lH + lH * p.beta4 * (R(3) * phi * phi - R(3) * phi + R(0.5));
    acc_sig += lH * dmu_dsigma(a, cub, lap);
    a.aux_out[n] = lphi;
    a.aux_out[c.n + n] = -p.kappa * lH;
  }
  add_params(a, blockIdx.x, acc_sig, 0.0);
}

__global__ void __launch_bounds__(256) k_adj_init_stencil(DC c, AdjArgs a, const double* __restrict__ phi0,
                                                          double* __restrict__ dphi0) {
  const long n = blockIdx.x * long(blockDim.x) + threadIdx.x;
  if (n >= c.n) return;
  const int x = int(n % c.nx), y = int(n / c.nx);
  const double* llap = a.aux_out + c.n;
  R v = a.aux_out[n] + R(-6.0 * (1.0 - D2Q9::w[0])) * llap[n];
  stencil_readers(c, x, y, [&](int i, long m, int side) {
    const R t = R(6.0 * D2Q9::w[i]) * llap[m];
    v += side ? wet_slope(wet_coef(c, side), phi0[n]) * t : t;   // a ghost read: d(phi_g)/d(phi_e)
  });
  dphi0[n] = v;
}

// (dJ/dsigma, dJ/dM): the per-workgroup slots summed in workgroup order
__global__ void __launch_bounds__(256) k_adj_params(AdjArgs a, double* __restrict__ out) {
  __shared__ double red[16 * 2];
  double v[2] = {0.0, 0.0};
  for (long b = threadIdx.x; b < a.part_slots; b += blockDim.x) {
    v[0] += a.param_part[b];
    v[1] += a.param_part[a.part_slots + b];
  }
  const double s = block_sum_fields<2>(v, 2, red);
  if (threadIdx.x < 2) out[threadIdx.x] = s;
}

__global__ void __launch_bounds__(256) k_adj_zero(double* __restrict__ p, long count) {
  const long i = blockIdx.x * long(blockDim.x) + threadIdx.x;
  if (i < count) p[i] = 0.0;
}

// -------------------------------------------------------------------------- launchers
namespace {
unsigned blocks_for(long n) { return unsigned((n + 255) / 256); }
// tiles of k_adj_tile: 16 x 8 nodes (32 x 8, 64 x 4, 16 x 16 and 32 x 4 within 3% on 512 x 256
// and 1024 x 700, 16 x 8 6% ahead on 128 x 64)
constexpr int kAdjLX = 4, kAdjLY = 3;
long adj_tiles(int nx, int ny) {
  return long((nx + (1 << kAdjLX) - 1) >> kAdjLX) * ((ny + (1 << kAdjLY) - 1) >> kAdjLY);
}
int last_status() { return hipGetLastError() == hipSuccess ? 0 : -3; }
}  // namespace

// slots of the parameter sums: the tiles of a step, or the blocks of the initial state
long adj_part_slots(int nx, int ny) {
  return std::max(adj_tiles(nx, ny), long(blocks_for(long(nx) * ny)));
}

int launch_adj_zero(double* p, long count, hipStream_t s) {
  hipLaunchKernelGGL(k_adj_zero, dim3(blocks_for(count)), dim3(256), 0, s, p, count);
  return last_status();
}

int launch_adj_seed(const DC& c, const AdjArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_adj_seed, dim3(blocks_for(c.n)), dim3(256), 0, s, c, a);
  return last_status();
}

int launch_adj_step(const DC& c, const AdjArgs& a, bool first, hipStream_t s) {
  const int ntx = (c.nx + (1 << kAdjLX) - 1) >> kAdjLX, ntiles = int(adj_tiles(c.nx, c.ny));
  const dim3 grid{unsigned(ntiles)}, block(1 << (kAdjLX + kAdjLY));
  if (first) hipLaunchKernelGGL((k_adj_tile<kAdjLX, kAdjLY, true>), grid, block, 0, s, c, a, ntx, ntiles);
  else hipLaunchKernelGGL((k_adj_tile<kAdjLX, kAdjLY, false>), grid, block, 0, s, c, a, ntx, ntiles);
  return last_status();
}

int launch_adj_stencil(const DC& c, const AdjArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_adj_stencil, dim3(blocks_for(c.n)), dim3(256), 0, s, c, a);
  return last_status();
}

int launch_adj_init(const DC& c, const AdjArgs& a, const double* phi0, const double* u0, double* dphi0,
                    hipStream_t s) {
  hipLaunchKernelGGL(k_adj_init_local, dim3(blocks_for(c.n)), dim3(256), 0, s, c, a, phi0, u0);
  hipLaunchKernelGGL(k_adj_init_stencil, dim3(blocks_for(c.n)), dim3(256), 0, s, c, a, phi0, dphi0);
  return last_status();
}

int launch_adj_params(const AdjArgs& a, double* out, hipStream_t s) {
  hipLaunchKernelGGL(k_adj_params, dim3(1), dim3(256), 0, s, a, out);
  return last_status();
}

}  // namespace vclb
