// The tile step of tile2d.hip as a device function, shared by the single-case kernel and
// the batched one.
#pragma once
#include <hip/hip_runtime.h>

#include "devcase.hpp"
#include "flat2d.hpp"

namespace vclb {

// Lanes of a workgroup for tiles of 2^LX x 2^LY nodes, with or without the helper wave.
constexpr int tile2d_lanes(int LX, int LY, bool help) { return (1 << (LX + LY)) + (help ? 64 : 0); }

// The volume reductions of a tile of TX x TY nodes from (x0, y0), by one whole wave from the
// phi of its nodes in LDS (rows of PW entries): six sums over the wave once per tile.
template <int TX, int TY, int PW, class Case, class PhiPsi>
__device__ __forceinline__ void tile2d_sums(const Case& c, const PhiPsi* ring, int x0, int y0, double* __restrict__ part,
                                            long part_stride) {
  const int nx = c.nx, ny = c.ny;
  const bool wall = c.wall != 0;
  // A lane keeps to a column (or two, TX = 128), so only phi, phi dy, phi dy^2 add up per
  // node and the x moments follow.
  const int lane = threadIdx.x & 63;
  constexpr int kCols = TX > 64 ? TX / 64 : 1, kRowStep = TX < 64 ? 64 / TX : 1;
  double s[kMaxLabels][6];
  int cnt[kMaxLabels], bad[kMaxLabels];
#pragma unroll
  for (int k = 0; k < kMaxLabels; ++k) {
    cnt[k] = bad[k] = 0;
#pragma unroll
    for (int j = 0; j < 6; ++j) s[k][j] = 0.0;
  }
#pragma unroll
  for (int h = 0; h < kCols; ++h) {
    const int rx = lane % TX + 64 * h, x = x0 + rx;
    double dx[kMaxLabels], s0[kMaxLabels], s1[kMaxLabels], s2[kMaxLabels];
#pragma unroll
    for (int k = 0; k < kMaxLabels; ++k) {
      dx[k] = min_image(double(x) - c.cen[k][0], nx, true);
      s0[k] = s1[k] = s2[k] = 0.0;
    }
#pragma unroll
    for (int i = 0; i < TY / kRowStep; ++i) {
      const int ry = lane / TX + i * kRowStep, y = y0 + ry;
      const double ph = x < nx && y < ny ? double(ring[ry * PW + rx].phi) : 0.0;
      double dy[kMaxLabels];
#pragma unroll
      for (int k = 0; k < kMaxLabels; ++k) dy[k] = min_image(double(y) - c.cen[k][1], ny, !wall);
      const int lab = c.nl > 1 && dx[1] * dx[1] + dy[1] * dy[1] < dx[0] * dx[0] + dy[0] * dy[0] ? 1 : 0;
#pragma unroll
      for (int k = 0; k < kMaxLabels; ++k) {
        if (k >= c.nl) break;
        const double w = lab == k ? ph : 0.0;
        s0[k] += w;
        s1[k] += w * dy[k];
        s2[k] += w * dy[k] * dy[k];
        cnt[k] += __popcll(__ballot(lab == k && ph >= 0.5));
        bad[k] += __popcll(__ballot(lab == k && !isfinite(ph)));
      }
    }
#pragma unroll
    for (int k = 0; k < kMaxLabels; ++k) {
      s[k][0] += s0[k];
      s[k][1] += dx[k] * s0[k];
      s[k][2] += s1[k];
      s[k][3] += dx[k] * dx[k] * s0[k];
      s[k][4] += s2[k];
      s[k][5] += dx[k] * s1[k];
    }
  }
  // lane 16 i + 15 stores field i of each group of four
#pragma unroll
  for (int k = 0; k < kMaxLabels; ++k) {
    if (k >= c.nl) break;
    const double a = wave_sum4(s[k][0], s[k][1], s[k][2], s[k][3]);
    double b = wave_sum4(s[k][4], s[k][5], 0.0, 0.0);
    const int i = lane >> 4;
    if (i >= 2) b = double(i == 2 ? cnt[k] : bad[k]);
    if ((lane & 15) == 15) {
      // fields: sum, count, x, y, z, xx, yy, zz, xy, xz, yz, not finite
      const int fa = i == 0 ? 0 : (i == 1 ? 2 : (i == 2 ? 3 : 5)), fb = i == 0 ? 6 : (i == 1 ? 8 : (i == 2 ? 1 : 11));
      const int fz = i == 0 ? 4 : (i == 1 ? 7 : (i == 2 ? 9 : 10));
      stg(part, long(k * 12 + fa) * part_stride, a);
      stg(part, long(k * 12 + fb) * part_stride, b);
      stg(part, long(k * 12 + fz) * part_stride, 0.0);
    }
  }
}

// f of a node just updated, on its way to a 2-byte storage: a value is rounded either to 4
// bytes first or once, together with the multiply-add that forms it.  Which of the two is
// that of the march the case would otherwise run, so that its results are the march's bit
// for bit: the compiled march of a single case rounds the directions that take no wall term
// once, a batch's strips none and its bands direction 0 (`band`).  These directions are
// encoded first, before the wall terms.
enum class Once { Level, OfBand };
template <class St, Once ONCE>
constexpr bool encoded_first(int i) {
  return sizeof(typename St::S) == 2 && D2Q9::cy[i] == 0 && (ONCE == Once::Level || i == 0);
}
template <class St, Once ONCE>
__device__ __forceinline__ void encode_first(const typename St::R (&f)[9], bool band, typename St::S (&e)[4]) {
  if constexpr (sizeof(typename St::S) == 2) {
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      if (!encoded_first<St, ONCE>(i)) continue;
      unsigned u = __half_as_ushort(St::enc(f[i]));
      asm("" : "+v"(u));   // on its own: not converted after the choice below
      e[i & 3] = __ushort_as_half((unsigned short)u);
      if (ONCE != Once::Level) {
        const typename St::S b = St::enc(rounded(f[i]));   // both, with no branch (which would part the update)
        e[i & 3] = band ? e[i & 3] : b;
      }
    }
  }
}

// One step (time level t) of tile `tile` of case c, by one whole workgroup; ntx tiles span
// a row of tiles.  part: this tile's slot of the reduction partials (field j of label k at
// [(k * 12 + j) * part_stride]), null when the step records none.
//
// LX, LY: log2 of the tile's sides.  HELP: one more wave, which pulls the first 64 halo cells and
// sums the tile's reductions while the others update.  That takes both off the critical
// path of a step that waits for one launch (128 x 128 FP64: 7.4 -> 5.2 us, the reductions
// free), but a wave in three idles; large grids, which need every wave
// (1501 x 1003 FP16S: 27.7 -> 31.3 us), leave both to the tile's own lanes.
// NT: stores of the populations and loads of f with the non-temporal hint.
// ONCE: the directions of f that may be rounded once: all on the level, or direction 0 of a
// case that a batch's runs would do in bands (`band`).
template <class St, bool COUPLED, bool UNIT, bool VISC, int LX, int LY, bool HELP, bool NT, Once ONCE>
__device__ __forceinline__ void tile2d_step(const DevCase<D2Q9, St>& c, long t, int tile, int ntx,
                                            double* __restrict__ part, long part_stride, bool band) {
  using L = D2Q9;
  using R = typename St::R;
  using S = typename St::S;
  constexpr int Q = 9;
  struct alignas(2 * sizeof(R)) PhiPsi {
    R phi, psi;
  };
  constexpr int TX = 1 << LX, TY = 1 << LY, PW = TX + 2, nodes = TX * TY;
  constexpr int nring = 2 * PW + 2 * TY;   // halo cells
  static_assert(nring <= nodes && nodes % 64 == 0, "a halo cell per lane");
  __shared__ PhiPsi ring[PW * (TY + 2)];   // the tile and its halo
  const int ty_i = tile / ntx, tx_i = tile - ty_i * ntx;
  const int nx = c.nx, ny = c.ny, ns = int(c.ns);
  const int x0 = tx_i * TX, y0 = ty_i * TY;
  const int tid = threadIdx.x;
  const bool helper = HELP && tid >= nodes;   // the last wave has no node of its own
  const int tx = tid % TX, ty = tid / TX;
  const int xg = x0 + tx, yg = y0 + ty;
  const bool active = !helper && xg < nx && yg < ny;
  const bool wall = c.wall != 0;
  // column and row whose populations a ring position holds: the periodic image, or, past
  // a wall, the edge row (whose wetting ghost the ring then holds)
  auto col_of = [&](int x) { return x >= 0 && x < nx ? x : (x % nx + nx) % nx; };
  auto row_of = [&](int y) {
    if (y >= 0 && y < ny) return y;
    if (wall) return y < 0 ? 0 : ny - 1;
    return (y % ny + ny) % ny;
  };
  const int xw = col_of(xg), yw = row_of(yg);
  const int par = int(t & 1), dst = par ^ 1;
  const S* gsrc[Q];
  const S* fsrc[Q];
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    gsrc[i] = c.pop[0][par] + long(i) * ns;
    fsrc[i] = COUPLED ? c.pop[1][par] + long(i) * ns : nullptr;
  }
  const float* phis = c.phis[par];
  const unsigned nn = unsigned(xw + nx * yw);
  // every load of this lane before the first use: its node's g, a halo cell's g, f, J
  R g[Q], ps[Q], f[Q], J[2], gh[Q], hps[Q];
  if (!helper) pull9_flat<St>(gsrc, phis, xw, yw, nx, ny, ns, wall, g, ps);
  // halo cells, one per lane: the helper wave first, then the tile's lanes from lane 0
  const int cell = !HELP ? tid : (helper ? tid - nodes : tid + 64);
  int px = 0, py = 0;
  if (cell < nring) {
    if (cell < 2 * PW) {
      py = cell < PW ? 0 : TY + 1;
      px = cell < PW ? cell : cell - PW;
    } else {
      const int k = cell - 2 * PW;
      py = 1 + (k >> 1);
      px = (k & 1) ? PW - 1 : 0;
    }
    pull9_flat<St>(gsrc, phis, col_of(x0 - 1 + px), row_of(y0 - 1 + py), nx, ny, ns, wall, gh, hps);
  }
  if (active) {
    if constexpr (COUPLED) pull9_flat<St, NT>(fsrc, phis, xw, yw, nx, ny, ns, wall, f, nullptr);
    J[0] = ldg(c.J, nn);
    J[1] = ldg(c.J + ns, nn);
  }
  // the vortex factors of the tile's columns, rows and the step, once per tile and not per
  // node: sin(pi x / nx), sin(2 pi x / nx) of column i at [i], of row i at [TX + i]
  __shared__ R trig[COUPLED ? 1 : 2][COUPLED ? 1 : TX + TY + 1];
  if constexpr (!COUPLED) {
    if (tid < TX) vortex_factors<R>(col_of(x0 + tid), nx, trig[0][tid], trig[1][tid]);
    else if (tid < TX + TY) vortex_factors<R>(row_of(y0 + tid - TX), ny, trig[0][tid], trig[1][tid]);
    else if (tid == TX + TY) trig[0][tid] = vortex_phase<R>(c.np.T, t);
  }
  auto form = [&](R (&v)[Q], const R (&vps)[Q], int y, int at) {
    R ph = phi_of_pulled<L, St>(v, vps, c.np.rest);
    if (wall && y < 0) ph = wet_ghost<R>(ph, c.np.wet_lo);
    else if (wall && y >= ny) ph = wet_ghost<R>(ph, c.np.wet_hi);
    ring[at] = PhiPsi{ph, psi_of<R>(ph, c.np.W4, c.np.xi)};
  };
  const int own = (ty + 1) * PW + tx + 1;
  if (!helper) form(g, ps, yg, own);
  if (cell < nring) form(gh, hps, y0 - 1 + py, py * PW + px);
  __syncthreads();
  if (active) {
    NodeIn<L, R> in;
#pragma unroll
    for (int i = 0; i < Q; ++i) {
      const PhiPsi v = ring[own + L::cy[i] * PW + L::cx[i]];
      in.nphi[i] = v.phi;
      in.npsi[i] = v.psi;
    }
    if constexpr (!COUPLED) {
      vortex_from_factors<R>(c.np.U0, trig[0][tx], trig[1][tx], trig[0][TX + ty], trig[1][TX + ty], trig[0][TX + TY],
                             in.u[0], in.u[1]);
    }
    NodeOut<L, R> out;
    node_update_d2q9<R, COUPLED, St::shifted, UNIT, VISC, !COUPLED>(c.np, in, g, f, J, out);
    auto store_f = [&](int i, S e) {
      if constexpr (NT) St::store_s_nt(c.pop[1][dst] + long(i) * ns, nn, e);
      else St::store_s(c.pop[1][dst] + long(i) * ns, nn, e);
    };
    if constexpr (COUPLED) {
      S e[4];
      encode_first<St, ONCE>(f, band, e);
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (encoded_first<St, ONCE>(i)) store_f(i, e[i]);
    }
    R res = R(0);   // rounding of the stored g deviations, taken off the stored phi
#pragma unroll
    for (int i = 0; i < Q; ++i) {
      R d = g[i];
      if constexpr (St::shifted)   // relative to the reader's phi (encode_dev)
        d = encode_dev(g[i], c.np.rest[i], in.nphi[0],
                       leaves_through_wall<L>(i, yw, ny, wall) ? in.nphi[0] : in.nphi[i]);
      if constexpr (NT) St::store_nt(c.pop[0][dst] + long(i) * ns, nn, d);
      else St::store(c.pop[0][dst] + long(i) * ns, nn, d);
      if constexpr (St::fold) res += St::rounding(d);
    }
    if constexpr (COUPLED) {
      if (wall && yw == 0) {
#pragma unroll
        for (int i = 0; i < Q; ++i)
          if (L::cy[i] < 0) f[i] += c.np.wb[i] * out.rho;
      }
      if (wall && yw == ny - 1) {
#pragma unroll
        for (int i = 0; i < Q; ++i)
          if (L::cy[i] > 0) f[i] += c.np.wt[i] * out.rho;
      }
#pragma unroll
      for (int i = 0; i < Q; ++i)
        if (!encoded_first<St, ONCE>(i)) store_f(i, St::enc(f[i]));
    }
    stg(c.Jw, nn, J[0]);
    stg(c.Jw + ns, nn, J[1]);
    if constexpr (St::shifted) stg(c.phis[dst], nn, float(in.nphi[0] - res));
  }
  // this tile's volume reductions, by one wave from the ring's phi: the helper, or the last
  // wave (the first ones pull the halo).  Six sums over the wave once per tile instead of
  // once per wave: 1501 x 1003 FP16S 34.9 -> 27.7 us.
  if (!part || tid < (HELP ? nodes : nodes - 64)) return;
  tile2d_sums<TX, TY, PW>(c, ring + PW + 1, x0, y0, part, part_stride);
}

// Up to three steps (time levels t to t + n - 1) of tile `tile` in one go, by one whole
// workgroup: the state of the last goes to memory, those between stay in LDS.
//
// The workgroup pulls the tile and kHalo nodes around it from memory, one lane per node,
// and each step updates the nodes that the later ones still need: a step reaches two
// nodes (the stencils of phi and psi, whose nodes pull from one further).  The lanes keep
// their nodes over the steps, and J with them; the populations between two steps go
// through LDS in the storage's precision.  Rows and columns past a periodic face hold the
// images, updated along; rows past a wall only the wetting ghost.  part: as in tile2d_step,
// the steps' partials part_set apart, for the steps of the mask `reduce`.
//
// One loop body serves every step of the launch and launches of one step: the results do
// not depend on how steps are grouped.
//
// What bounds it: a step's instructions in one wave per SIMD (some 900 of 4 cycles, 1.2 us
// with the waits), after 3 us of launch, pulls and stores, against 5 us a step when each is
// a launch.  Three steps, because an odd number keeps the state in the buffers of its
// parity; five would repeat 24 x 24 nodes for 8 x 8.  The updates of the halo are four
// times (8 x 8) or two and a quarter (16 x 16) those of the tile, free only while the CUs
// hold one workgroup.  The helper's sums add 0.2 us (8 x 8) to 0.7 us a step (16 x 16);
// with the sums over the wave moved past the barrier they were no cheaper (more registers).
constexpr int kMultiSteps = 3, kMultiHalo = 2 * (kMultiSteps - 1);
constexpr int tile2d_multi_nodes(int LX, int LY) { return ((1 << LX) + 2 * kMultiHalo) * ((1 << LY) + 2 * kMultiHalo); }
constexpr int tile2d_multi_lanes(int LX, int LY) { return tile2d_multi_nodes(LX, LY) + 64; }

template <class St, bool COUPLED, bool UNIT, bool VISC, int LX, int LY>
__device__ __forceinline__ void tile2d_multi(const DevCase<D2Q9, St>& c, long t, int n, int tile, int ntx, int reduce,
                                             double* __restrict__ part, long part_stride, long part_set) {
  using L = D2Q9;
  using R = typename St::R;
  using S = typename St::S;
  constexpr int Q = 9, H = kMultiHalo;
  struct alignas(2 * sizeof(R)) PhiPsi {
    R phi, psi;
  };
  constexpr int TX = 1 << LX, TY = 1 << LY, RX = TX + 2 * H, RY = TY + 2 * H, PW = RX + 2;
  constexpr int nodes = tile2d_multi_nodes(LX, LY);
  constexpr int nring = 2 * PW + 2 * RY;   // halo cells of the whole region
  static_assert(nring <= nodes && nodes % 64 == 0, "a halo cell per lane");
  __shared__ PhiPsi ring[PW * (RY + 2)];
  __shared__ S pops[COUPLED ? 2 : 1][Q][nodes];
  __shared__ float phl[St::shifted ? nodes : 1];
  const int ty_i = tile / ntx, tx_i = tile - ty_i * ntx;
  const int nx = c.nx, ny = c.ny, ns = int(c.ns);
  const int x0 = tx_i * TX, y0 = ty_i * TY;
  const int tid = threadIdx.x;
  const bool helper = tid >= nodes;   // the last wave: halo cells and reductions
  const int rx = tid % RX, ry = tid / RX;
  const int xg = x0 - H + rx, yg = y0 - H + ry;
  const bool wall = c.wall != 0;
  auto col_of = [&](int x) { return x >= 0 && x < nx ? x : (x % nx + nx) % nx; };
  auto row_of = [&](int y) {
    if (y >= 0 && y < ny) return y;
    if (wall) return y < 0 ? 0 : ny - 1;
    return (y % ny + ny) % ny;
  };
  const int xw = col_of(xg), yw = row_of(yg);
  // how far the node lies outside the tile: step k from the last updates those within 2 k
  const int dx = rx < H ? H - rx : (rx >= H + TX ? rx - (H + TX - 1) : 0);
  const int dy = ry < H ? H - ry : (ry >= H + TY ? ry - (H + TY - 1) : 0);
  const int dist = helper ? 1 << 20 : (dx > dy ? dx : dy);
  const bool node = !wall || (yg >= 0 && yg < ny);
  const int par = int(t & 1), dst = (par + n) & 1;
  const S* gsrc[Q];
  const S* fsrc[Q];
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    gsrc[i] = c.pop[0][par] + long(i) * ns;
    fsrc[i] = COUPLED ? c.pop[1][par] + long(i) * ns : nullptr;
  }
  const float* phis = c.phis[par];
  const unsigned nn = unsigned(xw + nx * yw);
  // every load of this lane before the first use
  R g[Q], ps[Q], f[Q], J[2], gh[Q], hps[Q];
  if (dist <= 2 * n - 1) pull9_flat<St>(gsrc, phis, xw, yw, nx, ny, ns, wall, g, ps);
  const int cell = n < kMultiSteps ? nring : (helper ? tid - nodes : tid + 64);
  int px = 0, py = 0;
  if (cell < nring) {
    if (cell < 2 * PW) {
      py = cell < PW ? 0 : RY + 1;
      px = cell < PW ? cell : cell - PW;
    } else {
      const int k = cell - 2 * PW;
      py = 1 + (k >> 1);
      px = (k & 1) ? PW - 1 : 0;
    }
    pull9_flat<St>(gsrc, phis, col_of(x0 - H - 1 + px), row_of(y0 - H - 1 + py), nx, ny, ns, wall, gh, hps);
  }
  if (dist <= 2 * (n - 1) && node) {
    if constexpr (COUPLED) pull9_flat<St>(fsrc, phis, xw, yw, nx, ny, ns, wall, f, nullptr);
    J[0] = ldg(c.J, nn);
    J[1] = ldg(c.J + ns, nn);
  }
  __shared__ R trig[COUPLED ? 1 : 2][COUPLED ? 1 : RX + RY + kMultiSteps];
  if constexpr (!COUPLED) {
    if (tid < RX) vortex_factors<R>(xw, nx, trig[0][tid], trig[1][tid]);
    else if (tid < RX + RY) vortex_factors<R>(row_of(y0 - H + tid - RX), ny, trig[0][tid], trig[1][tid]);
    else if (tid < RX + RY + n) trig[0][tid] = vortex_phase<R>(c.np.T, t + (tid - RX - RY));
  }
  auto form = [&](R (&v)[Q], const R (&vps)[Q], int y, int at) {
    R ph = phi_of_pulled<L, St>(v, vps, c.np.rest);
    if (wall && y < 0) ph = wet_ghost<R>(ph, c.np.wet_lo);
    else if (wall && y >= ny) ph = wet_ghost<R>(ph, c.np.wet_hi);
    ring[at] = PhiPsi{ph, psi_of<R>(ph, c.np.W4, c.np.xi)};
  };
  const int own = (ry + 1) * PW + rx + 1;
  if (cell < nring) form(gh, hps, y0 - H - 1 + py, py * PW + px);
#pragma clang loop unroll(disable)
  for (int m = n - 1;; --m) {   // m steps follow this one
    if (dist <= 2 * m + 1) form(g, ps, yg, own);
    __syncthreads();
    if (dist <= 2 * m && node) {
      NodeIn<L, R> in;
#pragma unroll
      for (int i = 0; i < Q; ++i) {
        const PhiPsi v = ring[own + L::cy[i] * PW + L::cx[i]];
        in.nphi[i] = v.phi;
        in.npsi[i] = v.psi;
      }
      if constexpr (!COUPLED)
        vortex_from_factors<R>(c.np.U0, trig[0][rx], trig[1][rx], trig[0][RX + ry], trig[1][RX + ry],
                               trig[0][RX + RY + n - 1 - m], in.u[0], in.u[1]);
      NodeOut<L, R> out;
      node_update_d2q9<R, COUPLED, St::shifted, UNIT, VISC, !COUPLED>(c.np, in, g, f, J, out);
      S e[4];
      if constexpr (COUPLED) encode_first<St, Once::Level>(f, false, e);
      R res = R(0);   // rounding of the stored g deviations, taken off the stored phi
#pragma unroll
      for (int i = 0; i < Q; ++i) {
        if constexpr (St::shifted)   // relative to the reader's phi (encode_dev)
          g[i] = encode_dev(g[i], c.np.rest[i], in.nphi[0],
                            leaves_through_wall<L>(i, yw, ny, wall) ? in.nphi[0] : in.nphi[i]);
        if constexpr (St::fold) res += St::rounding(g[i]);
      }
      if constexpr (COUPLED) {
        if (wall && yw == 0) {
#pragma unroll
          for (int i = 0; i < Q; ++i)
            if (L::cy[i] < 0) f[i] += c.np.wb[i] * out.rho;
        }
        if (wall && yw == ny - 1) {
#pragma unroll
          for (int i = 0; i < Q; ++i)
            if (L::cy[i] > 0) f[i] += c.np.wt[i] * out.rho;
        }
      }
      auto stored_f = [&](int i) -> S { return encoded_first<St, Once::Level>(i) ? e[i & 3] : St::enc(f[i]); };
      const float own_phi = St::shifted ? float(in.nphi[0] - res) : 0.0f;
      if (m > 0) {
#pragma unroll
        for (int i = 0; i < Q; ++i) {
          pops[0][i][tid] = St::enc(g[i]);
          if constexpr (COUPLED) pops[1][i][tid] = stored_f(i);
        }
        if constexpr (St::shifted) phl[tid] = own_phi;
      } else if (xg < nx && yg < ny) {
#pragma unroll
        for (int i = 0; i < Q; ++i) {
          St::store(c.pop[0][dst] + long(i) * ns, nn, g[i]);
          if constexpr (COUPLED) St::store_s(c.pop[1][dst] + long(i) * ns, nn, stored_f(i));
        }
        stg(c.Jw, nn, J[0]);
        stg(c.Jw + ns, nn, J[1]);
        if constexpr (St::shifted) stg(c.phis[dst], nn, own_phi);
      }
    }
    if (helper && (reduce >> (n - 1 - m) & 1))
      tile2d_sums<TX, TY, PW>(c, ring + (H + 1) * (PW + 1), x0, y0, part + (n - 1 - m) * part_set, part_stride);
    if (m == 0) break;
    __syncthreads();
    if (dist <= 2 * m - 1) {
      // the node's populations, or the edge row's for a ghost past a wall
      const int at = tid + (wall ? RX * (yw - yg) : 0);
#pragma unroll
      for (int i = 0; i < Q; ++i) {
        const bool back = wall && ((yw == 0 && L::cy[i] > 0) || (yw == ny - 1 && L::cy[i] < 0));
        const int k = back ? L::opp[i] : i, from = back ? at : at - L::cx[i] - RX * L::cy[i];
        g[i] = St::dec(pops[0][k][from]);
        if constexpr (COUPLED) f[i] = St::dec(pops[1][k][from]);
        if constexpr (St::shifted) ps[i] = R(phl[at]);
      }
    }
  }
}

}  // namespace vclb
