// One D2Q9 step with one lane per node: the step of single cases whose grid does not keep
// the row march of step2d.hpp busy.
//
// A march hides its memory round trips behind the rows that follow; a grid of a few
// hundred thousand nodes leaves each workgroup only a handful of rows, and the step then
// costs that many round trips in a row.  Here a workgroup owns a tile of 2^lx x 2^ly
// nodes, every lane requests all populations of its node and its share of the halo ring's
// g at once, phi and psi go to LDS, and after one barrier every lane updates its node: one
// round trip per step, and with nothing carried from row to row 54 registers in FP32 and
// 92 in FP64, so that 8 and 5 waves per SIMD hide it.  Measured per step, march against
// tiles, with the reductions:
//   66 x 24 FP32 (walls)   29 -> 4.9 us      128 x 128 FP64   31 -> 5.9 us
//   512 x 256 FP64         47 -> 9.7 us      777 x 1333 FP32  62 -> 30 us (36.7 GLUPS)
//   1501 x 1003 FP16S      40 -> 29 us       2048 x 2048 FP64 275 -> 248 us
// Small tiles are bound by the chain of one launch: dispatch, pull, stencil, update, store
// (about 5 us); large ones by memory.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "devcase.hpp"
#include "flat2d.hpp"
#include "launch.hpp"

namespace vclb {

// LX, LY: log2 of the tile's sides.  HELP: one more wave, which pulls the first 64 halo cells and
// sums the tile's reductions while the others update.  That takes both off the critical
// path of a step that waits for one launch (128 x 128 FP64: 7.4 -> 5.9 us, of which the
// reductions now cost 0.6), but a wave in three idles; large grids, which need every wave
// (1501 x 1003 FP16S: 27.7 -> 31.3 us), leave both to the tile's own lanes.
// NT: stores of the populations and loads of f with the non-temporal hint.
template <class St, bool COUPLED, bool UNIT, bool VISC, int LX, int LY, bool HELP, bool NT>
__global__ void __launch_bounds__((1 << (LX + LY)) + (HELP ? 64 : 0))
    k_tile2d(DevCase<D2Q9, St> c, int ntx, int ntiles, int reduce) {
  using L = D2Q9;
  using R = typename St::R;
  using S = typename St::S;
  constexpr int Q = 9;
  // fields of the observation that are not zero in 2D (the others are z moments)
  constexpr int kFields = 8;
  constexpr int field[kFields] = {0, 1, 2, 3, 5, 6, 8, 11};
  // the first workgroups sum the previous step's partials beside the tiles, a field each:
  // one workgroup for all fields was still at it when the tiles were done
  const int extra = c.pend_nb > 0 ? c.nl * kFields : 0;
  if (int(blockIdx.x) < extra) {
    const int k = blockIdx.x / kFields, j = blockIdx.x % kFields;
    fold_field(c, k, field[j]);
    if (j == 0 && threadIdx.x < 4) {
      constexpr int zero[4] = {4, 7, 9, 10};
      c.pend_dest[k * kObsFields + zero[threadIdx.x]] = 0.0;
    }
    return;
  }
  struct alignas(2 * sizeof(R)) PhiPsi {
    R phi, psi;
  };
  constexpr int TX = 1 << LX, TY = 1 << LY, PW = TX + 2, nodes = TX * TY;
  constexpr int nring = 2 * PW + 2 * TY;   // halo cells
  static_assert(nring <= nodes && nodes % 64 == 0, "a halo cell per lane");
  __shared__ PhiPsi ring[PW * (TY + 2)];   // the tile and its halo
  const int tile = xcd_tile(int(blockIdx.x) - extra, ntiles);
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
  const int par = int(c.t & 1), dst = par ^ 1;
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
    else if (tid == TX + TY) trig[0][tid] = vortex_phase<R>(c.np.T, c.t);
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
    node_update_d2q9<R, COUPLED, St::shifted, UNIT, VISC>(c.np, in, g, f, J, out);
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
      for (int i = 0; i < Q; ++i) {
        if constexpr (NT) St::store_nt(c.pop[1][dst] + long(i) * ns, nn, f[i]);
        else St::store(c.pop[1][dst] + long(i) * ns, nn, f[i]);
      }
    }
    stg(c.J, nn, J[0]);
    stg(c.J + ns, nn, J[1]);
    if constexpr (St::shifted) stg(c.phis[dst], nn, float(in.nphi[0] - res));
  }
  // this tile's volume reductions, by one wave from the ring's phi: the helper, or the last
  // wave (the first ones pull the halo).  Six sums over the wave once per tile instead of
  // once per wave: 1501 x 1003 FP16S 34.9 -> 27.7 us.
  if (!reduce || tid < (HELP ? nodes : nodes - 64)) return;
  // A lane keeps to a column (or two, TX = 128), so only phi, phi dy, phi dy^2 add up per
  // node and the x moments follow.
  const int lane = tid & 63;
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
      const double ph = x < nx && y < ny ? double(ring[(ry + 1) * PW + rx + 1].phi) : 0.0;
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
      double* p = c.part_w + tile;
      // fields: sum, count, x, y, z, xx, yy, zz, xy, xz, yz, not finite
      const int fa = i == 0 ? 0 : (i == 1 ? 2 : (i == 2 ? 3 : 5)), fb = i == 0 ? 6 : (i == 1 ? 8 : (i == 2 ? 1 : 11));
      const int fz = i == 0 ? 4 : (i == 1 ? 7 : (i == 2 ? 9 : 10));
      stg(p, long(k * 12 + fa) * ntiles, a);
      stg(p, long(k * 12 + fb) * ntiles, b);
      stg(p, long(k * 12 + fz) * ntiles, 0.0);
    }
  }
}

template <class St, bool COUPLED>
int launch_tile2d(const DevCase<D2Q9, St>& c, int lx, int ly, int reduce, hipStream_t s) {
  if (!tile2d_shape_ok(lx, ly)) return -1;
  const int ntx = (c.nx + (1 << lx) - 1) >> lx, nty = (c.ny + (1 << ly) - 1) >> ly;
  const int ntiles = ntx * nty, lanes = 1 << (lx + ly);
  const bool help = tile2d_helper(lx, ly);
  // the non-temporal hint where it pays: rows of whole cache lines (every store of a wave
  // fills its lines; else the hint evicts lines that the next tile completes, 2951 x 2937
  // FP32 348 -> 420 us) of grids whose two population sets exceed the 256 MB last-level
  // cache (2048 x 2048 FP32 145 -> 131, FP64 268 -> 248; within it 1024 x 1024 FP32 29.5 -> 43)
  const size_t set = size_t(c.ns) * 9 * sizeof(typename St::S) * (COUPLED ? 4 : 2);
  const bool nt = lx == 7 && size_t(c.nx) * sizeof(typename St::S) % 128 == 0 && set > (size_t(256) << 20);
  const dim3 grid(unsigned(ntiles + (c.pend_nb > 0 ? c.nl * 8 : 0))), block(unsigned(lanes + (help ? 64 : 0)));
  auto go = [&](auto unit, auto visc) {
    constexpr bool U = decltype(unit)::value, V = decltype(visc)::value;
    auto run = [&](auto kern) { hipLaunchKernelGGL(kern, grid, block, 0, s, c, ntx, ntiles, reduce); };
    if (help) run(k_tile2d<St, COUPLED, U, V, 4, 3, true, false>);
    else if (lx == 6) run(k_tile2d<St, COUPLED, U, V, 6, 2, false, false>);
    else if (nt) run(k_tile2d<St, COUPLED, U, V, 7, 2, false, true>);
    else run(k_tile2d<St, COUPLED, U, V, 7, 2, false, false>);
  };
  auto pick_visc = [&](auto unit) {
    if constexpr (COUPLED) {
      if (c.visc) {
        go(unit, std::true_type{});
        return;
      }
    }
    go(unit, std::false_type{});
  };
  if (c.unit_rates) pick_visc(std::true_type{});
  else pick_visc(std::false_type{});
  return hipGetLastError() == hipSuccess ? 0 : -3;
}

template int launch_tile2d<StoreF64, true>(const DevCase<D2Q9, StoreF64>&, int, int, int, hipStream_t);
template int launch_tile2d<StoreF64, false>(const DevCase<D2Q9, StoreF64>&, int, int, int, hipStream_t);
template int launch_tile2d<StoreF32, true>(const DevCase<D2Q9, StoreF32>&, int, int, int, hipStream_t);
template int launch_tile2d<StoreF32, false>(const DevCase<D2Q9, StoreF32>&, int, int, int, hipStream_t);
template int launch_tile2d<StoreF16S, true>(const DevCase<D2Q9, StoreF16S>&, int, int, int, hipStream_t);
template int launch_tile2d<StoreF16S, false>(const DevCase<D2Q9, StoreF16S>&, int, int, int, hipStream_t);

}  // namespace vclb
