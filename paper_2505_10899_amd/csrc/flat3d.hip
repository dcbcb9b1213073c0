// One D3Q19 step in two passes over the nodes in stored order, one lane per node.
//
// The section march of kernels3d.hip reads every population once, but its section has to
// fit the grid: rows that do not start on cache lines split every access of a wave, widths
// and heights off the section's leave lanes idle, and a march of a few planes pays a
// memory round trip for each.  Here lane and node number go together: every wave stores
// whole cache lines whatever the widths, and no lane idles.
//   k_pairs3d  forms phi and psi of every node, side by side, and sums the step's volume
//              reductions;
//   k_node3d   updates every node, its 18 neighbours' pairs read through the caches.
// g is read twice and the pairs once each way: 432 instead of 336 bytes a node in FP32,
// 242 instead of 184 in FP16S, 840 instead of 656 in FP64.  Against the march (us a step,
// 36 x 60 x 54 to 113 x 97 x 301 nodes, periodic):
//                      FP64           FP32          FP16S
//   36 x 60 x 54      66 -> 21       62 -> 16       55 -> 15
//   46 x 26 x 265     87 -> 47       61 -> 28       56 -> 23
//   75 x 86 x 348    446 -> 366     252 -> 200     174 -> 132
//   113 x 97 x 301   676 -> 527     430 -> 283     307 -> 191
// A box of nodes per workgroup with its phi and psi in LDS, one pass, was 1-2 us faster on
// grids below 100 k nodes and up to 60% slower above: its halo shell holds as many cells
// as the box has nodes.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "devcase.hpp"
#include "launch.hpp"
#include "step3d.hpp"

namespace vclb {

namespace {
constexpr int kBlock = 256;

// coordinates of node n in stored order (n < 2^31)
struct Node3 {
  int x, y, z;
};
__device__ __forceinline__ Node3 node3(unsigned n, int nx, int ny) {
  const unsigned row = n / unsigned(nx), z = row / unsigned(ny);
  return Node3{int(n - row * unsigned(nx)), int(row - z * unsigned(ny)), int(z)};
}

// a pair as one 2-word access
template <class R>
using Pair = R __attribute__((ext_vector_type(2)));
}  // namespace

// phi and psi of every node of chunk b, and the partial reductions.  The first workgroups
// sum the previous step's partials, a field each.  by_xcd: chunks in XCD-aware order.
template <class St, bool WALL>
__global__ void __launch_bounds__(kBlock) k_pairs3d(DevCase<D3Q19, St> c, long nb, long chunk, int by_xcd, int reduce) {
  using L = D3Q19;
  using R = typename St::R;
  const int extra = c.pend_nb > 0 ? c.nl * 12 : 0;
  if (int(blockIdx.x) < extra) {
    fold_field(c, blockIdx.x / 12, blockIdx.x % 12);
    return;
  }
  const int i = int(blockIdx.x) - extra;
  const long b = by_xcd ? xcd_tile(i, int(nb)) : i;
  auto* pairs = reinterpret_cast<Pair<R>*>(c.tmp_phi);   // two scratch arrays of n, back to back
  const int par = int(c.t & 1);
  Acc acc;
  acc.zero();
  const long hi = min(c.n, (b + 1) * chunk);
#pragma unroll 2
  for (long n = b * chunk + threadIdx.x; n < hi; n += kBlock) {
    const Node3 p = node3(unsigned(n), c.nx, c.ny);
    R g[L::Q], ps[L::Q];
    pull19_ptr<St, unsigned>(c.pop[0][par], c.phis[par], c.ns,
                             nbr3(p.x, p.y, p.z, c.nx, c.ny, c.nz, c.nx * c.ny, WALL && c.wall != 0), g, ps);
    const R ph = phi_of_pulled<L, St>(g, ps, c.np.rest);
    stg(pairs, unsigned(n), Pair<R>{ph, psi_of<R>(ph, c.np.W4, c.np.xi)});
    if (reduce) accumulate(c, acc, double(ph), p.x, p.y, p.z);
  }
  if (reduce) write_partials(acc, c.nl, c.part_w, nb, b);
}

// Waves per SIMD the registers are sized for: 88-100 registers with 4-byte arithmetic and unit
// rates (109-119 with general ones), 150 in FP64, which does not fit 4 waves.  With walls or
// general rates FP64 fills the 168 of 3 waves and spills 2-10 (the march's kernel with walls
// fills 256 and spills 21).  by_xcd: blocks in XCD-aware order; either way the last
// block goes first, where the pass before ended.  NT: population stores with the
// non-temporal hint.
template <class St, bool UNIT, bool VISC, bool WALL, bool NT>
__global__ void __launch_bounds__(kBlock, (sizeof(typename St::R) == 8 ? 3 : 4))
    k_node3d(DevCase<D3Q19, St> c, int by_xcd) {
  using L = D3Q19;
  using R = typename St::R;
  using IX = unsigned;
  constexpr int Q = L::Q;
  // APART: sums as the march's compiled form has them in FP32, whose one kernel tests for walls:
  // grad phi with each product made once, fused into the first component that takes it, and g's
  // inverse transform with its products rounded (bit for bit the march's results).
  constexpr bool APART = sizeof(typename St::S) == 4;
  // AHEAD: the pairs are requested before the sums over them, like the populations.  Without,
  // the compiler waits for them one after the other where the sums are spelled out (FP16S
  // periodic, 128 x 128 x 200: 187 -> 172 us, with general rates 206 -> 173) or walls stand
  // between them (FP32, 61 x 45 x 130: 34.3 -> 31.8).
  constexpr bool AHEAD = sizeof(typename St::S) == (WALL ? 4 : 2);
  const int last = int(gridDim.x) - 1 - int(blockIdx.x);
  const unsigned n = unsigned(by_xcd ? xcd_tile(last, gridDim.x) : last) * kBlock + threadIdx.x;
  if (long(n) >= c.n) return;
  const int nx = c.nx, ny = c.ny, nz = c.nz;
  const Node3 p = node3(n, nx, ny);
  const bool wall = WALL && c.wall != 0;
  const int par = int(c.t & 1), dst = par ^ 1;
  const Nbr3 o = nbr3(p.x, p.y, p.z, nx, ny, nz, nx * ny, wall);
  R g[Q], ps[Q], f[Q], J[L::D];
  pull19_ptr<St, IX>(c.pop[0][par], c.phis[par], c.ns, o, g, ps);
  pull19_ptr<St, IX>(c.pop[1][par], c.phis[par], c.ns, o, f, nullptr);
#pragma unroll
  for (int d = 0; d < L::D; ++d) J[d] = ldg(c.J + d * c.ns, n);
  // stencils of Eqs. 39-40 over the neighbours' pairs
  const auto* pairs = reinterpret_cast<const Pair<R>*>(c.tmp_phi);
  auto pair_of = [&](auto I) {
    constexpr int i = decltype(I)::value;
    int m = o.s0;
    if constexpr (L::cx[i] > 0) m += o.xp;
    if constexpr (L::cx[i] < 0) m += o.xm;
    if constexpr (L::cz[i] > 0) m += o.zp;
    if constexpr (L::cz[i] < 0) m += o.zm;
    if constexpr (L::cy[i] > 0) m += o.hi ? 0 : o.yp;
    if constexpr (L::cy[i] < 0) m += o.lo ? 0 : o.ym;
    return ldg(pairs, unsigned(m));
  };
  Pair<R> pre[AHEAD ? Q : 1];
  if constexpr (AHEAD) {
    static_for<1, Q>([&](auto I) { pre[decltype(I)::value] = pair_of(I); });
    __builtin_amdgcn_sched_barrier(0);
  }
  R nphi[Q];
  StencilOut<L, R> st;
  st.phi = nphi[0] = ldg(pairs, n).x;
  st.lap = R(0);
#pragma unroll
  for (int d = 0; d < 3; ++d) st.gphi[d] = st.gpsi[d] = R(0);
  static_for<1, Q>([&](auto I) {
    constexpr int i = decltype(I)::value;
    Pair<R> v;
    if constexpr (AHEAD) v = pre[i];
    else v = pair_of(I);
    if constexpr (WALL && L::cy[i] != 0) {   // behind a wall: the edge row's wetting ghost
      if (L::cy[i] > 0 ? o.hi : o.lo) {
        v.x = wet_ghost<R>(v.x, L::cy[i] > 0 ? c.np.wet_hi : c.np.wet_lo);
        v.y = psi_of<R>(v.x, c.np.W4, c.np.xi);
      }
    }
    nphi[i] = v.x;
    constexpr int cc[3] = {L::cx[i], L::cy[i], L::cz[i]};
    if constexpr (APART) {
      st.lap = fma_of(R(6.0 * L::w[i]), v.x - st.phi, st.lap);
      constexpr int lead = cc[0] != 0 ? 0 : cc[1] != 0 ? 1 : 2;
#pragma unroll
      for (int d = 0; d < 3; ++d)
        if (cc[d] != 0) {
          const R a = R(3.0 * L::w[i] * cc[d]);
          st.gphi[d] = d == lead ? fma_of(a, v.x, st.gphi[d]) : st.gphi[d] + rounded(a * v.x);
          st.gpsi[d] = fma_of(a, v.y, st.gpsi[d]);
        }
    } else {
      st.lap += R(6.0 * L::w[i]) * (v.x - st.phi);
#pragma unroll
      for (int d = 0; d < 3; ++d)
        if (cc[d] != 0) {
          st.gphi[d] += R(3.0 * L::w[i] * cc[d]) * v.x;
          st.gpsi[d] += R(3.0 * L::w[i] * cc[d]) * v.y;
        }
    }
  });
  (void)phi_of_pulled<L, St>(g, ps, c.np.rest);
  NodeOut<L, R> out;
  node_update_mom_s<L, R, true, St::shifted, UNIT, VISC, true, APART>(c.np, st, g, f, J, out);
  // with walls the march adds the wall terms to f, and converts it, in other blocks than those
  // that form it
  if constexpr (WALL && sizeof(R) == 4) {
#pragma unroll
    for (int i = 0; i < Q; ++i) f[i] = formed(f[i]);
  }
  R res = R(0);   // rounding of the stored g deviations, taken off the stored phi
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    R e = g[i];
    if constexpr (St::shifted)   // relative to the reader's phi (encode_dev)
      e = encode_dev(g[i], c.np.rest[i], st.phi, leaves_through_wall<L>(i, p.y, ny, wall) ? st.phi : nphi[i]);
    if constexpr (NT) St::store_nt(c.pop[0][dst] + i * c.ns, n, e);
    else St::store(c.pop[0][dst] + i * c.ns, n, e);
    if constexpr (St::fold) res += St::rounding(e);
  }
  if (wall && p.y == 0) {   // moving-wall term of the populations the bottom wall returns
#pragma unroll
    for (int i = 0; i < Q; ++i)
      if (L::cy[i] < 0) f[i] += c.np.wb[i] * out.rho;
  }
  if (wall && p.y == ny - 1) {
#pragma unroll
    for (int i = 0; i < Q; ++i)
      if (L::cy[i] > 0) f[i] += c.np.wt[i] * out.rho;
  }
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    if constexpr (NT) St::store_nt(c.pop[1][dst] + i * c.ns, n, f[i]);
    else St::store(c.pop[1][dst] + i * c.ns, n, f[i]);
  }
#pragma unroll
  for (int d = 0; d < L::D; ++d) stg(c.J + d * c.ns, n, J[d]);
  if constexpr (St::shifted) stg(c.phis[dst], n, float(st.phi - res));
}

template <class St>
int launch_flat3d(const DevCase<D3Q19, St>& c, int reduce, hipStream_t s) {
  // While both population sets fit the 256 MB last-level cache: XCD-aware order, so that
  // an XCD's L2 holds the planes its blocks share (46 x 26 x 265 FP64 52 -> 47 us), and
  // plain stores (with the hint 59).  Beyond: linear order, so that the second pass, which
  // goes backwards, finds the g and pairs that the first read and wrote last, and the hint
  // on stores that are not read back before they are evicted (113 x 97 x 301 FP64 568 -> 527,
  // FP32 303 -> 283).
  const bool cached = size_t(c.ns) * 19 * 4 * sizeof(typename St::S) <= (size_t(256) << 20);
  const long chunk = flat3d_chunk(c.n), nb = (c.n + chunk - 1) / chunk;
  const dim3 grid1(unsigned(nb + (c.pend_nb > 0 ? c.nl * 12 : 0))), grid2(unsigned((c.n + kBlock - 1) / kBlock));
  const int xcd = cached ? 1 : 0;
  auto go = [&](auto unit, auto visc, auto wall) {
    constexpr bool U = decltype(unit)::value, V = decltype(visc)::value, W = decltype(wall)::value;
    hipLaunchKernelGGL((k_pairs3d<St, W>), grid1, dim3(kBlock), 0, s, c, nb, chunk, xcd, reduce);
    if (cached) hipLaunchKernelGGL((k_node3d<St, U, V, W, false>), grid2, dim3(kBlock), 0, s, c, xcd);
    else hipLaunchKernelGGL((k_node3d<St, U, V, W, true>), grid2, dim3(kBlock), 0, s, c, xcd);
  };
  auto pick_wall = [&](auto unit, auto visc) {
    if (c.wall) go(unit, visc, std::true_type{});
    else go(unit, visc, std::false_type{});
  };
  auto pick_visc = [&](auto unit) {
    if (c.visc) pick_wall(unit, std::true_type{});
    else pick_wall(unit, std::false_type{});
  };
  if (c.unit_rates) pick_visc(std::true_type{});
  else pick_visc(std::false_type{});
  return hipGetLastError() == hipSuccess ? 0 : -3;
}

template int launch_flat3d<StoreF64>(const DevCase<D3Q19, StoreF64>&, int, hipStream_t);
template int launch_flat3d<StoreF32>(const DevCase<D3Q19, StoreF32>&, int, hipStream_t);
template int launch_flat3d<StoreF16S>(const DevCase<D3Q19, StoreF16S>&, int, hipStream_t);

}  // namespace vclb
