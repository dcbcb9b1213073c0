// D2Q9 steps with one lane per node: the step of single cases whose grid does not keep the
// row march of step2d.hpp busy, and of batches of few nodes.
//
// A march hides its memory round trips behind the rows that follow; a grid of a few
// hundred thousand nodes leaves each workgroup only a handful of rows, and the step then
// costs that many round trips in a row.  Here a workgroup owns a tile of 2^lx x 2^ly
// nodes, every lane requests all populations of its node and its share of the halo ring's
// g at once, phi and psi go to LDS, and after one barrier every lane updates its node: one
// round trip per step, and with nothing carried from row to row 50-66 registers in FP32 and
// 78-96 in FP64, so that 7-8 and 5-6 waves per SIMD hide it.  On the smallest grids, where the
// chain of a launch (dispatch, pull, stencil, update, store: 5 us) is nearly all of a step,
// a launch takes three (tile2d_multi).  Measured per step, march against tiles, with the
// reductions:
//   66 x 24 FP32 (walls)   29 -> 4.7 us, in threes 2.7
//   128 x 128 FP64         31 -> 5.2, in threes 3.6
//   256 x 256 FP64 vortex  32 -> 6.4, in threes 4.5
//   512 x 256 FP64         47 -> 9.5 us      777 x 1333 FP32  62 -> 29 us (36 GLUPS)
//   1501 x 1003 FP16S      40 -> 28 us       2048 x 2048 FP64 275 -> 246 us
// Large ones are bound by memory.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "devcase.hpp"
#include "launch.hpp"
#include "tile2d.hpp"

namespace vclb {

template <class St, bool COUPLED, bool UNIT, bool VISC, int LX, int LY, bool HELP, bool NT>
__global__ void __launch_bounds__(tile2d_lanes(LX, LY, HELP))
    k_tile2d(DevCase<D2Q9, St> c, int ntx, int ntiles, int reduce) {
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
  const int tile = xcd_tile(int(blockIdx.x) - extra, ntiles);
  tile2d_step<St, COUPLED, UNIT, VISC, LX, LY, HELP, NT, Once::Level>(c, c.t, tile, ntx,
                                                                      reduce ? c.part_w + tile : nullptr, ntiles, false);
}

// Up to three steps in one launch (tile2d_multi).  As above, the first workgroups sum the
// partials of the launch before, of one step or of up to three.
template <class St, bool COUPLED, bool UNIT, bool VISC, int LX, int LY>
__global__ void __launch_bounds__(tile2d_multi_lanes(LX, LY))
    k_tile2d_multi(DevCase<D2Q9, St> c, int ntx, int ntiles, int reduce) {
  constexpr int kFields = 8;
  constexpr int field[kFields] = {0, 1, 2, 3, 5, 6, 8, 11};
  const int per_set = c.nl * kFields;
  const int extra = c.pend_nb > 0 ? per_set * (c.pend_mask > 1 ? kMultiSteps : 1) : 0;
  if (int(blockIdx.x) < extra) {
    const int set = blockIdx.x / per_set, b = blockIdx.x - set * per_set;
    if (!(c.pend_mask >> set & 1)) return;
    const int k = b / kFields, j = b % kFields;
    const long step = c.pend_step + set;
    double* dest = c.hist + (step % kHistory) * c.nl * kObsFields;
    fold_field(c.part_r + long(set) * c.nl * 12 * c.pend_nb, c.pend_nb, dest, step, k, field[j]);
    if (j == 0 && threadIdx.x < 4) {
      constexpr int zero[4] = {4, 7, 9, 10};
      dest[k * kObsFields + zero[threadIdx.x]] = 0.0;
    }
    return;
  }
  const int tile = xcd_tile(int(blockIdx.x) - extra, ntiles);
  tile2d_multi<St, COUPLED, UNIT, VISC, LX, LY>(c, c.t, c.steps, tile, ntx, reduce, c.part_w + tile, ntiles,
                                                long(c.nl) * 12 * ntiles);
}

template <class St, bool COUPLED>
int launch_tile2d(const DevCase<D2Q9, St>& c, int lx, int ly, int reduce, hipStream_t s) {
  using R = typename St::R;
  if (!tile2d_shape_ok(lx, ly) || (lx == 4 && ly == 4 && COUPLED && sizeof(R) == 8)) return -1;
  const int ntx = (c.nx + (1 << lx) - 1) >> lx, nty = (c.ny + (1 << ly) - 1) >> ly;
  const int ntiles = ntx * nty, lanes = 1 << (lx + ly);
  const bool help = tile2d_helper(lx, ly);
  // the non-temporal hint where it pays: rows of whole cache lines (every store of a wave
  // fills its lines; else the hint evicts lines that the next tile completes, 2951 x 2937
  // FP32 348 -> 420 us) of grids whose two population sets exceed the 256 MB last-level
  // cache (2048 x 2048 FP32 145 -> 131, FP64 268 -> 246; within it 1024 x 1024 FP32 29.5 -> 43)
  const size_t set = size_t(c.ns) * 9 * sizeof(typename St::S) * (COUPLED ? 4 : 2);
  const bool nt = lx == 7 && size_t(c.nx) * sizeof(typename St::S) % 128 == 0 && set > (size_t(256) << 20);
  const int sets = c.pend_mask > 1 ? kMultiSteps : 1;
  const dim3 grid(unsigned(ntiles + (c.pend_nb > 0 ? c.nl * 8 * sets : 0)));
  const dim3 block(unsigned(tile2d_multi_ok(lx, ly) ? tile2d_multi_lanes(lx, ly) : lanes + (help ? 64 : 0)));
  auto go = [&](auto unit, auto visc) {
    constexpr bool U = decltype(unit)::value, V = decltype(visc)::value;
    auto run = [&](auto kern) { hipLaunchKernelGGL(kern, grid, block, 0, s, c, ntx, ntiles, reduce); };
    constexpr bool kWide = !COUPLED || sizeof(R) == 4;   // LDS of 16 x 16 tiles
    if (lx == 3) run(k_tile2d_multi<St, COUPLED, U, V, 3, 3>);
    else if (lx == 4 && ly == 4) run(k_tile2d_multi<St, COUPLED, U, V, kWide ? 4 : 3, kWide ? 4 : 3>);
    else if (help) run(k_tile2d<St, COUPLED, U, V, 4, 3, true, false>);
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

// One step of every case of a batch in lane tiles: workgroup i does tile tiles[i].y of case
// tiles[i].x (the tile's complement for a case that runs would do in bands), after one workgroup per case that sums the previous step's partials.
template <class St, bool UNIT, bool VISC, int LX, int LY, bool HELP>
__global__ void __launch_bounds__(tile2d_lanes(LX, LY, HELP))
    k_batch_tile2d(const DevCase<D2Q9, St>* __restrict__ cases, BatchArgs a) {
  const int extra = a.pend ? a.ncases : 0;
  if (int(blockIdx.x) < extra) {
    fold_case(cases[blockIdx.x], a, blockIdx.x);
    return;
  }
  const int i = xcd_tile(int(blockIdx.x) - extra, a.ntiles);
  const int2 w = a.tiles[i];
  const DevCase<D2Q9, St>& c = cases[w.x];
  tile2d_step<St, true, UNIT, VISC, LX, LY, HELP, false, Once::OfBand>(
      c, a.t, w.y < 0 ? ~w.y : w.y, (c.nx + (1 << LX) - 1) >> LX, a.reduce ? a.part_w + i : nullptr, a.nitems, w.y < 0);
}

template <class St>
int launch_batch_tile2d(const void* cases, const BatchArgs& a, int lx, int ly, hipStream_t s) {
  const auto* cs = static_cast<const DevCase<D2Q9, St>*>(cases);
  if (lx != 4 || ly != 3) return -1;
  const dim3 grid(unsigned(a.ntiles + (a.pend ? a.ncases : 0))), block(tile2d_lanes(4, 3, true));
  auto by_tile = [&](auto unit, auto visc) {
    hipLaunchKernelGGL((k_batch_tile2d<St, decltype(unit)::value, decltype(visc)::value, 4, 3, true>), grid, block, 0,
                       s, cs, a);
  };
  auto by_visc = [&](auto unit) {
    if (a.visc) by_tile(unit, std::true_type{});
    else by_tile(unit, std::false_type{});
  };
  if (a.unit) by_visc(std::true_type{});
  else by_visc(std::false_type{});
  return hipGetLastError() == hipSuccess ? 0 : -3;
}
template int launch_batch_tile2d<StoreF64>(const void*, const BatchArgs&, int, int, hipStream_t);
template int launch_batch_tile2d<StoreF32>(const void*, const BatchArgs&, int, int, hipStream_t);
template int launch_batch_tile2d<StoreF16S>(const void*, const BatchArgs&, int, int, hipStream_t);

template int launch_tile2d<StoreF64, true>(const DevCase<D2Q9, StoreF64>&, int, int, int, hipStream_t);
template int launch_tile2d<StoreF64, false>(const DevCase<D2Q9, StoreF64>&, int, int, int, hipStream_t);
template int launch_tile2d<StoreF32, true>(const DevCase<D2Q9, StoreF32>&, int, int, int, hipStream_t);
template int launch_tile2d<StoreF32, false>(const DevCase<D2Q9, StoreF32>&, int, int, int, hipStream_t);
template int launch_tile2d<StoreF16S, true>(const DevCase<D2Q9, StoreF16S>&, int, int, int, hipStream_t);
template int launch_tile2d<StoreF16S, false>(const DevCase<D2Q9, StoreF16S>&, int, int, int, hipStream_t);

}  // namespace vclb
