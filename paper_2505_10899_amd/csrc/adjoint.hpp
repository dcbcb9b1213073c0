// Buffers and launchers of the FP64 D2Q9 adjoint (adjoint.hip).
#pragma once
#include <hip/hip_runtime.h>

#include "devcase.hpp"

namespace vclb {

constexpr int kSeedFields = 10;   // per label: sum, d[3], dd[6] (xx, yy, zz, xy, xz, yz)

// Device buffers of one backward sweep, each N-major ([component][node]).
struct AdjArgs {
  const double* lg_in;    // [9][N] lg of step t + 1
  const double* lf_in;    // [9][N]
  const double* lJ_in;    // [2][N]
  double* lg_out;         // [9][N] lg of step t
  double* lf_out;         // [9][N]
  double* lJ_out;         // [2][N]
  double* lphi;           // [N] adjoint of phi: the seed's, and that of the first step
  const double* aux_in;   // [7][N] stencil-input adjoints of step t + 1, and its phi
  double* aux_out;        // [7][N] the same of step t
  double* param_part;     // [2][part_slots] running (dJ/dsigma, dJ/dM) per workgroup
  long part_slots;
  const double* seed;     // [labels][kSeedFields] device copy of the moment weights
  double beta4_per_sigma;   // 4 beta / sigma = 48 / W
  double kappa_per_sigma;   // kappa / sigma = 3 W / 2
  unsigned mobility_rows;   // bit k: s_k^g is the default 1 / tau_g
  double normal_tau2;       // n is held fixed (no derivative) where |grad psi|^2 < normal_tau2
};

long adj_part_slots(int nx, int ny);
int launch_adj_zero(double* p, long count, hipStream_t s);
int launch_adj_seed(const DevCase<D2Q9, StoreF64>& c, const AdjArgs& a, hipStream_t s);
// one backward step (first: the last step of the run, from the seed); the lphi its aux stands for
int launch_adj_step(const DevCase<D2Q9, StoreF64>& c, const AdjArgs& a, bool first, hipStream_t s);
int launch_adj_stencil(const DevCase<D2Q9, StoreF64>& c, const AdjArgs& a, hipStream_t s);
int launch_adj_init(const DevCase<D2Q9, StoreF64>& c, const AdjArgs& a, const double* phi0, const double* u0,
                    double* dphi0, hipStream_t s);
int launch_adj_params(const AdjArgs& a, double* out, hipStream_t s);

}  // namespace vclb
