"""D3Q19 cases stepped in two passes in stored order (flat3d.hip): one step from the oracle's
state against the oracle's own step, and the recorded reductions, at sizes around the
blocks of 256 nodes (one block, a ragged last block, one node more than a block) and on
either side of the 256 MB cache rule (81^3 in FP64: chunks of four nodes a lane, linear
order, non-temporal stores).

Tolerances, set before the first run: those of the 2D lane tiles (test_gpu_lane_tiles.py):
FP64 1e-13 and FP32 1e-6 plus the conditioning bound of the unit normal; FP16S against
the plain path within one spacing of its stored deviations, 2^-15, plus 2e-6."""
import numpy as np
import pytest

import workloads as W
from oracle.model import Model, observables_from_phi

from test_gpu_parity import normal_conditioning

pytestmark = pytest.mark.gpu

SMALL = [(8, 8, 4), (257, 1, 1), (5, 3, 17), (3, 2, 4), (17, 19, 9), (33, 8, 12)]
CASES = [(s, st, wall, 3.75 if k % 2 else 1.0, 1 + k % 2) for k, s in enumerate(SMALL)
         for st in ("fp64", "fp32", "fp16s") for wall in (False, True) if not (wall and s[1] < 2)]
CASES += [((81, 81, 81), "fp64", False, 1.0, 1), ((81, 81, 81), "fp32", True, 1.0, 2)]
IDS = ["%dx%dx%d-%s-%s-%g-%d" % (*c[0], c[1], "w" if c[2] else "p", *c[3:]) for c in CASES]


@pytest.mark.parametrize("size,storage,wall,visc,nl", CASES, ids=IDS)
def test_one_step_and_reductions(size, storage, wall, visc, nl):
    from paper_2505_10899_amd import vclb as v
    nx, ny, nz = size
    print("case:", size, storage, wall, visc, nl, flush=True)
    c1 = (0.31 * nx + 0.13, 0.47 * ny + 0.21, 0.37 * nz + 0.17)
    c2 = (0.73 * nx + 0.07, 0.52 * ny + 0.11, 0.71 * nz + 0.09)
    p = W.CaseParams(nx=nx, ny=ny, nz=nz, lattice="D3Q19", wall_y=wall, rho_light=0.2, label_centres=[c1, c2][:nl])
    if wall:
        p = p.replace(wall_u_bottom=(-0.02, 0.0, 0.01), wall_u_top=(0.015, 0.0, 0.0), wall_cos_bottom=0.4,
                      wall_cos_top=-0.3)
    if visc != 1.0:
        p = p.replace(nu_light=p.nu * visc)
    m_ = min(nx, ny, nz)
    phi0 = np.clip(W.drops_phi(p, [(*c1, min(16.0, max(1.5, 0.3 * m_))), (*c2, min(10.0, max(1.0, 0.2 * m_)))]), 0.0, 1.0)
    m = Model(p).init(phi0, W.couette_u(p) if wall else None)
    m.step(1)
    c = v.Case(p.replace(storage=storage))
    c.set_state(m.g, m.f, m.Jprev, m.t)
    field = lambda: observables_from_phi(p, c.observe(v.FIELD_PHI)["phi"])
    obs = [field()]
    if storage == "fp16s":
        d = v.Case(p.replace(storage=storage))
        d.set_state(m.g, m.f, m.Jprev, m.t)
        c.step(1)
        d.step_plain(1)
        for a, b in zip(c.get_state(), d.get_state()):
            assert float(np.max(np.abs(a - b))) <= 2.0 ** -15 + 2e-6
    else:
        base, eps = (1e-13, 2.2e-16) if storage == "fp64" else (1e-6, 6e-8)
        tol = base + 2.0 * normal_conditioning(m, m.fields(), eps=eps)
        c.step(1)
        m.step(1)
        g, f, J = c.get_state()
        assert float(np.max(np.abs(g - m.g) / tol[None])) <= 1.0
        assert float(np.max(np.abs(f - m.f) / tol[None])) <= 1.0
        assert float(np.max(np.abs(J - m.Jprev))) <= base
    obs.append(field())
    c.step(1)                                   # its first pass sums the first step's partials
    h = c.history(1, 2)
    rtol = {"fp64": 1e-12, "fp32": 2e-6, "fp16s": 2e-4}[storage]
    scale = {"sum_phi": 1.0, "sum_phi_d": max(size), "sum_phi_dd": max(size) ** 2}
    for t in range(2):
        total = np.abs(obs[t]["sum_phi"]).sum() + 1.0
        for k, s in scale.items():
            assert float(np.max(np.abs(h[k][t] - obs[t][k]))) <= rtol * s * total, (t, k)
        assert not h["nonfinite"].any()


@pytest.mark.parametrize("which", ["below_2GiB", "above_2GiB"])
def test_the_march_either_side_of_the_buffer_limit(which, monkeypatch):
    """FP16S columns step in two passes by default; the section march that set_tile chooses
    still changes its form of access at arrays of 2 GiB."""
    import test_gpu_max_size as M
    from paper_2505_10899_amd import vclb

    class March(vclb.Case):
        def __init__(self, *a, **k):
            super().__init__(*a, **k)
            self.set_tile(32, 19, 8)

    monkeypatch.setattr(vclb, "Case", March)
    M.test_d3q19_fp16s_either_side_of_the_buffer_limit(which)
