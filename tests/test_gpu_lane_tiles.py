"""Single 2D cases stepped with one lane per node (tile2d.hip): one step from the oracle's
state against the oracle's own step, and the recorded reductions, at the edges of the
tiles (16 x 8 with a helper wave, 64 x 4, 128 x 4 plain and with the non-temporal hint).

Tolerances, set before the first run: FP64 populations 1e-13 plus the conditioning bound of
the unit normal, FP32 the same at FP32's unit round-off with a base of 1e-6 (both as in the
one-step checks of test_gpu_parity.py).  FP16S stores deviations below 2^-4 whose spacing
is 2^-15 at most: against the plain path, one spacing plus the paths' 2e-6."""
import numpy as np
import pytest

import workloads as W
from oracle.model import Model, observables_from_phi

from test_gpu_parity import normal_conditioning

pytestmark = pytest.mark.gpu

# nx, ny, storage, walls, mode, viscosity ratio, labels
SMALL = [(16, 8), (17, 9), (15, 7), (32, 24), (5, 3), (2, 3), (1, 9), (130, 3), (37, 70)]
CASES = [(nx, ny, st, wall, "coupled", 3.75 if k % 3 == 0 else 1.0, 1 + k % 2)
         for k, (nx, ny) in enumerate(SMALL) for st in ("fp64", "fp32", "fp16s") for wall in (False, True)]
CASES += [(70, 33, st, False, "vortex", 1.0, 1) for st in ("fp64", "fp32", "fp16s")]
CASES += [(1031, 523, "fp32", True, "coupled", 1.0, 2),      # 64 x 4, ragged
          (1024, 515, "fp64", False, "coupled", 3.75, 1),
          (1003, 527, "fp64", False, "vortex", 1.0, 1),
          (1021, 1033, "fp64", True, "coupled", 1.0, 1),     # 128 x 4
          (1024, 1027, "fp64", False, "coupled", 1.0, 2)]    # 128 x 4, non-temporal
TEST_IDS = ["%dx%d-%s-%s-%s-%g-%d" % (c[0], c[1], c[2], "w" if c[3] else "p", *c[4:]) for c in CASES]


def _case(nx, ny, storage, wall, mode, visc, nl):
    m = min(nx, ny)
    c1, c2 = (0.31 * nx + 0.13, 0.47 * ny + 0.21, 0.0), (0.73 * nx + 0.07, 0.52 * ny + 0.11, 0.0)
    p = W.CaseParams(nx=nx, ny=ny, storage="fp64", wall_y=wall, mode=mode, rho_light=0.2,
                     label_centres=[c1, c2][:nl])
    if wall:
        p = p.replace(wall_u_bottom=(-0.02, 0.0, 0.0), wall_u_top=(0.015, 0.0, 0.0), wall_cos_bottom=0.4,
                      wall_cos_top=-0.3)
    if visc != 1.0:
        p = p.replace(nu_light=p.nu * visc)
    if mode == "vortex":
        p = p.replace(U0=0.04, T=400.0, mobility=0.02)
    phi0 = W.drops_phi(p, [(*c1, min(20.0, max(1.5, 0.2 * m))), (*c2, min(12.0, max(1.0, 0.1 * m)))])
    return p, np.clip(phi0, 0.0, 1.0), (W.couette_u(p) if wall else None)


@pytest.mark.parametrize("nx,ny,storage,wall,mode,visc,nl", CASES, ids=TEST_IDS)
def test_one_step_and_reductions(nx, ny, storage, wall, mode, visc, nl):
    from paper_2505_10899_amd import vclb as v
    p, phi0, u0 = _case(nx, ny, storage, wall, mode, visc, nl)
    print("case:", nx, ny, storage, wall, mode, visc, nl, flush=True)
    m = Model(p).init(phi0, u0)
    m.step(1)
    c = v.Case(p.replace(storage=storage))
    c.set_state(m.g, m.f if mode == "coupled" else None, m.Jprev, m.t)
    # the recorded reductions are compared with those of the very field they were taken of
    field = lambda: observables_from_phi(p, c.observe(v.FIELD_PHI)["phi"])
    obs = [field()]
    if storage == "fp16s":
        d = v.Case(p.replace(storage=storage))
        d.set_state(m.g, m.f if mode == "coupled" else None, m.Jprev, m.t)
        c.step(1)
        d.step_plain(1)
        for a, b in zip(c.get_state(), d.get_state()):
            if a is not None:
                assert float(np.max(np.abs(a - b))) <= 2.0 ** -15 + 2e-6
    else:
        base, eps = (1e-13, 2.2e-16) if storage == "fp64" else (1e-6, 6e-8)
        tol = base + 2.0 * normal_conditioning(m, m.fields(), eps=eps)
        c.step(1)
        m.step(1)
        g, f, J = c.get_state()
        assert float(np.max(np.abs(g - m.g) / tol[None])) <= 1.0
        assert float(np.max(np.abs(J - m.Jprev))) <= base
        if mode == "coupled":
            assert float(np.max(np.abs(f - m.f) / tol[None])) <= 1.0
    obs.append(field())
    c.step(1)                                   # its launch sums the first step's partials
    h = c.history(1, 2)
    rtol = {"fp64": 1e-12, "fp32": 2e-6, "fp16s": 2e-4}[storage]
    scale = {"sum_phi": 1.0, "sum_phi_d": max(nx, ny), "sum_phi_dd": max(nx, ny) ** 2}
    for t in range(2):
        total = np.abs(obs[t]["sum_phi"]).sum() + 1.0
        for k, s in scale.items():
            assert float(np.max(np.abs(h[k][t] - obs[t][k]))) <= rtol * s * total, (t, k)
        assert not h["nonfinite"].any()


@pytest.mark.parametrize("storage", ["fp64", "fp32", "fp16s"])
@pytest.mark.parametrize("visc", [1.0, 3.75])
def test_batch_one_step(storage, visc):
    """A batch small enough for lane tiles: each case's step from the oracle's state against
    the oracle's own (FP16S: against the plain path), and its recorded sum of phi."""
    from paper_2505_10899_amd import vclb as v
    cases = [_case(nx, ny, storage, k % 2 == 1, "coupled", visc if k % 3 else 1.0, 1) for k, (nx, ny) in enumerate(SMALL)]
    b = v.Batch([p.replace(storage=storage) for p, _, _ in cases])
    models = []
    for c, (p, phi0, u0) in zip(b.cases, cases):
        m = Model(p).init(phi0, u0)
        m.step(1)
        c.set_state(m.g, m.f, m.Jprev, m.t)
        models.append(m)
    field = lambda: [observables_from_phi(p, c.observe(v.FIELD_PHI)["phi"])["sum_phi"][0]
                     for c, (p, _, _) in zip(b.cases, cases)]
    sums = [field()]
    b.step(1)
    for k, (c, m) in enumerate(zip(b.cases, models)):
        print("case:", k, SMALL[k], storage, visc, flush=True)
        got = c.get_state()
        if storage == "fp16s":
            d = v.Case(m.p.replace(storage=storage))
            d.set_state(m.g, m.f, m.Jprev, m.t)
            d.step_plain(1)
            for x, y in zip(got, d.get_state()):
                assert float(np.max(np.abs(x - y))) <= 2.0 ** -15 + 2e-6
            continue
        base, eps = (1e-13, 2.2e-16) if storage == "fp64" else (1e-6, 6e-8)
        tol = base + 2.0 * normal_conditioning(m, m.fields(), eps=eps)
        m.step(1)
        assert float(np.max(np.abs(got[0] - m.g) / tol[None])) <= 1.0
        assert float(np.max(np.abs(got[1] - m.f) / tol[None])) <= 1.0
        assert float(np.max(np.abs(got[2] - m.Jprev))) <= base
    sums.append(field())
    b.step(1)
    h = b.history(1, 2)["sum_phi"][:, :, 0]
    rtol = {"fp64": 1e-12, "fp32": 2e-6, "fp16s": 2e-4}[storage]
    assert np.all(np.abs(h - np.array(sums)) <= rtol * (1.0 + np.abs(np.array(sums))))
    r = b.reduce()
    assert np.all(np.abs(r["sum_phi"][:, 0] - np.array(field())) <= rtol * (1.0 + np.abs(np.array(sums[1]))))


def test_history_over_the_end_of_the_ring():
    """The last HISTORY steps in one call (the ring wraps inside) equal single steps read
    one by one before and after the wrap."""
    from paper_2505_10899_amd import vclb
    p = W.CaseParams(nx=8, ny=6, storage="fp32", label_centres=[(4.2, 3.1, 0.0)])
    c = vclb.Case(p).init(W.drops_phi(p, [(4.2, 3.1, 0.0, 2.0)]))
    c.step(vclb.HISTORY + 7)
    h = c.history(7, vclb.HISTORY)
    assert np.array_equal(h["step"][:, 0], np.arange(7, vclb.HISTORY + 7))
    for t in (7, vclb.HISTORY - 1, vclb.HISTORY, vclb.HISTORY + 6):
        one = c.history(t, 1)
        assert all(np.array_equal(one[k][0], h[k][t - 7]) for k in one)
