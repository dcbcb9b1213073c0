"""The fused backward step (16 x 8 tiles, a halo of one node for phi and psi and of two for
the stencil adjoints) at the edges of its tiles: one tile exactly, one node less and more
on each side, sizes that wrap onto themselves; periodic and between wetting walls, one and
two labels, unequal viscosities.  Gradients against the oracle's complex step to 1e-6, the
bound of test_gpu_adjoint.py."""
import numpy as np
import pytest

import workloads as W
from oracle import gradient as OG

pytestmark = pytest.mark.gpu

TOL = 1e-6
CASES = [(16, 8, False, 1), (17, 9, True, 1), (15, 7, False, 2), (32, 16, True, 2), (33, 23, False, 1), (10, 20, True, 1)]


@pytest.mark.parametrize("nx,ny,wall,nl", CASES, ids=["%dx%d-%s-%d" % (c[0], c[1], "w" if c[2] else "p", c[3]) for c in CASES])
def test_gradients_match_complex_step(nx, ny, wall, nl):
    from paper_2505_10899_amd import vclb as v
    m = min(nx, ny)
    c1, c2 = (0.31 * nx + 0.13, 0.47 * ny + 0.21, 0.0), (0.73 * nx + 0.07, 0.52 * ny + 0.11, 0.0)
    p = W.CaseParams(nx=nx, ny=ny, wall_y=wall, rho_light=0.3, W=3.0, label_centres=[c1, c2][:nl])
    if wall:
        p = p.replace(wall_u_bottom=(-0.01, 0.0, 0.0), wall_u_top=(0.01, 0.0, 0.0), wall_cos_bottom=0.5,
                      wall_cos_top=-0.3, nu_light=0.3)
    phi0 = 0.02 + 0.94 * np.clip(W.drops_phi(p, [(*c1, 0.28 * m), (*c2, 0.16 * m)]), 0.0, 1.0)   # off the clip
    u0 = W.couette_u(p) if wall else None
    n = 20
    rng = np.random.Generator(np.random.PCG64(7))
    w = rng.uniform(0.5, 1.5, (nl, 5))
    w[:, 3] = 0.0
    d = rng.standard_normal(phi0.shape) * 4.0 * phi0 * (1.0 - phi0)
    print("case:", nx, ny, wall, nl, flush=True)
    c = v.Case(p)
    c.adjoint_record(phi0, u0, nsteps=n, every=6)
    raw = c.reduce_raw()
    dphi, ds, dm = c.adjoint_run(v.obs_seed(raw, nl, w))
    got = {"sigma": ds, "mobility": dm, "phi0": float((dphi.cpu().numpy().reshape(phi0.shape) * d).sum())}
    for wrt, val in got.items():
        ref = float((OG.complex_step(p, phi0, u0, n, wrt, direction=d) * w).sum())
        print("  d/d%s: gpu %.12e complex step %.12e" % (wrt, val, ref), flush=True)
        assert abs(val - ref) <= TOL * max(abs(ref), 1e-3)


@pytest.mark.parametrize("nsteps,every", [(0, 0), (1, 1), (13, 4)])
def test_a_lent_store_gives_the_bits_of_the_library_s_own(nsteps, every):
    """vclb_adjoint_set_store: exactly vclb_adjoint_bytes of memory; too little or misaligned
    memory is refused; the binding's own record on another stream gives the same bits."""
    import ctypes

    import torch
    from paper_2505_10899_amd import vclb as v
    L = v.lib()
    p = W.CaseParams(nx=33, ny=23, rho_light=0.3, W=3.0, label_centres=[(10.2, 11.1, 0.0)])
    phi0 = torch.as_tensor(0.02 + 0.94 * W.drops_phi(p, [(10.2, 11.1, 0.0, 6.0)]), dtype=torch.float64, device="cuda").contiguous()
    seed = np.ones((1, v.SEED_FIELDS))
    n = ctypes.c_size_t()
    v.check(L.vclb_adjoint_bytes(ctypes.byref(v.to_cparams(p)), nsteps, every, ctypes.byref(n)))
    mem = torch.empty(n.value + 256, dtype=torch.uint8, device="cuda")
    base = (mem.data_ptr() + 255) // 256 * 256

    def record(c):
        return L.vclb_adjoint_record(c.h, ctypes.c_void_p(phi0.data_ptr()), None, v.DEVICE, nsteps, every, v._stream_handle(None))

    runs = []
    c = v.Case(p)
    for lend in (None, base, None):
        v.check(L.vclb_adjoint_set_store(c.h, ctypes.c_void_p(lend), n.value))
        with pytest.raises(v.VclbError):
            c.adjoint_run(seed)                       # what was recorded is dropped
        v.check(record(c))
        dphi, ds, dm = c.adjoint_run(seed)
        runs.append((dphi.cpu().numpy(), ds, dm))
    assert L.vclb_adjoint_set_store(c.h, ctypes.c_void_p(base + 8), n.value) == v.VCLB_EINVAL
    v.check(L.vclb_adjoint_set_store(c.h, ctypes.c_void_p(base), n.value - 1))
    assert record(c) == v.VCLB_ENOMEM
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    c.adjoint_record(phi0, nsteps=nsteps, every=every, stream=s)
    dphi, ds, dm = c.adjoint_run(seed, stream=s)
    torch.cuda.synchronize()
    runs.append((dphi.cpu().numpy(), ds, dm))
    for r in runs[1:]:
        assert np.array_equal(r[0], runs[0][0]) and r[1:] == runs[0][1:]
