"""The forms of a step (row or section march, lane tiles, a batch's runs) of one case give the
same state bit for bit, so that neither the library's choice of a form nor its autotuner
changes results.  No tolerance: states are compared for equality."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

# a size per default shape of the lane tiles: 8 x 8 and 16 x 16 (three steps in a launch),
# 16 x 8, 64 x 4, 128 x 4 plain and (rows of whole lines) with the non-temporal hint
SIZES = [(66, 45), (251, 200), (333, 301), (801, 777), (2051, 1843), (2048, 1843)]


def _case(nx, ny, storage, wall, visc=1.0, general=False, nl=1, mode="coupled"):
    m = min(nx, ny)
    c1, c2 = (0.31 * nx + 0.13, 0.47 * ny + 0.21, 0.0), (0.73 * nx + 0.07, 0.52 * ny + 0.11, 0.0)
    p = W.CaseParams(nx=nx, ny=ny, storage=storage, wall_y=wall, rho_light=0.1, label_centres=[c1, c2][:nl], mode=mode)
    if mode == "vortex":
        p = p.replace(U0=0.04, T=400.0, mobility=0.02)
    if wall:
        p = p.replace(wall_u_bottom=(-0.02, 0.0, 0.0), wall_u_top=(0.015, 0.0, 0.0), wall_cos_bottom=0.4,
                      wall_cos_top=-0.3)
    if visc != 1.0:
        p = p.replace(nu_light=p.nu * visc)
    if general:
        p = p.replace(s_g=(0.0, 1.3, 1.2) + (0.0,) * 6, s_f=(0.0, 1.1, 1.25) + (0.0,) * 6)
    phi0 = W.drops_phi(p, [(*c1, min(24.0, 0.19 * m)), (*c2, min(15.0, 0.1 * m))])
    y, x = np.mgrid[0:ny, 0:nx]
    u0 = 0.02 * np.stack([np.sin(2 * np.pi * y / ny), np.sin(2 * np.pi * x / nx)])[:, None]
    if wall:
        u0[1] = 0.0
    return p, np.clip(phi0, 0.0, 1.0), u0


def _states(p, phi0, u0, steps, tile=None):
    from paper_2505_10899_amd import vclb as v
    c = v.Case(p).init(phi0, u0)
    if tile is not None:
        c.set_tile(*tile)
    c.step(steps)
    return c.get_state()


def _same(a, b):
    for name, x, y in zip("gfJ", a, b):
        assert (x is None) == (y is None)
        assert x is None or np.array_equal(x, y), (name, float(np.abs(x - y).max()), float(np.mean(x != y)))


@pytest.mark.parametrize("wall,visc,general", [(False, 1.0, False), (True, 3.75, False), (True, 1.0, True),
                                               (False, 3.75, True)])
@pytest.mark.parametrize("nx,ny", SIZES)
@pytest.mark.parametrize("storage", ["fp64", "fp32", "fp16s"])
def test_lane_tiles_equal_the_march(nx, ny, storage, wall, visc, general):
    print("case:", nx, ny, storage, wall, visc, general, flush=True)
    args = _case(nx, ny, storage, wall, visc, general, nl=2 if general else 1)
    _same(_states(*args, 10), _states(*args, 10, tile=(64, 16)))


@pytest.mark.parametrize("nx,ny", SIZES)
@pytest.mark.parametrize("storage", ["fp64", "fp32", "fp16s"])
def test_lane_tiles_equal_the_march_vortex(nx, ny, storage):
    print("case:", nx, ny, storage, flush=True)
    for general in (False, True):
        p, phi0, _ = _case(nx, ny, storage, False, general=general, mode="vortex")
        _same(_states(p, phi0, None, 10), _states(p, phi0, None, 10, tile=(64, 16)))


@pytest.mark.parametrize("wall,visc,general", [(False, 1.0, False), (True, 3.75, False), (True, 1.0, True),
                                               (False, 3.75, True)])
@pytest.mark.parametrize("nx,ny,nz", [(36, 30, 40), (61, 45, 130), (64, 16, 24), (96, 80, 250)])
@pytest.mark.parametrize("storage", ["fp64", "fp32", "fp16s"])
def test_two_passes_equal_the_march(nx, ny, nz, storage, wall, visc, general):
    print("case:", nx, ny, nz, storage, wall, visc, general, flush=True)
    c1 = (0.47 * nx + 0.13, 0.52 * ny + 0.21, 0.0)
    p = W.CaseParams(lattice="D3Q19", nx=nx, ny=ny, nz=nz, storage=storage, sigma=0.005, nu=0.05, rho_light=0.1,
                     wall_y=wall, label_centres=[c1])
    if wall:
        p = p.replace(wall_u_bottom=(-0.01, 0.0, 0.0), wall_u_top=(0.01, 0.0, 0.005), wall_cos_bottom=0.4,
                      wall_cos_top=-0.3)
    if visc != 1.0:
        p = p.replace(nu_light=p.nu * visc)
    if general:
        p = p.replace(s_g=(0.0, 1.3, 1.2) + (0.0,) * 16, s_f=(0.0, 1.1, 1.25) + (0.0,) * 16)
    z, y, x = np.mgrid[0:nz, 0:ny, 0:nx]
    R = min(nx, ny) / 5.0 * (1.0 + 0.1 * np.cos(2 * np.pi * z / nz))
    phi0 = 0.5 + 0.5 * np.tanh(2.0 * (R - np.hypot(x - c1[0], y - c1[1])) / p.W)
    u0 = 0.02 * np.stack([np.sin(2 * np.pi * y / ny), np.zeros(x.shape), np.cos(2 * np.pi * x / nx)])
    ref = _states(p, phi0, u0, 6)
    _same(ref, _states(p, phi0, u0, 6, tile=(32, 8, 8)))
    if storage != "fp64":
        _same(ref, _states(p, phi0, u0, 6, tile=(96, 8, 8)))   # 768 lanes
    if general:
        c2 = (0.8 * nx, 0.25 * ny, 0.0)                          # two labels
        _same(ref, _states(p.replace(label_centres=[c1, c2]), phi0, u0, 6, tile=(32, 8, 8)))


@pytest.mark.parametrize("storage", ["fp64", "fp32", "fp16s"])
def test_batch_lane_tiles_equal_the_runs(storage):
    """Cases that the runs do in bands (narrow against a run's 512 lanes) and in strips."""
    from paper_2505_10899_amd import vclb as v
    sizes = [(130, 67), (64, 64), (300, 90), (512, 40), (70, 333), (1024, 30), (48, 48), (150, 300)]
    sims = [_case(nx, ny, storage, k % 2 == 1) for k, (nx, ny) in enumerate(sizes)]
    got = []
    for runs in (False, True):
        b = v.Batch([p for p, _, _ in sims])
        b.init([(phi, u) for _, phi, u in sims])
        if runs:
            b.set_tile(*b.tile()[:2])   # the default run shape
        b.step(10)
        got.append([c.get_state() for c in b.cases])
    for k, (x, y) in enumerate(zip(*got)):
        print("case:", sizes[k], storage, flush=True)
        _same(x, y)


@pytest.mark.parametrize("storage,side,inside,beyond", [("fp64", 262, 10, 12), ("fp32", 262, 17, 20),
                                                        ("fp16s", 262, 31, 38)])
def test_batch_leaves_lane_tiles_before_the_cache_is_full(storage, side, inside, beyond):
    """Lane tiles lose to the runs where the state fills the last-level cache; the recorded sums
    tell the two apart, as each adds in the order of its own workgroups."""
    from paper_2505_10899_amd import vclb as v
    for n, runs in ((inside, False), (beyond, True)):
        print("case:", storage, n, flush=True)
        p, phi0, u0 = _case(side, side, storage, False)
        got = []
        for chosen in (False, True):
            b = v.Batch([p] * n)
            b.init([(phi0, u0)] * n)
            if chosen:
                b.set_tile(*b.tile()[:2])   # the default run shape
            b.step(3)
            h = [c.history(0, 3) for c in b.cases]
            got.append([[x[k].ravel() for x in h] for k in ("sum_phi", "sum_phi_d", "sum_phi_dd")])
        assert all(np.array_equal(x, y) for x, y in zip(*got)) == runs


LANE_SHAPES = [(8, 8), (16, 16), (16, 8), (64, 4), (128, 4)]


@pytest.mark.parametrize("mode,wall,visc,general", [("coupled", False, 1.0, False), ("coupled", True, 3.75, True),
                                                    ("vortex", False, 1.0, False), ("vortex", False, 1.0, True)])
@pytest.mark.parametrize("storage", ["fp64", "fp32", "fp16s"])
def test_every_form_of_a_case(storage, mode, wall, visc, general):
    """Every tile shape and march that the autotuner chooses from, chosen by name."""
    from paper_2505_10899_amd import vclb as v
    p, phi0, u0 = _case(133, 70, storage, wall, visc, general, nl=2, mode=mode)
    u0 = u0 if mode == "coupled" else None
    ref = _states(p, phi0, u0, 11, tile=(64, 16))
    shapes = [s for s in LANE_SHAPES if s != (16, 16) or mode == "vortex" or storage != "fp64"]
    tiles = [(64, 8), (128, 32), (256, 64)] + ([(512, 16), (1024, 8)] if storage != "fp64" else [])
    for form in [("lane_tiles", *s) for s in shapes] + tiles:
        print("case:", storage, mode, wall, visc, general, form, flush=True)
        c = v.Case(p).init(phi0, u0)
        if form[0] == "lane_tiles":
            c.set_form(*form)
            assert c.form() == form
        else:
            c.set_tile(*form)
            assert c.form() == ("march", 0, 0) and c.tile()[:2] == form
        c.step(11)
        _same(c.get_state(), ref)


def test_form_is_read_and_restored():
    from paper_2505_10899_amd import vclb as v
    p, phi0, u0 = _case(66, 45, "fp32", False)
    c = v.Case(p).init(phi0, u0)
    tile, form = c.tile(), c.form()
    assert form == ("lane_tiles", 8, 8)
    c.set_tile(*tile)
    assert c.form() == ("march", 0, 0) and c.tile() == tile
    c.step(2)
    c.set_form(*form)
    assert c.form() == form and c.tile() == tile
    c.step(4)
    _same(c.get_state(), _states(p, phi0, u0, 6))
    for bad in [("two_passes",), ("lane_tiles", 8, 4), ("lane_tiles", 0, 0), ("lane_tiles", 2, 2), ("lane_tiles", 128, 8)]:
        with pytest.raises(v.VclbError) as e:
            c.set_form(*bad)
        assert e.value.code == v.VCLB_EINVAL
    # three steps per launch need room that a case of a batch, and a large one, do not have
    big = v.Case(p.replace(nx=300, ny=300, label_centres=[]))
    view = v.Batch([p]).cases[0]
    coupled64 = v.Case(p.replace(storage="fp64"))
    for case, shape in ((big, (8, 8)), (view, (8, 8)), (coupled64, (16, 16))):
        with pytest.raises(v.VclbError):
            case.set_form("lane_tiles", *shape)
    p3 = W.CaseParams(lattice="D3Q19", nx=32, ny=16, nz=12, storage="fp64")
    c3 = v.Case(p3)
    assert c3.form() == ("two_passes", 0, 0)
    c3.set_form("march")
    assert c3.form() == ("march", 0, 0)
    c3.set_form("two_passes")
    with pytest.raises(v.VclbError):
        c3.set_form("lane_tiles", 16, 8)
