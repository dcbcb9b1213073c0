"""Three steps in one launch (tile2d_multi: tiles of 8 x 8 nodes, or of 16 x 16 on larger grids,
with four nodes around them).

One step of the same kernel is checked against the oracle in test_gpu_lane_tiles.py; here
groups of three must give the bits of single launches, states and recorded reductions alike
(tolerance zero: one loop body serves every step), at the edges of the tiles and of their
halos, on grids that wrap onto themselves within the halo, at walls, in every storage."""
import numpy as np
import pytest

from test_gpu_lane_tiles import _case

pytestmark = pytest.mark.gpu

SIZES = [(8, 8), (9, 7), (7, 9), (16, 12), (5, 3), (2, 3), (1, 9), (13, 4), (66, 24), (37, 70), (130, 3)]
CASES = [(nx, ny, st, wall, "coupled", 3.75 if k % 3 == 0 else 1.0, 1 + k % 2)
         for k, (nx, ny) in enumerate(SIZES) for st in ("fp64", "fp32", "fp16s") for wall in (False, True)]
CASES += [(35, 20, st, False, "vortex", 1.0, 2) for st in ("fp64", "fp32", "fp16s")]
# 16 x 16 tiles: more than 256 of 8 x 8
CASES += [(nx, ny, st, wall, "coupled", visc, nl) for nx, ny, wall, visc, nl in
          ((131, 129, False, 1.0, 1), (145, 127, True, 3.75, 2), (256, 256, False, 1.0, 1)) for st in ("fp32", "fp16s")]
CASES += [(nx, ny, st, False, "vortex", 1.0, 1) for nx, ny in ((131, 129), (256, 241)) for st in ("fp64", "fp32", "fp16s")]
CASES += [(131, 129, "fp64", True, "coupled", 1.0, 1)]       # single steps in 16 x 8 tiles
IDS = ["%dx%d-%s-%s-%s-%g-%d" % (c[0], c[1], c[2], "w" if c[3] else "p", *c[4:]) for c in CASES]


def same(a, b):
    for x, y in zip(a.get_state(), b.get_state()):
        assert (x is None) == (y is None)
        if x is not None:
            assert np.array_equal(x, y, equal_nan=True), float(np.abs(x - y).max())


@pytest.mark.parametrize("nx,ny,storage,wall,mode,visc,nl", CASES, ids=IDS)
def test_groups_of_three_equal_single_steps(nx, ny, storage, wall, mode, visc, nl):
    from paper_2505_10899_amd import vclb as v
    p, phi0, u0 = _case(nx, ny, storage, wall, mode, visc, nl)
    print("case:", nx, ny, storage, wall, mode, visc, nl, flush=True)
    p = p.replace(storage=storage)
    a, b = v.Case(p).init(phi0, u0), v.Case(p).init(phi0, u0)
    for n in (1, 3, 2, 7):          # groups that start at even and at odd steps
        a.step(n)
        for _ in range(n):
            b.step(1)
        same(a, b)
    ha, hb = a.history(0, 13), b.history(0, 13)
    assert all(np.array_equal(ha[k], hb[k], equal_nan=True) for k in ha)
    assert np.array_equal(ha["step"][:, 0], np.arange(13))


@pytest.mark.parametrize("every", [0, 1, 2, 3, 5])
def test_state_goes_on_from_any_step(every):
    """Sparse recording, checkpoints at odd and even steps, a march between groups, a second
    init after an odd step."""
    from paper_2505_10899_amd import vclb as v
    p, phi0, u0 = _case(24, 17, "fp64", True, "coupled", 1.0, 2)
    a, b = v.Case(p).init(phi0, u0), v.Case(p).init(phi0, u0)
    for c in (a, b):
        c.set_reduce_every(every)
    a.step(12)
    for _ in range(12):
        b.step(1)
    if every:
        for t in range(0, 12, every):
            ha, hb = a.history(t, 1), b.history(t, 1)
            assert all(np.array_equal(ha[k], hb[k]) for k in ha)
    a.step(9)
    blob = a.save()
    c = v.Case(p)
    c.load(blob)
    a.step(4)
    c.step(1)
    c.step(3)
    same(a, c)
    g, f, J = a.get_state()
    c = v.Case(p)
    c.init(phi0, u0)
    c.step(2)
    c.set_state(g, f, J, 25)
    a.step(6)
    c.step(6)
    same(a, c)
    a.step(3)                       # its reductions are pending when the march takes over
    a.set_tile(64, 8)
    a.step(1)
    c.step(3)
    c.step_plain(1)
    for x, y in zip(a.get_state(), c.get_state()):
        assert float(np.abs(x - y).max()) < 1e-12
    if every == 1:
        h = a.history(31, 4)
        assert np.array_equal(h["step"][:, 0], np.arange(31, 35))
    a.init(phi0, u0)                # after an even step, and the other after an odd one
    c.step(1)
    c.init(phi0, u0)
    d = v.Case(p).init(phi0, u0)
    d.step(3)
    c.step(3)
    same(c, d)
