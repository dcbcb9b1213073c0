"""The autotuners' tune files and timing."""
import json
import re

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _case(nx=130, ny=67, storage="fp32", **kw):
    p = W.CaseParams(nx=nx, ny=ny, storage=storage, label_centres=[(40.2, 30.3, 0.0)], **kw)
    return p, W.drops_phi(p, [(40.2, 30.3, 0.0, 12.0)])


def _lines(path):
    return open(path).read().strip().splitlines()


def test_case_entries_without_the_forms_are_timed_again(tmp_path):
    """An entry of a build that timed marches only says nothing of lane tiles."""
    from paper_2505_10899_amd import vclb as v
    path = str(tmp_path / "tiles.jsonl")
    p, phi0 = _case()
    v.Case(p).init(phi0).autotune(path, steps=3)
    (line,) = _lines(path)
    old = re.sub(r'"lane_tile": \[\d+, \d+\], "flat": \d, ', "", line)
    assert old != line
    open(path, "w").write(old + "\n")
    c = v.Case(p).init(phi0)
    c.autotune(path, steps=3)
    assert len(_lines(path)) == 2
    d = v.Case(p).init(phi0)
    d.autotune(path, steps=3)              # the new entry is found
    assert len(_lines(path)) == 2 and d.form() == c.form()


def test_batch_entries_without_lane_tiles_are_timed_again(tmp_path):
    from paper_2505_10899_amd import vclb as v
    path = str(tmp_path / "batch.jsonl")
    sims = [_case(nx, ny) for nx, ny in ((64, 48), (100, 70))]

    def tuned():
        b = v.Batch([p for p, _ in sims])
        b.init([(phi, None) for _, phi in sims])
        b.autotune(path, steps=2)
        return len(_lines(path))
    assert tuned() == 1
    line = _lines(path)[0]
    old = re.sub(r'"lane_tiles": \d, ', "", line)
    assert old != line
    open(path, "w").write(old + "\n")
    assert tuned() == 2 and tuned() == 2


def test_a_batch_view_does_not_read_a_case_of_its_own(tmp_path):
    """Three steps in a launch are for cases outside batches."""
    from paper_2505_10899_amd import vclb as v
    path = str(tmp_path / "tiles.jsonl")
    p, phi0 = _case()
    c = v.Case(p).init(phi0)
    c.autotune(path, steps=3)
    b = v.Batch([p])
    b.init([(phi0, None)])
    view = b.cases[0]
    view.autotune(path, steps=3)
    assert len(_lines(path)) == 2
    assert view.form()[1:] not in ((8, 8), (16, 16))
    c.step(4)
    view.step(4)
    for x, y in zip(c.get_state(), view.get_state()):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("steps", [1, 2, 5])
def test_three_steps_a_launch_are_timed_by_whole_launches(tmp_path, steps):
    """Single steps in such a tile cost about two; the entry says how many steps were timed,
    and lists every candidate with its form."""
    from paper_2505_10899_amd import vclb as v
    path = str(tmp_path / "tiles.jsonl")
    p, phi0 = _case(256, 256, "fp64", mode="vortex", U0=0.04, T=400.0, mobility=0.02)
    c = v.Case(p).init(phi0)
    c.autotune(path, steps=steps)
    (line,) = _lines(path)
    e = json.loads(line)
    lanes = [tuple(k[3:5]) for k in e["candidates"] if k[3]]
    assert lanes == [(3, 3), (4, 4), (4, 3), (6, 2), (7, 2)]
    assert e["timed"] % 3 == 0 and steps <= e["timed"] < steps + 3
    p, phi0 = _case(300, 333)              # none among the candidates
    c = v.Case(p).init(phi0)
    c.autotune(path, steps=steps)
    e = json.loads(_lines(path)[1])
    assert e["timed"] == steps and [tuple(k[3:5]) for k in e["candidates"] if k[3]] == [(4, 3), (6, 2), (7, 2)]


@pytest.mark.parametrize("nz", [1, 24])
@pytest.mark.parametrize("storage", ["fp64", "fp32", "fp16s"])
def test_no_candidate_changes_results(tmp_path, storage, nz):
    """Each candidate that the tuner lists, chosen through the tune file, continues the run as
    the default does, bit for bit."""
    from paper_2505_10899_amd import vclb as v
    path = str(tmp_path / "tiles.jsonl")
    nx, ny = (130, 67) if nz == 1 else (44, 30)
    c1 = (0.4 * nx + 0.2, 0.5 * ny + 0.3, 0.0)
    p = W.CaseParams(lattice="D2Q9" if nz == 1 else "D3Q19", nx=nx, ny=ny, nz=nz, storage=storage, rho_light=0.1,
                     label_centres=[c1])
    y, x = np.mgrid[0:ny, 0:nx]
    phi0 = np.broadcast_to(0.5 + 0.5 * np.tanh(2.0 * (0.25 * min(nx, ny) - np.hypot(x - c1[0], y - c1[1])) / p.W),
                           (nz, ny, nx)).copy()
    u0 = np.zeros((p.dim, nz, ny, nx))
    u0[0] = 0.02 * np.sin(2 * np.pi * y / ny)
    c = v.Case(p).init(phi0, u0)
    c.autotune(path, steps=3)
    (line,) = _lines(path)
    entry = json.loads(line)
    ref = v.Case(p).init(phi0, u0)
    ref.step(7)
    ref = ref.get_state()
    timed = [k for k in entry["candidates"] if k[-1] > 0]
    # 2D: lane tiles (16 x 16 not in coupled FP64) and 5 heights of 3 or 5 widths of march
    assert len(timed) >= ((4 + 15 if storage == "fp64" else 5 + 25) if nz == 1 else 10)
    for bx, ty, by3, lx, ly, flat, _ in timed:
        print("case:", storage, nz, (bx, ty, by3, lx, ly, flat), flush=True)
        new = dict(entry, bx=bx, ty=ty, by3=by3, lane_tile=[lx, ly], flat=flat)
        open(path, "w").write(json.dumps(new) + "\n")
        d = v.Case(p).init(phi0, u0)
        d.autotune(path, steps=3)
        assert len(_lines(path)) == 1
        assert d.form()[0] == ("lane_tiles" if lx else "two_passes" if flat else "march")
        d.step(7)
        for a, b in zip(d.get_state(), ref):
            assert np.array_equal(a, b)
