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
