"""The Python binding on its own (no GPU): which libraries it accepts, and what it asks of
torch and of the library in calls that a GPU test could only catch by chance."""
import ctypes

import pytest


def _vclb():
    from paper_2505_10899_amd import vclb
    return vclb


class _Fn:
    def __init__(self, result=0):
        self.result = result

    def __call__(self, *a):
        return self.result


class _OldLibrary:
    """A library of an earlier minor version: no entry points but these."""

    def __init__(self, version):
        self.vclb_version = _Fn(version)
        self.vclb_strerror = _Fn(b"")


@pytest.mark.parametrize("version", [20100, 10000, 30000])
def test_other_version_is_refused_by_its_number(monkeypatch, version):
    """Not by the first symbol that it lacks."""
    v = _vclb()
    monkeypatch.setattr(v, "_lib", None)
    monkeypatch.setattr(ctypes, "CDLL", lambda path: _OldLibrary(version))
    with pytest.raises(ImportError, match=str(version)):
        v.lib()


def test_adjoint_store_came_with_a_new_minor_version():
    v = _vclb()
    assert "vclb_adjoint_set_store" in v.exported_symbols()
    assert v.lib().vclb_version() == v.VERSION >= 20200


class _Library:
    """Every entry point succeeds, but for those given."""

    def __init__(self, **special):
        self.special = special
        self.calls = []

    def __getattr__(self, name):
        def call(*args):
            self.calls.append(name)
            f = self.special.get(name)
            return f(*args) if f else 0
        return call


@pytest.mark.parametrize("first", ["none", "memory", "hip"])
def test_memory_in_torchs_cache_is_given_back_to_the_library(monkeypatch, first):
    """A case's adjoint store (or workspace) stays in torch's cache after the case: a library
    call that then finds no memory is made again with the cache emptied."""
    import workloads as W
    v = _vclb()
    given_back = []
    status = {"none": [0], "memory": [v.VCLB_ENOMEM, 0], "hip": [v.VCLB_EHIP, 0]}[first]
    answers = iter(status)
    fake = _Library(vclb_batch_create=lambda *a: next(answers),
                    vclb_last_error=lambda: b"hipMalloc(&save, bytes): out of memory")
    monkeypatch.setattr(v, "lib", lambda: fake)
    monkeypatch.setattr(v.torch.cuda, "empty_cache", lambda: given_back.append(1))
    p, _, _ = W.two_droplets()
    v.Batch([p])
    assert fake.calls.count("vclb_batch_create") == len(status) and len(given_back) == len(status) - 1


def test_other_errors_are_not_tried_again(monkeypatch):
    import workloads as W
    v = _vclb()
    fake = _Library(vclb_batch_create=lambda *a: v.VCLB_EHIP, vclb_last_error=lambda: b"batch set-up: unknown error",
                    vclb_strerror=lambda rc: b"HIP error")
    monkeypatch.setattr(v, "lib", lambda: fake)
    monkeypatch.setattr(v.torch.cuda, "empty_cache", lambda: pytest.fail("not a lack of memory"))
    p, _, _ = W.two_droplets()
    with pytest.raises(v.VclbError):
        v.Batch([p])
    assert fake.calls.count("vclb_batch_create") == 1


class _Stream:
    def __init__(self, log, name, handle):
        self.log, self.name, self.cuda_stream = log, name, handle

    def synchronize(self):
        self.log.append(f"synchronize {self.name}")

    def wait_stream(self, other):
        self.log.append(f"{self.name} after {other.name}")


@pytest.mark.parametrize("call", ["init", "batch"])
def test_tensors_of_a_call_on_another_stream_live_until_it_is_done(monkeypatch, call):
    """init uploads its fields on torch's current stream and drops them at its end: the stream
    it was given has to come after their making, and has to be waited for."""
    import workloads as W
    v = _vclb()
    log = []
    cur, side = _Stream(log, "current", 1), _Stream(log, "side", 2)
    fake = _Library(vclb_case_init=lambda *a: log.append(f"launch on {a[-1].value}") or 0,
                    vclb_batch_init=lambda *a: log.append(f"launch on {a[-1].value}") or 0)
    monkeypatch.setattr(v, "lib", lambda: fake)
    monkeypatch.setattr(v.torch.cuda, "Stream", _Stream)
    monkeypatch.setattr(v.torch.cuda, "current_stream", lambda *a: cur)
    p, phi0, u0 = W.two_droplets()
    if call == "init":
        c = v.Case(p, device="cpu", _borrowed=(object(), ctypes.c_void_p()))
        c.init(phi0, u0, stream=side)
    else:
        v.Batch([p], device="cpu").init([(phi0, u0)], stream=side)
    assert log == ["side after current", "launch on 2", "synchronize side"]
    log.clear()
    if call == "init":
        c.init(phi0, u0)
        assert log == ["launch on 1", "synchronize current"]
