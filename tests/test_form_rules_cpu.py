"""Which form of the step a case gets by default, at sizes on either side of each rule's line
where the two forms' measured times differ.  No GPU: a case is created over memory that is
never touched."""
import ctypes

import pytest

import workloads as W


def _form(p):
    from paper_2505_10899_amd import vclb as v
    L = v.lib()
    h = ctypes.c_void_p()
    # only the address and the size are looked at
    assert L.vclb_case_create(ctypes.byref(v.to_cparams(p)), ctypes.c_void_p(1 << 20), v.workspace_bytes(p),
                              ctypes.byref(h)) == v.VCLB_OK
    f, w, k = ctypes.c_int32(), ctypes.c_int32(), ctypes.c_int32()
    assert L.vclb_case_get_form(h, ctypes.byref(f), ctypes.byref(w), ctypes.byref(k)) == v.VCLB_OK
    L.vclb_case_destroy(h)
    return (v.FORMS[f.value], w.value, k.value) if w.value else v.FORMS[f.value]


GENERAL = dict(s_g=(0.0, 1.3, 1.2) + (0.0,) * 16)


@pytest.mark.parametrize("storage,size,form,change", [
    ("fp64", (64, 64, 350), "march", {}), ("fp64", (96, 96, 200), "march", {}), ("fp64", (256, 64, 64), "march", {}),
    ("fp64", (96, 96, 384), "march", {}), ("fp64", (96, 96, 200), "march", dict(wall_y=True)),
    ("fp64", (32, 32, 256), "two_passes", {}), ("fp64", (72, 72, 400), "two_passes", {}),
    ("fp64", (100, 96, 384), "two_passes", {}), ("fp64", (80, 80, 300), "two_passes", {}),
    ("fp32", (96, 96, 200), "march", {}), ("fp32", (96, 8, 2000), "march", {}), ("fp32", (96, 96, 384), "march", {}),
    ("fp32", (96, 96, 200), "two_passes", GENERAL), ("fp32", (192, 32, 200), "two_passes", {}),
    ("fp32", (64, 64, 350), "two_passes", {}), ("fp32", (90, 90, 400), "two_passes", {}),
    ("fp16s", (64, 64, 378), "march", {}), ("fp16s", (96, 8, 2000), "march", {}), ("fp16s", (64, 16, 1500), "march", {}),
    ("fp16s", (32, 64, 1000), "march", {}), ("fp16s", (32, 8, 15625), "march", {}),
    ("fp16s", (64, 64, 378), "two_passes", dict(wall_y=True)), ("fp16s", (32, 64, 1000), "two_passes", GENERAL),
    ("fp16s", (64, 64, 352), "two_passes", {}), ("fp16s", (64, 64, 396), "two_passes", {}),
    ("fp16s", (72, 72, 299), "two_passes", {}), ("fp16s", (320, 16, 303), "two_passes", {}),
    ("fp16s", (96, 96, 384), "two_passes", {}), ("fp16s", (256, 256, 100), "two_passes", {}),
    ("fp16s", (32, 8, 3000), "two_passes", {})])
def test_d3q19(storage, size, form, change):
    nx, ny, nz = size
    assert _form(W.CaseParams(lattice="D3Q19", nx=nx, ny=ny, nz=nz, storage=storage).replace(**change)) == form


@pytest.mark.parametrize("storage,size,form", [
    ("fp64", (128, 128), ("lane_tiles", 8, 8)), ("fp64", (512, 256), ("lane_tiles", 16, 8)),
    ("fp32", (777, 1333), ("lane_tiles", 64, 4)), ("fp64", (2048, 2048), ("lane_tiles", 128, 4)),
    ("fp32", (4096, 4096), "march"), ("fp16s", (4096, 2048), "march")])
def test_d2q9(storage, size, form):
    assert _form(W.CaseParams(nx=size[0], ny=size[1], storage=storage)) == form
