"""Workspace sizes are a function of the tasks alone: no plan entry and no
device changes them (CPU only)."""
import ctypes

import pytest

from paper_2308_02329_amd import _lib as L
from paper_2308_02329_amd import api

torch = pytest.importorskip("torch")


def _task(n, d, r, precision=L.CHYM_PREC_F32, j_dtype=L.CHYM_J_I8, steps=10):
    p = L.ChymProblem(n=n, d=d, j_dtype=j_dtype, reserved=0, j=0x1000, eps=0.1, btil=1.0, eta=0.0, reserved_f=0.0)
    run = L.ChymRun(r=r, steps=steps, start_step=0, precision=precision, dt=0.01, reserved_f=0.0, pump=0x2000, x=0x3000,
                    alpha=0x4000)
    return L.ChymTask(prob=p, run=run, out=L.ChymOut())


def _size(*tasks):
    lib = L.load()
    arr = (L.ChymTask * len(tasks))(*tasks)
    out = ctypes.c_size_t()
    assert lib.chym_batch_workspace_size(arr, len(tasks), ctypes.byref(out)) == L.CHYM_OK, lib.chym_last_error()
    return out.value


@pytest.mark.parametrize("n,d,r,kernel,waves", [(200, 3, 40, "SLAB", 8), (300, 4, 12, "SLAB", 8), (100, 3, 4096, "LDSJ", 4),
                                                (100, 2, 65536, "PIPE", 4), (20, 1, 5000, "REGJ", 1)])
def test_batch_size_does_not_depend_on_plans(n, d, r, kernel, waves, tmp_path):
    tasks = [_task(n, d, r), _task(n, d, 7), _task(50, 2, 33)]
    before = _size(*tasks)
    f = tmp_path / "plans"
    api.chym_plan_set(n, d, "f32", torch.int8, getattr(api, "CHYM_KERNEL_" + kernel), waves)
    try:
        assert _size(*tasks) == before
        api.chym_plan_save(str(f))
    finally:
        api.chym_plan_set(n, d, "f32", torch.int8, api.CHYM_KERNEL_AUTO)
    api.chym_plan_load(str(f))
    try:
        assert _size(*tasks) == before
    finally:
        api.chym_plan_set(n, d, "f32", torch.int8, api.CHYM_KERNEL_AUTO)
    assert _size(*tasks) == before
