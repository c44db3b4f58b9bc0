"""Batches created while another thread changes the plan of their shape: the
work list and the launch follow one reading of the plan."""
import threading

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2308_02329_amd import api, synth  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def test_batches_beside_changing_plans():
    n, d, steps, reps = 40, 2, 8, 700
    g = synth.rng(88)
    J = torch.from_numpy(synth.sk_pm1(n, 88, n)).to(DEV)
    alpha = torch.ones((steps, d), device=DEV)
    x0 = [torch.from_numpy((g.standard_normal((n, reps, d)) * 0.3).astype(np.float32)).to(DEV) for _ in range(40)]
    pump = torch.from_numpy(g.uniform(0.5, 2.0, reps).astype(np.float32)).to(DEV)

    def solve():
        tasks = [dict(J=J, pump=pump, x=x.clone(), alpha=alpha, eps=0.04, btil=1.0, eta=2e-4, dt=0.01, steps=steps) for x in x0]
        ws = api.chym_solve_batched(tasks)
        torch.cuda.synchronize()
        del ws
        return torch.stack([t["x"] for t in tasks])

    want = solve()
    stop = threading.Event()

    def change():
        kinds = [(api.CHYM_KERNEL_REGJ, 4), (api.CHYM_KERNEL_LDSJ, 4), (api.CHYM_KERNEL_LDSJ, 2), (api.CHYM_KERNEL_AUTO, 4)]
        k = 0
        while not stop.is_set():
            api.chym_plan_set(n, d, "f32", torch.int8, *kinds[k % 4])
            k += 1

    t = threading.Thread(target=change)
    t.start()
    try:
        wrong = sum(not torch.equal(solve().view(torch.int32), want.view(torch.int32)) for _ in range(50))
    finally:
        stop.set()
        t.join()
        api.chym_plan_set(n, d, "f32", torch.int8, api.CHYM_KERNEL_AUTO)
    assert wrong == 0
