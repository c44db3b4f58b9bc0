"""The packed streamed-J integrator (16 columns per block) against the slab
kernel of the same problem, bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2308_02329_amd import api, synth  # noqa: E402

pytestmark = pytest.mark.gpu

STEPS = 70  # enough for the narrow coupling formats of a single problem


def _couplings(n, form, dev):
    if form == "i8":
        return torch.from_numpy(synth.sk_pm1(n, 77, n)).to(dev)
    J = torch.from_numpy(synth.gaussian_j(n, 77, n)).to(dev)
    if form == "bf16":
        return J.to(torch.bfloat16)
    return api.chym_quantize_fp8(J) if form == "fp8" else J


def _problem(n, d, r, form):
    dev = torch.device("cuda:0")
    g = synth.rng(81, n, d)
    pump = torch.from_numpy(g.uniform(0.5, 2.0, r).astype(np.float32)).to(dev)
    x = torch.from_numpy((g.standard_normal((n, r, d)) * 0.3).astype(np.float32)).to(dev)
    alpha = torch.from_numpy(g.uniform(0.0, 1.0, (STEPS + 3, d)).astype(np.float32)).to(dev)
    return dict(J=_couplings(n, form, dev), pump=pump, x=x, alpha=alpha, eps=0.04, btil=1.0, eta=2e-4, dt=0.01,
                start_step=2)


def _chosen(n, d, prec, J, fn):
    """fn() with the slab kernel chosen by the caller."""
    api.chym_plan_set(n, d, prec, J.dtype, api.CHYM_KERNEL_SLAB, 8)
    try:
        return fn()
    finally:
        api.chym_plan_set(n, d, prec, J.dtype, api.CHYM_KERNEL_AUTO)


def _single(p, prec, steps):
    x = p["x"].clone()
    api.chym_integrate(p["J"], p["pump"], x, p["alpha"], precision=prec, steps=steps,
                       **{k: p[k] for k in ("eps", "btil", "eta", "dt", "start_step")})
    return x


def _same(a, b):
    return torch.equal(a.view(torch.int32), b.view(torch.int32))


# 17 tiles, the wavefronts' tile counts at their edges (24|25, .. 56|57), the largest operand in two LDS buffers
# (26|27 chunks for three terms), and the largest problem
@pytest.mark.parametrize("n", [257, 272, 384, 385, 400, 512, 513, 640, 641, 768, 769, 832, 833, 896, 897, 1000, 1024])
@pytest.mark.parametrize("prec,form", [("f32", "i8"), ("f32", "fp8"), ("f32", "bf16"), ("f32", "f32"), ("bf16", "i8"),
                                       ("bf16", "bf16")])
def test_single_equals_slab(n, prec, form):
    for d, r in ((1, 37), (2, 9), (3, 5), (4, 5)):
        p = _problem(n, d, r, form)
        for steps in (STEPS, 9):  # narrow and bf16 staging
            got = _single(p, prec, steps)
            assert _same(got, _chosen(n, d, prec, p["J"], lambda: _single(p, prec, steps))), (d, steps)


@pytest.mark.parametrize("n,d,prec,forms", [(400, 4, "f32", ["i8", "i8"]), (390, 3, "f32", ["fp8"]),
                                            (800, 4, "f32", ["i8"]), (600, 2, "bf16", ["bf16"]), (300, 3, "f32", ["f32"])])
def test_batch_equals_slab(n, d, prec, forms):
    probs = [_problem(n, d, 6 + 11 * i, f) for i, f in enumerate(forms)]

    def run():
        tasks = [dict(p, x=p["x"].clone(), steps=STEPS - 3 * i, precision=prec) for i, p in enumerate(probs)]
        b = api.chym_batch_create(tasks)
        for _ in range(2):
            b.launch()
        torch.cuda.synchronize()
        b.destroy()
        return [t["x"] for t in tasks]

    for a, b in zip(run(), _chosen(n, d, prec, probs[0]["J"], run)):
        assert _same(a, b)


def test_batch_of_all_d_and_sizes_equals_singles():
    """The packed groups of a batch hold problems of every D and of several
    sizes, the recorded graph runs them beside the other groups."""
    shapes = [(257, 1, 5), (390, 2, 11), (512, 3, 7), (300, 4, 3), (800, 4, 6), (770, 2, 9), (40, 3, 20), (130, 2, 8)]
    probs = [_problem(n, d, r, "i8") for n, d, r in shapes]
    tasks = [dict(p, x=p["x"].clone(), steps=STEPS - i, precision="f32") for i, p in enumerate(probs)]
    b = api.chym_batch_create(tasks)
    for _ in range(2):
        for t, p in zip(tasks, probs):
            t["x"].copy_(p["x"])
        b.launch()
    torch.cuda.synchronize()
    b.destroy()
    for i, (t, p) in enumerate(zip(tasks, probs)):
        assert _same(t["x"], _single(p, "f32", STEPS - i)), shapes[i]
