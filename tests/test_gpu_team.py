"""The team integrator (row tiles spread over a block's wavefronts) against the
other integrators of the same problem, bit for bit: a problem padded with
uncoupled zero rows beyond 16 row tiles runs on the streamed-J kernel, and many
replicas of a small one on one wavefront per 16 replicas."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2308_02329_amd import api, synth  # noqa: E402

pytestmark = pytest.mark.gpu

STEPS = 40


def _inputs(n, d, r, j, seed=3):
    dev = torch.device("cuda:0")
    g = synth.rng(77, n, d, seed)
    J = synth.gaussian_j(n, 77, n) if j != "i8" else synth.sk_pm1(n, 77, n)
    J = torch.from_numpy(J).to(dev)
    J = J.to(torch.bfloat16) if j == "bf16" else J
    pump = torch.from_numpy(g.uniform(0.5, 2.0, r).astype(np.float32)).to(dev)
    x = torch.from_numpy((g.standard_normal((n, r, d)) * 0.3).astype(np.float32)).to(dev)
    alpha = torch.from_numpy(g.uniform(0.0, 1.0, (STEPS + 3, d)).astype(np.float32)).to(dev)
    return J, pump, x, alpha


def _run(J, pump, x, alpha, prec, **kw):
    x = x.clone()
    args = dict(eps=0.04, btil=1.0, eta=2e-4, dt=0.01, steps=STEPS, start_step=2)
    args.update(kw)
    api.chym_integrate(J, pump, x, alpha, precision=prec, **args)
    return x


def _padded(J, pump, x, alpha, prec, m=272):
    n = x.shape[0]
    Jp = torch.zeros((m, m), dtype=J.dtype, device=J.device)
    Jp[:n, :n] = J
    xp = torch.zeros((m,) + tuple(x.shape[1:]), device=x.device)
    xp[:n] = x
    return _run(Jp, pump, xp, alpha, prec)[:n]


def _same(a, b):
    return torch.equal(a.view(torch.int32), b.view(torch.int32))


@pytest.mark.parametrize("n", [1, 16, 17, 31, 32, 33, 48, 63, 64, 65, 96, 100, 112, 127, 128, 129, 145, 192, 193, 225, 256])
@pytest.mark.parametrize("form", [("f32", "i8"), ("bf16", "bf16"), ("f32", "f32")])
def test_packed_layout_equals_streamed(n, form):
    for d in (1, 2, 3, 4):
        J, pump, x, alpha = _inputs(n, d, 37, form[1])
        assert _same(_run(J, pump, x, alpha, form[0]), _padded(J, pump, x, alpha, form[0])), d


@pytest.mark.parametrize("n,d,r", [(30, 3, 8203), (33, 3, 4109), (100, 3, 2053), (112, 3, 2053), (128, 2, 4101),
                                   (150, 4, 2053), (200, 3, 2053), (256, 3, 2050), (256, 4, 2050)])
@pytest.mark.parametrize("form", [("f32", "i8"), ("bf16", "bf16"), ("f32", "f32")])
def test_plane_layout_equals_streamed(n, d, r, form):
    J, pump, x, alpha = _inputs(n, d, r, form[1])
    assert _same(_run(J, pump, x, alpha, form[0]), _padded(J, pump, x, alpha, form[0]))


@pytest.mark.parametrize("n,d", [(100, 1), (48, 2), (112, 3), (50, 4)])
@pytest.mark.parametrize("r", [37, 4200])
def test_team_equals_one_wavefront(n, d, r):
    """Also where amplitudes overflow: 16384 replicas run one wavefront each
    16 of them, and a replica's values do not depend on the others."""
    J, pump, x, alpha = _inputs(n, d, 16384, "i8")
    kw = dict(btil=0.0, eta=0.0, dt=1.0)
    pump = pump * 200.0
    some = _run(J, pump[:r].contiguous(), x[:, :r].contiguous(), alpha, "f32", **kw)
    full = _run(J, pump, x, alpha, "f32", **kw)[:, :r].contiguous()
    assert not torch.isfinite(full).all()
    assert torch.equal(torch.isnan(some), torch.isnan(full))
    assert _same(torch.nan_to_num(some, nan=1.0), torch.nan_to_num(full, nan=1.0))


@pytest.mark.parametrize("j", ["i8", "bf16", "fp8", "f32"])
@pytest.mark.parametrize("n", [5, 31, 70, 99, 131])
def test_coupling_reads_at_every_alignment(n, j):
    """Rows whose length is no multiple of four: the four-column reads start
    at every byte alignment and the last columns are read one by one."""
    dev = torch.device("cuda:0")
    Jf = torch.from_numpy(synth.gaussian_j(n, 78, n)).to(dev)
    if j == "i8":
        Jf = torch.round(Jf * 20)
    stored = {"i8": lambda: Jf.to(torch.int8), "bf16": lambda: Jf.to(torch.bfloat16),
              "fp8": lambda: api.chym_quantize_fp8(Jf), "f32": lambda: Jf}[j]()
    if j == "fp8":
        e = torch.exp2(stored[n].double() - 127.0)[:, None]
        val = stored[:n].view(torch.float8_e4m3fn).double() * e
    else:
        val = stored.double()
    _, pump, x, alpha = _inputs(n, 2, 19, "f32")
    # one step from x with no gain and no loss: x + dt eps alpha J x
    out = _run(stored, torch.ones_like(pump), x, alpha, "f32", btil=0.0, eta=0.0, eps=1.0, steps=1, start_step=0)
    g = torch.matmul(val, x.double().reshape(n, -1)).view_as(x)
    ref = x.double() + np.float32(0.01) * alpha[0].double() * g
    # float32 sums of n products, one rounding each for weight, update and result
    tol = (n + 4) * 2.0**-24 * (x.double().abs() + 0.01 * torch.matmul(val.abs(), x.double().abs().reshape(n, -1)).view_as(x))
    assert bool(((out.double() - ref).abs() <= tol + 1e-30).all())


@pytest.mark.parametrize("n,d,prec,reps", [(20, 3, "f32", [5, 33]), (100, 3, "f32", [32, 7, 100]), (100, 1, "f32", [300] * 40),
                                           (100, 3, "bf16", [500] * 9), (200, 4, "bf16", [33, 2100]), (150, 2, "f32", [40])])
def test_batches_take_the_team_and_equal_a_chosen_kernel(n, d, prec, reps):
    """Default plans (packed and plane layouts, ragged replica counts) against
    a kernel chosen by the caller."""
    J, _, _, alpha = _inputs(n, d, 1, "i8")
    g = synth.rng(79, n, d)
    xs = [torch.from_numpy((g.standard_normal((n, r, d)) * 0.3).astype(np.float32)).to(J.device) for r in reps]
    pumps = [torch.from_numpy(g.uniform(0.5, 2.0, r).astype(np.float32)).to(J.device) for r in reps]

    def run():
        tasks = [dict(J=J, pump=p, x=x.clone(), alpha=alpha, eps=0.04, btil=1.0, eta=2e-4, dt=0.01, steps=STEPS - i,
                      start_step=1, precision=prec) for i, (x, p) in enumerate(zip(xs, pumps))]
        b = api.chym_batch_create(tasks)
        b.launch()
        torch.cuda.synchronize()
        b.destroy()
        return [t["x"] for t in tasks]

    team = run()
    slab = n > (144 if d == 2 else 128) and d > 1
    api.chym_plan_set(n, d, prec, torch.int8, api.CHYM_KERNEL_SLAB if slab else api.CHYM_KERNEL_REGJ, 8 if slab else 4)
    try:
        chosen = run()
    finally:
        api.chym_plan_set(n, d, prec, torch.int8, api.CHYM_KERNEL_AUTO)
    for a, b in zip(team, chosen):
        assert _same(a, b)
