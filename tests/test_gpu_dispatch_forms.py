"""Dispatched forms against a kernel that the caller chose, bit for bit: the
team integrator against the streamed-J slab kernel (which shares no code of its
lanes with it), entries of the autotuner and of plan files that give way, the
packed streamed-J integrator with several blocks to a compute unit; and the
batched energies beside a task of the largest size."""
import contextlib

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2308_02329_amd import api, synth  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
STEPS = 70


@contextlib.contextmanager
def chosen(n, d, prec, dtype, kernel, waves=8):
    api.chym_plan_set(n, d, prec, dtype, kernel, waves)
    try:
        yield
    finally:
        api.chym_plan_set(n, d, prec, dtype, api.CHYM_KERNEL_AUTO)


def _problem(n, d, r, j, seed=0):
    g = synth.rng(84, n, d, seed)
    J = torch.from_numpy(synth.sk_pm1(n, 84, n) if j == "i8" else synth.gaussian_j(n, 84, n)).to(DEV)
    if j == "bf16":
        J = J.to(torch.bfloat16)
    pump = torch.from_numpy(g.uniform(0.5, 2.0, r).astype(np.float32)).to(DEV)
    x = torch.from_numpy((g.standard_normal((n, r, d)) * 0.3).astype(np.float32)).to(DEV)
    alpha = torch.from_numpy(g.uniform(0.0, 1.0, (STEPS + 1, d)).astype(np.float32)).to(DEV)
    return dict(J=J, pump=pump, x=x, alpha=alpha, eps=0.04, btil=1.0, eta=2e-4, dt=0.01, start_step=1)


def _single(p, prec, steps=STEPS):
    x = p["x"].clone()
    api.chym_integrate(p["J"], p["pump"], x, p["alpha"], precision=prec, steps=steps,
                       **{k: p[k] for k in ("eps", "btil", "eta", "dt", "start_step")})
    return x


def _batch(probs, prec):
    tasks = [dict(p, x=p["x"].clone(), steps=STEPS, precision=prec) for p in probs]
    b = api.chym_batch_create(tasks)
    b.launch()
    torch.cuda.synchronize()
    b.destroy()
    return [t["x"] for t in tasks]


def _same(a, b):
    return torch.equal(a.view(torch.int32), b.view(torch.int32))


@pytest.mark.parametrize("n", [1, 16, 17, 32, 33, 64, 65, 100, 128, 129, 192, 225, 256])
@pytest.mark.parametrize("prec,j", [("f32", "i8"), ("bf16", "bf16"), ("f32", "f32")])
def test_team_equals_slab(n, prec, j):
    """The slab kernel takes the problem padded with uncoupled zero rows."""
    m = 272
    for d in (1, 2, 3, 4):
        p = _problem(n, d, 37, j)
        Jp = torch.zeros((m, m), dtype=p["J"].dtype, device=DEV)
        Jp[:n, :n] = p["J"]
        xp = torch.zeros((m, 37, d), device=DEV)
        xp[:n] = p["x"]
        with chosen(m, d, prec, Jp.dtype, api.CHYM_KERNEL_SLAB):
            ref = _single(dict(p, J=Jp, x=xp), prec)[:n].contiguous()
        assert _same(_single(p, prec), ref), d


@pytest.mark.parametrize("n,d,prec,kernel,waves", [(100, 3, "f32", "REGJ", 4), (100, 2, "f32", "PIPE", 4), (60, 1, "bf16", "LDSJ", 4),
                                                   (200, 3, "f32", "SLAB", 8), (230, 2, "bf16", "SLAB", 16),
                                                   (600, 4, "f32", "SLAB", 8)])
def test_entry_of_a_plan_file_gives_way(n, d, prec, kernel, waves, tmp_path):
    """An underfilled batch takes the team or the packed streamed-J integrator
    although a plan file names another kernel; chym_plan_get still reports the
    entry, and the results are those of the entry's kernel."""
    probs = [_problem(n, d, r, "i8", r) for r in (5, 33)]
    path = str(tmp_path / "plans")
    with chosen(n, d, prec, torch.int8, getattr(api, "CHYM_KERNEL_" + kernel), waves):
        want = _batch(probs, prec)
        api.chym_plan_save(path)
    api.chym_plan_load(path)
    try:
        entry = api.chym_plan_get(n, d, prec, torch.int8)
        assert entry["kernel"] == getattr(api, "CHYM_KERNEL_" + kernel) and entry["waves"] == waves
        got = _batch(probs, prec)
        if kernel == "SLAB":
            got.append(_single(probs[0], prec))
            want.append(want[0])
    finally:
        api.chym_plan_set(n, d, prec, torch.int8, api.CHYM_KERNEL_AUTO)
    for a, b in zip(got, want):
        assert _same(a, b)


@pytest.mark.parametrize("n,d,j,r", [(520, 4, "i8", 1030), (600, 4, "i8", 3069), (1024, 3, "i8", 1500), (520, 3, "f32", 2045),
                                     (800, 4, "f32", 1100)])
def test_packed_streamed_with_several_blocks_per_unit(n, d, j, r):
    """257 to 768 blocks of four replicas on 256 compute units."""
    p = _problem(n, d, r, j)
    with chosen(n, d, "f32", p["J"].dtype, api.CHYM_KERNEL_SLAB):
        want = _single(p, "f32")
    assert _same(_single(p, "f32"), want)


@pytest.mark.parametrize("n,d,prec,j", [(257, 4, "f32", "i8"), (400, 2, "f32", "i8"), (833, 3, "f32", "i8"), (289, 3, "f32", "f32"),
                                        (520, 1, "bf16", "i8")])
def test_packed_streamed_equals_slab_where_amplitudes_overflow(n, d, prec, j):
    """Infinities and NaN stay in their replicas, and odd tile counts leave half a
    chunk without rows."""
    p = dict(_problem(n, d, 21, j), btil=0.0, eta=0.0, dt=1.0)
    p["pump"][::2] *= 200.0
    p["pump"][1::2] = 0.9
    p["eps"] = 0.001
    with chosen(n, d, prec, p["J"].dtype, api.CHYM_KERNEL_SLAB):
        want = _single(p, prec)
    got = _single(p, prec)
    assert torch.isnan(want[:, ::2]).any() and torch.isfinite(want[:, 1::2]).all()
    assert torch.equal(torch.isnan(got), torch.isnan(want))
    assert _same(torch.nan_to_num(got, nan=1.0), torch.nan_to_num(want, nan=1.0))


def test_batched_energies_beside_the_largest_size():
    """A task of N = 1024 gives its blocks 147 KB of LDS, and a sparse one of
    more than 1024 spins takes a wavefront per replica; the small tasks share
    their launches."""
    tasks, singles = [], []
    g = synth.rng(85)
    for n, d, r, j in ((1024, 4, 5, "f32"), (17, 2, 33, "f32"), (2000, 2, 3, "ell"), (40, 3, 21, "bf16"), (1024, 1, 18, "bf16"),
                       (100, 3, 50, "i8")):
        x = torch.from_numpy(g.standard_normal((n, r, d)).astype(np.float32)).to(DEV)
        J = (torch.from_numpy(api.ell_pack(synth.regular3_pm1(n, 86, n))).to(DEV) if j == "ell" else _problem(n, 1, 1, j)["J"])

        def outs():
            return dict(spins=torch.empty((r, api.spin_words(n)), dtype=torch.int64, device=DEV),
                        e_ising_f64=torch.empty(r, dtype=torch.float64, device=DEV),
                        e_hs=torch.empty(r, dtype=torch.float64, device=DEV))

        tasks.append(dict(J=J, pump=torch.ones(r, device=DEV), x=x, alpha=torch.ones((1, d), device=DEV), eps=0.1, btil=1.0,
                          eta=0.0, dt=0.01, steps=0, **outs()))
        s = outs()
        api.chym_readout(x, s["spins"], None, None)
        api.chym_ising_energy(J, s["spins"], None, s["e_ising_f64"])
        api.chym_hs_energy(J, x, s["e_hs"])
        singles.append(s)
    plan = api.chym_batch_create(tasks)
    plan.launch()
    torch.cuda.synchronize()
    plan.destroy()
    for t, s in zip(tasks, singles):
        for k, v in s.items():
            assert torch.equal(t[k], v), (k, tuple(t["x"].shape))
