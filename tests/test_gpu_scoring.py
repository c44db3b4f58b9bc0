"""Readout and energies at the edges of their tiles and chunks, against plain
numpy of their definitions: 16-row segments and 64-bit words, 16-replica and
16/d-replica groups, couplings in every storage, single calls and batches."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2308_02329_amd import api, synth  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _state(n, r, d, seed=0):
    g = synth.rng(91, n, r, d, seed)
    x = g.standard_normal((n, r, d)).astype(np.float32)
    x[g.random((n, r)) < 0.02] = 0.0  # zero hyperspins
    x[0, 0, 0] = -0.0
    if r > 2:
        x[n - 1, 1, d - 1] = np.inf
        x[n // 2, 2, 0] = np.nan
    if r > 3:
        x[n - 1, 3, 0] = 1500.0
    return x


def _couplings(n, j):
    g = synth.rng(92, n)
    J = g.standard_normal((n, n)).astype(np.float32)  # not symmetric, diagonal set
    if j == "i8":
        J = np.clip(np.round(J * 40), -128, 127)
        stored = torch.from_numpy(J.astype(np.int8)).to(DEV)
        return stored, J.astype(np.float64)
    t = torch.from_numpy(J).to(DEV)
    if j == "f32":
        return t, J.astype(np.float64)
    if j == "bf16":
        return t.to(torch.bfloat16), t.to(torch.bfloat16).double().cpu().numpy()
    q = api.chym_quantize_fp8(t)
    val = q[:n].view(torch.float8_e4m3fn).double() * torch.exp2(q[n].double() - 127.0)[:, None]
    return q, val.cpu().numpy()


def _words(x):
    n, r, _ = x.shape
    w = np.zeros((r, (n + 63) // 64), dtype=np.uint64)
    for p in range(n):
        w[:, p // 64] |= (x[p, :, 0] >= 0).astype(np.uint64) << np.uint64(p % 64)
    return w.view(np.int64)


def _share(x):
    x2 = x * x
    tot = x2[:, :, 0].copy()
    ext = np.zeros_like(tot)
    for mu in range(1, x.shape[2]):
        tot = tot + x2[:, :, mu]
        ext = ext + x2[:, :, mu]
    with np.errstate(all="ignore"):
        q = np.where(tot > 0, ext / tot, 0)
    return np.where(np.isnan(q), 0, q).max(axis=0)


@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 64, 65, 127, 128, 129, 255, 257, 1000, 3000])
@pytest.mark.parametrize("d,r", [(1, 5), (2, 64), (3, 65), (4, 130)])
def test_readout(n, d, r):
    x = _state(n, r, d)
    xd = torch.from_numpy(x).to(DEV)
    spins = torch.empty((r, api.spin_words(n)), dtype=torch.int64, device=DEV)
    ext = torch.empty(r, dtype=torch.float64, device=DEV)
    div = torch.empty(r, dtype=torch.uint8, device=DEV)
    api.chym_readout(xd, spins, ext, div)
    assert np.array_equal(spins.cpu().numpy(), _words(x))
    with np.errstate(all="ignore"):
        bad = (~np.isfinite(x) | (np.abs(x) > 1e3)).any(axis=(0, 2))
    assert np.array_equal(div.cpu().numpy().astype(bool), bad)
    # float32 squares and sums in component order, the same as numpy's; one division
    np.testing.assert_allclose(ext.cpu().numpy(), _share(x).astype(np.float64), rtol=2.0**-22)


@pytest.mark.parametrize("n", [1, 3, 15, 16, 17, 50, 64, 65, 100, 129, 200, 333, 1024, 1100])
@pytest.mark.parametrize("j", ["i8", "f32", "bf16", "fp8"])
def test_energies(n, j):
    J, Jd = _couplings(n, j)
    for d, r in ((1, 17), (2, 9), (3, 16), (4, 5)):
        x = np.where(np.isfinite(_state(n, r, d)), _state(n, r, d), np.float32(0.5))
        xd = torch.from_numpy(x).to(DEV)
        spins = torch.from_numpy(_words(x)).to(DEV)
        e64 = torch.empty(r, dtype=torch.float64, device=DEV)
        e32 = torch.empty(r, dtype=torch.int32, device=DEV) if j == "i8" else None
        api.chym_ising_energy(J, spins, e32, e64)
        s = np.where(x[:, :, 0] >= 0, 1.0, -1.0)
        ref = -np.einsum("pr,pr->r", s, Jd @ s)
        if j == "i8":
            assert np.array_equal(e32.cpu().numpy(), ref.astype(np.int32))
            assert np.array_equal(e64.cpu().numpy(), ref)
        scale = np.abs(Jd).sum()
        assert np.abs(e64.cpu().numpy() - ref).max() <= 2 * n * 2.0**-53 * scale + 1e-300
        nrm = np.sqrt((x.astype(np.float64)**2).sum(axis=2, keepdims=True))
        u = np.where(nrm > 0, x / np.where(nrm > 0, nrm, 1), 0)
        ref = -sum(np.einsum("pr,pr->r", u[:, :, m], Jd @ u[:, :, m]) for m in range(d))
        hs = torch.empty(r, dtype=torch.float64, device=DEV)
        api.chym_hs_energy(J, xd, hs)
        assert np.abs(hs.cpu().numpy() - ref).max() <= 4 * (n + 4) * 2.0**-53 * scale + 1e-300


def test_batched_scoring_equals_single_calls():
    """Tasks whose replicas share a block's range: ragged counts, every
    storage and dimension, sparse rows, and a size beyond the block kernels."""
    tasks, singles = [], []
    g = synth.rng(93)
    for n, d, r, j in ((100, 3, 7, "i8"), (17, 1, 33, "f32"), (65, 2, 16, "bf16"), (40, 4, 3, "fp8"), (64, 3, 50, "ell"),
                       (200, 2, 41, "i8"), (1, 1, 1, "i8"), (333, 3, 5, "f32"), (100, 4, 21, "ell")):
        if j == "ell":
            J = torch.from_numpy(api.ell_pack(synth.regular3_pm1(n, 94, n))).to(DEV)
        else:
            J, _ = _couplings(n, j)
        x = torch.from_numpy(g.standard_normal((n, r, d)).astype(np.float32)).to(DEV)

        def outs():
            o = dict(spins=torch.empty((r, api.spin_words(n)), dtype=torch.int64, device=DEV),
                     e_ising_f64=torch.empty(r, dtype=torch.float64, device=DEV),
                     e_hs=torch.empty(r, dtype=torch.float64, device=DEV),
                     extra_frac=torch.empty(r, dtype=torch.float64, device=DEV),
                     diverged=torch.empty(r, dtype=torch.uint8, device=DEV))
            if j == "i8":
                o["e_ising"] = torch.empty(r, dtype=torch.int32, device=DEV)
            return o

        o = outs()
        tasks.append(dict(J=J, pump=torch.ones(r, device=DEV), x=x, alpha=torch.ones((1, d), device=DEV), eps=0.1,
                          btil=1.0, eta=0.0, dt=0.01, steps=0, **o))
        s = outs()
        api.chym_readout(x, s["spins"], s["extra_frac"], s["diverged"])
        api.chym_ising_energy(J, s["spins"], s.get("e_ising"), s["e_ising_f64"])
        api.chym_hs_energy(J, x, s["e_hs"])
        singles.append(s)
    plan = api.chym_batch_create(tasks)
    for _ in range(2):
        plan.launch()
    torch.cuda.synchronize()
    for t, s in zip(tasks, singles):
        for k, v in s.items():
            assert torch.equal(t[k], v), (k, tuple(t["x"].shape))
    plan.destroy()
