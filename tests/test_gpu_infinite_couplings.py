"""Energies of couplings that hold infinities (float storage accepts them): the
sum of the definition's terms, each a coupling times a product of spins or of
unit vectors, in float64."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2308_02329_amd import api  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _sum(terms):
    """-sum of the terms: infinite with all infinities of one sign, NaN else."""
    with np.errstate(invalid="ignore"):
        return -terms.sum()


@pytest.mark.parametrize("n", [1, 5, 16, 17, 33, 65, 100, 333])
@pytest.mark.parametrize("j", ["f32", "bf16"])
@pytest.mark.parametrize("where", ["last", "first", "both signs"])
def test_infinite_couplings(n, j, where):
    g = np.random.default_rng([n, len(where)])
    J = g.standard_normal((n, n)).astype(np.float32)
    p, q = (n - 1, n // 2) if where == "last" else (0, n // 3)
    J[p, q] = J[q, p] = np.inf
    if where == "both signs":
        J[n - 1, 0] = J[0, n - 1] = -np.inf
    Jd = torch.from_numpy(J).to(DEV)
    if j == "bf16":
        Jd = Jd.to(torch.bfloat16)
        J = Jd.float().cpu().numpy()
    J = J.astype(np.float64)
    for d, r in ((1, 17), (2, 9), (3, 11), (4, 6)):
        x = g.standard_normal((n, r, d)).astype(np.float32)
        xd = torch.from_numpy(x).to(DEV)
        spins = api.chym_sign_words(xd)
        e = torch.empty(r, dtype=torch.float64, device=DEV)
        hs = torch.empty(r, dtype=torch.float64, device=DEV)
        api.chym_ising_energy(Jd, spins, None, e)
        api.chym_hs_energy(Jd, xd, hs)
        u = x.astype(np.float64)
        u = u / np.sqrt((u * u).sum(axis=2, keepdims=True))
        s = np.where(x[:, :, 0] >= 0, 1.0, -1.0)
        tol = 8 * (n + 4) * 2.0**-53 * np.abs(J[np.isfinite(J)]).sum()
        for k in range(r):
            for got, want in ((e[k].item(), _sum(J * np.outer(s[:, k], s[:, k]))), (hs[k].item(), _sum(J * (u[:, k] @ u[:, k].T)))):
                assert np.array_equal(got, want, equal_nan=True) or abs(got - want) <= tol, (d, k, got, want)
