"""The gather integrator's forms (rows in registers, in LDS, in global memory;
blocks of one to sixteen replicas) against float64 and each other."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2308_02329_amd import api, synth  # noqa: E402

pytestmark = pytest.mark.gpu


def _rows(n, w, g):
    """Dense couplings with at most w in a row, and their packed rows in
    which some entries, not the last alone, are missing."""
    J = np.zeros((n, n), np.float32)
    rows = np.zeros((n + 1, 2 * w), np.int32)
    rows[0, :2] = n, w
    for p in range(n):
        q = g.choice(n, min(w, n), replace=False)
        v = g.standard_normal(len(q)).astype(np.float32)
        gone = g.random(len(q)) < 0.2
        J[p, q[~gone]] = v[~gone]
        rows[p + 1, :w] = -1
        rows[p + 1, :len(q)] = np.where(gone, g.choice([-1, n, n + 7]), q)
        rows[p + 1, w:w + len(q)] = v.view(np.int32)
    return J, rows


def _run(rows, x, pump, alpha, steps, **kw):
    x = x.clone()
    api.chym_integrate(rows, pump, x, alpha, steps=steps, start_step=1, precision="f32", **kw)
    return x


# rows up to three couplings in registers; longer ones eight, four and one at a
# time, in LDS or (n = 300, w = 90) beyond its budget; n = 1025, 4061: four and one replica
# of a block at most
@pytest.mark.parametrize("n,w", [(1, 1), (5, 3), (64, 2), (200, 3), (1025, 3), (4061, 3), (50, 4), (65, 7), (65, 8), (120, 13),
                                 (150, 31), (300, 90), (700, 20)])
def test_rows_of_every_length(n, w):
    dev = torch.device("cuda:0")
    g = synth.rng(91, n, w)
    J, rows = _rows(n, w, g)
    rows = torch.from_numpy(rows).to(dev)
    for d in (1, 2, 3, 4):
        few, many = 3, 300 if n > 1000 else 4500
        x = torch.from_numpy((g.standard_normal((n, many, d)) * 0.3).astype(np.float32)).to(dev)
        pump = torch.from_numpy(g.uniform(0.5, 2.0, many).astype(np.float32)).to(dev)
        alpha = torch.from_numpy(g.uniform(0.0, 1.0, (12, d)).astype(np.float32)).to(dev)
        # one step with no gain and no loss: x + dt eps alpha J x
        out = _run(rows, x, torch.ones_like(pump), alpha, 1, eps=1.0, btil=0.0, eta=0.0, dt=0.01)
        Jd = torch.from_numpy(J).to(dev).double()
        lin = torch.matmul(Jd, x.double().reshape(n, -1)).view_as(x)
        mag = torch.matmul(Jd.abs(), x.double().abs().reshape(n, -1)).view_as(x)
        ref = x.double() + np.float32(0.01) * alpha[1].double() * lin
        # float32 sums of w products, one rounding each for weight, update and result
        tol = (w + 4) * 2.0**-24 * (x.double().abs() + 0.01 * mag)
        assert bool(((out.double() - ref).abs() <= tol + 1e-30).all()), d
        # a replica's values do not depend on the others
        kw = dict(eps=0.1, btil=1.0, eta=2e-4, dt=0.01)
        a = _run(rows, x, pump, alpha, 9, **kw)[:, :few].contiguous()
        b = _run(rows, x[:, :few].contiguous(), pump[:few].contiguous(), alpha, 9, **kw)
        assert torch.equal(a.view(torch.int32), b.view(torch.int32)), d
