"""The map's two column layouts (16 columns per block, or 16 replicas x D
planes) at the edges of their tiles and chunks: a launch of many replicas
takes the planes where they are built (D > 1), one of its replicas alone the
packed columns; a replica's values do not depend on the others."""
import numpy as np
import pytest

from paper_2308_02329_amd import api, synth

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _replicas(n, d):
    """Enough that packed blocks are more than the rule takes: 16 to a CU for one
    chunk of rows, 8 for two, 4 beyond; and a ragged last block."""
    per_cu = 16 if n <= 32 else 8 if n <= 64 else 4
    return 256 * per_cu * (16 // {1: 1, 2: 2, 3: 4, 4: 4}[d]) + 16 + 5


@pytest.mark.parametrize("n", [7, 16, 17, 32, 33, 64, 65, 96, 112])
@pytest.mark.parametrize("d", [1, 2, 3, 4])
@pytest.mark.parametrize("precision", ["f32", "bf16"])
def test_layouts_agree(n, d, precision):
    steps, r = 30, _replicas(n, d)
    g = synth.rng(83, n, d)
    J = torch.from_numpy(synth.sk_pm1(n, 83, n)).to(DEV)
    h = torch.from_numpy(g.uniform(0.1, 0.5, r).astype(np.float32)).to(DEV)
    x = torch.from_numpy((g.standard_normal((n, r, d)) * 0.05).astype(np.float32)).to(DEV)
    alpha = torch.from_numpy(g.uniform(0.0, 1.0, (steps + 2, d)).astype(np.float32)).to(DEV)
    kw = dict(b=0.01, loss=0.01, kl=0.1, beta_b2=25.0, jmag=0.05, steps=steps, start_step=2, precision=precision)
    for lo, hi in ((0, 21), (r - 22, r)):
        some, hs = x[:, lo:hi].contiguous(), h[lo:hi].contiguous()
        full = x.clone()
        api.chym_map_integrate(J, h, full, alpha, **kw)
        api.chym_map_integrate(J, hs, some, alpha, **kw)
        assert not torch.equal(some, x[:, lo:hi])
        assert torch.equal(full[:, lo:hi].contiguous().view(torch.int32), some.view(torch.int32))
