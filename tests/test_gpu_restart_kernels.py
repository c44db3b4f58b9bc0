"""Kernels of the restart decision and the network at the edges of their tiles
and blocks, against the float64 reference."""
import numpy as np
import pytest

import oracle
from oracle import mlp
from paper_2308_02329_amd import api, synth

torch = pytest.importorskip("torch")
from gpu_helpers import pack_spins, to_dev  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,r,d", [(1, 3, 1), (15, 33, 2), (16, 32, 3), (17, 31, 4), (63, 1, 2), (64, 70, 3), (65, 16, 1),
                                   (129, 40, 4), (333, 20, 3), (1000, 35, 2), (1300, 17, 3), (2300, 18, 1), (2600, 5, 2)])
@pytest.mark.parametrize("j", ["i8", "f32", "bf16", "fp8"])
def test_features_edges(n, r, d, j):
    """32 replicas a block, 16 beyond about 1100 spins, one a wavefront beyond
    about 2400; ragged replica counts; couplings that are not symmetric."""
    g = np.random.default_rng([n, r])
    Jf = g.standard_normal((n, n)).astype(np.float32)
    if j == "i8":
        Jf = np.clip(np.round(Jf * 30), -128, 127).astype(np.float32)
        J, val = to_dev(Jf.astype(np.int8)), Jf
    elif j == "fp8":
        J = api.chym_quantize_fp8(to_dev(Jf))
        val = (J[:n].view(torch.float8_e4m3fn).double() * torch.exp2(J[n].double() - 127.0)[:, None]).cpu().numpy()
    else:
        J = to_dev(Jf) if j == "f32" else to_dev(Jf).to(torch.bfloat16)
        val = J.double().cpu().numpy()
    x_prev = g.standard_normal((n, r, d)).astype(np.float32)
    x = (x_prev + 0.7 * g.standard_normal((n, r, d))).astype(np.float32)
    if r > 4:
        x[:, 4] = 0.0
    words = api.chym_sign_words(to_dev(x_prev))
    np.testing.assert_array_equal(words.cpu().numpy(), pack_spins(oracle.readout(x_prev)))
    feat = torch.zeros((r, 32), dtype=torch.float32, device="cuda")
    api.chym_features(J, to_dev(x), words, feat, 5)
    ref, sig = mlp.features(val, x, oracle.readout(x_prev))
    f = feat.cpu().numpy()
    assert not f[:, :20].any() and not f[:, 24:].any()
    # float32 chains of n products per column and n / 64 columns per class, then 6 sums
    x1 = x[:, :, 0].astype(np.float64)
    s1 = np.maximum((x1 * x1).sum(0), 1e-30)
    ops = (n + n / 64 + 10) * 2.0**-24
    tol0 = ops * np.einsum("pr,pr->r", np.abs(x1), np.abs(val).T @ np.abs(x1)) / (n * s1) + 1e-7
    assert np.all(np.abs(f[:, 20] - ref[:, 0]) <= tol0 + 2.0**-22 * np.abs(ref[:, 0]))
    assert np.all(np.abs(f[:, 21] - ref[:, 1]) <= ops * np.abs(val).sum() / n + 1e-7)
    np.testing.assert_allclose(f[:, 22], ref[:, 2], rtol=ops + 2.0**-22)
    np.testing.assert_array_equal(f[:, 23], ref[:, 3].astype(np.float32))
    np.testing.assert_array_equal(words.cpu().numpy(), pack_spins(sig))


@pytest.mark.parametrize("groups,group", [(1, 1), (2, 255), (3, 256), (1, 257), (5, 1025), (2, 4100)])
def test_standardize_and_select_edges(groups, group):
    g = np.random.default_rng(group)
    F = (g.standard_normal((groups * group, 32)) * 2 - 1).astype(np.float32)
    F[:, 3] = 0.25
    S = api.chym_feature_standardize(to_dev(F), group).cpu().numpy()
    np.testing.assert_allclose(S, mlp.standardize(F, group), rtol=1e-4, atol=2e-5)
    score = np.round(g.standard_normal(groups * group) * 2, 1).astype(np.float32)
    score[:: 7] = np.nan
    score[:: 11] = np.inf
    score[3:: 13] = -np.inf
    score[5:: 17] = -0.0
    score[6:: 17] = 0.0
    for keep in sorted({1, max(1, group // 20), max(1, group // 2), group}):
        idx = api.chym_select_top(to_dev(score), group, keep).cpu().numpy()
        np.testing.assert_array_equal(idx, _select(score, group, keep))


def _select(score, group, keep):
    """The keep highest of each group by the order of the float bits (-0 below
    +0, NaN lowest), equal ones by index, ascending."""
    b = score.view(np.uint32).astype(np.int64)
    key = np.where(np.isnan(score), 0, np.where(b >> 31, 0xFFFFFFFF - b, b + 0x80000000))
    out = []
    for k in range(score.size // group):
        sl = slice(k * group, (k + 1) * group)
        out.append(np.sort(np.argsort(-key[sl], kind="stable")[:keep]) + k * group)
    return np.array(out, dtype=np.int32)


@pytest.mark.parametrize("b", [1, 15, 16, 17, 31, 33, 64, 1000, 8192, 8193, 20000])
def test_network_passes_at_ragged_batches(b):
    """Forward and backward at the edges of the 16-sample groups, the 32-sample
    chunks and the blocks' chunk loop, against float64 on the GPU's own
    activations: the gradient's float32 sums of b products, the loss terms."""
    g = np.random.default_rng(b)
    w = to_dev((g.standard_normal(mlp.PARAMS) * 0.2).astype(np.float32))
    wb = api.chym_to_bf16(w)
    p = (wb.to(torch.int32) << 16).view(torch.float32).double()
    W1, b1, W2, b2, w3, b3 = torch.split(p, [4096, 128, 16384, 128, 128, 1])
    W1, W2 = W1.view(128, 32), W2.view(128, 128)
    x = to_dev(g.standard_normal((b, 32)).astype(np.float32))
    y = to_dev((g.random(b) < 0.3).astype(np.float32))
    f = lambda *s: torch.full(s, float("nan"), device="cuda")  # noqa: E731
    logit, h1, h2, loss, grad = f(b), f(b, 128), f(b, 128), f(b), f(mlp.PARAMS)
    api.chym_mlp_forward(x, wb, logit, h1, h2)
    only = api.chym_mlp_forward(x, wb)
    assert torch.equal(only, logit)
    xb = x.to(torch.bfloat16).double()
    a1 = torch.relu(xb @ W1.T + b1)
    # h1: within one bf16 step of the float64 activation
    assert bool(((h1.double() - a1).abs() <= a1 * 2.0**-8 + 1e-5).all())
    a2 = torch.relu(h1.double() @ W2.T + b2)
    s2 = h1.double().abs() @ W2.abs().T + b2.abs()
    assert bool(((h2.double() - a2).abs() <= 140 * 2.0**-24 * s2).all())
    z = h2.double() @ w3 + b3
    assert bool(((logit.double() - z).abs() <= 140 * 2.0**-24 * (h2.double() @ w3.abs() + b3.abs())).all())
    scratch = torch.full((api.chym_mlp_scratch_floats(b),), float("nan"), device="cuda")
    api.chym_mlp_backward(x, y, wb, logit, h1, h2, scratch, grad, loss)
    zd, yd = logit.double(), y.double()
    ref = torch.nn.functional.softplus(zd) - yd * zd
    assert bool(((loss.double() - ref).abs() <= 8 * 2.0**-24 * (1 + zd.abs())).all())
    dz = (torch.sigmoid(zd) - yd) / b
    d2 = (dz[:, None] * w3) * (h2 > 0)
    d1 = (d2 @ W2) * (h1 > 0)
    m1 = (d2.abs() @ W2.abs()) * (h1 > 0)
    H1, H2 = h1.double(), h2.double()
    want = torch.cat([(d1.T @ xb).flatten(), d1.sum(0), (d2.T @ H1).flatten(), d2.sum(0), H2.T @ dz, dz.sum()[None]])
    size = torch.cat([(m1.T @ xb.abs()).flatten(), m1.sum(0), (d2.abs().T @ H1).flatten(), d2.abs().sum(0),
                      H2.T @ dz.abs(), dz.abs().sum()[None]])
    # the sigmoid to a few units of its value 1/b each, 128 products per d1, chains of 32 per chunk, the
    # blocks' chunks and the partial gradients
    ops = 8 + 130 + 32 + 64 + b / 8192
    slack = 4 * 2.0**-24 * torch.cat([((torch.ones_like(dz)[:, None] * w3.abs()) * (h2 > 0) @ W2.abs()).T.matmul(xb.abs()).flatten(),
                                      ((torch.ones_like(dz)[:, None] * w3.abs()) * (h2 > 0) @ W2.abs()).sum(0),
                                      ((w3.abs() * (h2 > 0)).T @ H1).flatten(), (w3.abs() * (h2 > 0)).sum(0), H2.sum(0),
                                      torch.full((1,), float(b), device="cuda", dtype=torch.float64)]) / b
    assert bool(((grad.double() - want).abs() <= ops * 2.0**-24 * size + slack).all())
