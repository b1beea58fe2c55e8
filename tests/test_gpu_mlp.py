"""GPU predictor kernels (features, inference, gradients, Adam training)
against the numpy FP64 oracle, and GPU training against a closed form (the
least-squares fit of an affine target, reached in the network's linear
regime)."""
import numpy as np
import pytest

import synthetic as syn
from oracle import mlp
from tests._mlp_cases import AFFINE_SCHEDULE, affine_case

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2105_14156_amd import smash
    assert torch.cuda.is_available()
    ctx = smash.Context(0)
    yield torch, smash, ctx
    ctx.close()


def _rel(a, b):
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-30))


def test_features_match_oracle(env, oracle_mod):
    torch, smash, ctx = env
    A = syn.rmat(12, 8, 21, np.float32)
    B = syn.uniform_k_per_row(A.cols, 3000, 7, 22, np.float32)
    for (X, Y) in ((A, A), (A, B)):
        F = ctx.features(smash.to_device(X), smash.to_device(Y)).cpu().numpy()
        ref = mlp.features(X, Y)
        np.testing.assert_allclose(F, ref, rtol=2e-6, atol=1e-6)


@pytest.mark.parametrize("m", [1, 63, 64, 192, 193, 257, 449])
def test_features_row_split(env, m):
    """Row analysis at the edges of its split (rows of up to 128 entries by
    eight lanes, longer ones by a wave each): every row count around whole
    waves and blocks, long and empty rows first, last and in clusters."""
    torch, smash, ctx = env
    lens = np.array([129, 0, 3000, 128, 1, 127, 513, 7])[np.arange(m) % 8]
    lens[-1] = 2000
    cols = 4000
    ptr = np.zeros(m + 1, np.int32)
    ptr[1:] = np.cumsum(lens)
    col = np.concatenate([np.arange(k, dtype=np.int32) + (i % 500) for i, k in enumerate(lens)])
    X = syn.CSR(m, cols, ptr, col, np.ones(len(col), np.float32))
    Y = syn.rmat_rect(cols, 4, 9, np.float32)
    F = ctx.features(smash.to_device(X), smash.to_device(Y)).cpu().numpy()
    np.testing.assert_allclose(F, mlp.features(X, Y), rtol=2e-6, atol=1e-6)


@pytest.mark.parametrize("m", [1, 400, 4095, 4096, 16383, 16384, 65536, 131073])
def test_features_long_row_split(env, m):
    """Rows at the limit between eight lanes and a wave (256 entries) and long
    ones at every number of rows that a wave looks at (1 to 64, by m)."""
    torch, smash, ctx = env
    lens = np.array([257, 1, 0, 255, 2, 256, 3, 1500])[(np.arange(m) + 7) % 8]
    if m > 5000:
        lens = np.where(np.arange(m) % 41 == 0, lens, np.arange(m) % 4)
    lens[-1] = 300
    cols = 2500
    ptr = np.zeros(m + 1, np.int32)
    ptr[1:] = np.cumsum(lens)
    col = (np.arange(ptr[-1]) - np.repeat(ptr[:-1], lens) + np.repeat(np.arange(m) % 900, lens)).astype(np.int32)
    X = syn.CSR(m, cols, ptr, col, np.ones(len(col), np.float32))
    Y = syn.rmat_rect(cols, 4, 9, np.float32)
    F = ctx.features(smash.to_device(X), smash.to_device(Y)).cpu().numpy()
    np.testing.assert_allclose(F, mlp.features(X, Y), rtol=2e-6, atol=1e-6)


@pytest.mark.parametrize("m", [3 << 19, (3 << 19) + 1])
def test_features_tall(env, m):
    """Rows around both limits between eight lanes and a wave (128 and 256
    entries) where the lower one begins to apply."""
    torch, smash, ctx = env
    lens = np.arange(m) % 2
    at = np.array([0, 1, 2, 63, 64, 1000, m // 2, m - 70, m - 2, m - 1])
    lens[at] = [127, 128, 129, 255, 256, 257, 1500, 200, 128, 129]
    cols = 2500
    ptr = np.zeros(m + 1, np.int32)
    ptr[1:] = np.cumsum(lens)
    col = (np.arange(ptr[-1]) - np.repeat(ptr[:-1], lens) + np.repeat(np.arange(m) % 900, lens)).astype(np.int32)
    X = syn.CSR(m, cols, ptr, col, np.ones(len(col), np.float32))
    Y = syn.rmat_rect(cols, 4, 9, np.float32)
    got = ctx.features(smash.to_device(X), smash.to_device(Y)).cpu().numpy()
    some = np.unique(np.concatenate([at, np.arange(0, m, 997)]))
    n = lens[some]
    sptr = np.concatenate([[0], np.cumsum(n)]).astype(np.int32)
    scol = np.concatenate([col[ptr[i]:ptr[i + 1]] for i in some])
    part = syn.CSR(len(some), cols, sptr, scol, np.ones(len(scol), np.float32))
    np.testing.assert_allclose(got[some], mlp.features(part, Y), rtol=2e-6, atol=1e-6)


def _setup(torch, n=3000, seed=3):
    F = np.abs(syn.normal01(seed, 0, n * 6).reshape(n, 6)) * 4
    y = F[:, 1] * 0.7 + np.sin(F[:, 0]) + 0.1 * syn.normal01(seed + 1, 0, n)
    mean, std = F.mean(0), F.std(0)
    ms = np.concatenate([mean, std])
    th = syn.mlp_init(seed) + 0.01 * syn.normal01(seed + 2, 0, syn.MLP_PARAMS)
    t = lambda a, dt=torch.float32: torch.from_numpy(np.ascontiguousarray(a)).to("cuda", dt)
    return F, y, ms, th, t


def test_predict_and_gradient_parity(env):
    torch, smash, ctx = env
    F, y, ms, th, t = _setup(torch)
    X = (F - ms[:6]) / ms[6:]
    yhat = ctx.mlp_predict(t(F), t(th), t(ms)).cpu().numpy()
    ref, _ = mlp.forward(th, X)
    assert np.max(np.abs(yhat - ref)) < 1e-4 * max(1.0, np.abs(ref).max())
    idx = np.sort((syn.uniform01(9, 0, 1000) * len(y)).astype(np.int32))
    loss, grad = ctx.mlp_loss_grad(t(F), t(y), t(idx, torch.int32), t(ms), t(th))
    rloss, rgrad = mlp.loss_grad(th, X[idx], y[idx])
    assert abs(loss - rloss) <= 1e-5 * rloss
    g = grad.cpu().numpy().astype(np.float64)
    pos = 0
    for name, shape in syn.MLP_LAYOUT:
        k = int(np.prod(shape))
        assert _rel(g[pos:pos + k], rgrad[pos:pos + k]) < 1e-4, name
        pos += k


@pytest.mark.parametrize("m", [1, 31, 32, 33, 129, 65536, 65573])
def test_predict_tile_edges(env, m):
    """Row counts around one tile of 32 rows, one block of four tiles and the
    largest grid (512 blocks: 65536 rows), where a wave takes a second tile.
    FP32 sums of 64 terms: as in the parity test above.  A NaN feature
    stays in its row."""
    torch, smash, ctx = env
    F, y, ms, th, t = _setup(torch, n=65573, seed=17)
    F = F[:m]
    X = (F - ms[:6]) / ms[6:]
    ref, _ = mlp.forward(th, X)
    feats = t(F)
    out = ctx.mlp_predict(feats, t(th), t(ms))
    assert out.shape[0] == m
    yhat = out.cpu().numpy()
    assert np.max(np.abs(yhat - ref)) < 1e-4 * max(1.0, np.abs(ref).max())
    feats[m // 2, 3] = float("nan")
    again = ctx.mlp_predict(feats, t(th), t(ms)).cpu().numpy()
    keep = np.arange(m) != m // 2
    assert np.array_equal(again[keep], yhat[keep])


@pytest.mark.parametrize("n", [1, 64, 65, 16384, 16449])
def test_gradient_tile_edges(env, n):
    """Batches around one tile of 64 samples and around one tile per block of
    the largest grid (256): one lane, a full tile, a remainder, a second tile
    in one block.  Gradients are FP64 sums rounded once (2^-24 relative), their
    FP32 terms carry the forward pass's roundings (about 70 dependent
    operations of 2^-24 each, amplified by cancellation): 1e-4 of each block's
    norm."""
    torch, smash, ctx = env
    F, y, ms, th, t = _setup(torch, n=3000, seed=13)
    X = (F - ms[:6]) / ms[6:]
    idx = (syn.uniform01(19, 0, n) * len(y)).astype(np.int32)
    loss, grad = ctx.mlp_loss_grad(t(F), t(y), t(idx, torch.int32), t(ms), t(th))
    rloss, rgrad = mlp.loss_grad(th, X[idx], y[idx])
    assert abs(loss - rloss) <= 1e-5 * rloss
    g = grad.cpu().numpy().astype(np.float64)
    pos = 0
    for name, shape in syn.MLP_LAYOUT:
        k = int(np.prod(shape))
        assert _rel(g[pos:pos + k], rgrad[pos:pos + k]) < 1e-4, name
        pos += k


def test_training_parity(env):
    torch, smash, ctx = env
    F, y, ms, th, t = _setup(torch, n=2000, seed=5)
    orders = syn.batch_orders(len(y), 4, 77)
    p = t(th)
    losses = ctx.mlp_train(t(F), t(y), t(ms), p, t(orders, torch.int32), batch=256, lr=1e-3)
    rth, rlosses = mlp.train(th, F, y, ms[:6], ms[6:], orders, 256, lr=1e-3)
    np.testing.assert_allclose(losses, rlosses, rtol=1e-3)
    assert _rel(p.cpu().numpy().astype(np.float64), rth) < 1e-4
    assert losses[-1] < losses[0]


def test_training_affine_target_reaches_lstsq(env):
    """smash_mlp_train (full-batch Adam, FP32) on an exact affine target from
    the linear regime ends at numpy's least-squares fit."""
    torch, smash, ctx = env
    F, y, mean, std, th, fitted = affine_case()
    n = len(y)
    t = lambda a, dt=torch.float32: torch.from_numpy(np.ascontiguousarray(a)).to("cuda", dt)
    ms = t(np.concatenate([mean, std]))
    p = t(th)
    for lr, epochs in AFFINE_SCHEDULE:
        losses = ctx.mlp_train(t(F), t(y), ms, p, t(syn.batch_orders(n, epochs, 3), torch.int32), batch=n, lr=lr)
    yhat = ctx.mlp_predict(t(F), p, ms).cpu().numpy().astype(np.float64)
    dev = float(np.max(np.abs(yhat - fitted)))
    print(f"max |yhat - lstsq fit| = {dev:.2e} (fit spread {fitted.std():.2f}); final loss {losses[-1]:.2e}")
    assert dev < 1e-2
    assert losses[-1] < 1e-5 * y.var()
