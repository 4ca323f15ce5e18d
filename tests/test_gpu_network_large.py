"""The network products on both sides of the line between their two tile sizes: the
hidden layers (256 columns) change to 64 x 64 tiles at 10,177 rows, the output
layer (48 columns) at 40,897.  Forward, gradient, and gathered rows, against the
FP64 network."""

import numpy as np
import pytest

from paper_1202_0098_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1202_0098_amd as ma
    ctx = ma.Context(0)
    ctx.build_tb(synth.config_diamond64())
    ctx.mlp_init(seed=3)
    yield torch, ctx
    ctx.close()


def _tables(ctx, n, seed):
    sh = ctx.mlp_shape()
    rng = np.random.default_rng(seed)
    x = rng.normal(size=(n, sh["n_in"])).astype(np.float32)
    return x, (rng.normal(size=(n, sh["n_out"])) * 0.1).astype(np.float32), \
        (sh["n_in"], sh["n_hidden"], sh["n_out"])


@pytest.mark.parametrize("n", [10176, 10177, 10300, 40896, 40897, 50000])
def test_forward_rows(env, n):
    """FP32 sums of at most 256 products in three layers: 3 x 256 x 2^-24 = 5e-5 of
    the magnitude that the network has with every product positive."""
    torch, ctx = env
    from oracle import mlp
    x, _, shape = _tables(ctx, n, n)
    y = torch.full((n + 1, shape[2]), 7.0, dtype=torch.float32, device="cuda")
    print(f"[gpu-case] FP32 forward of {n} rows", flush=True)
    ctx.mlp_forward(torch.from_numpy(x).cuda(), n, y, bf16=False)
    y = y.cpu().numpy()
    assert np.all(y[n] == 7.0)
    # the first and last rows, and those around every tile edge of the last tiles
    at = np.unique(np.concatenate([np.arange(70), np.arange(n - 200, n), np.arange(0, n, 997)]))
    params = ctx.mlp_get_params().astype(np.float64)
    W1, b1, W2, b2, W3, b3 = mlp.unpack(params, *shape)
    ref = mlp.forward(params, x[at].astype(np.float64), shape)
    ref = ref[0] if isinstance(ref, tuple) else ref
    m = (np.abs(x[at]) @ np.abs(W1) + np.abs(b1)) @ np.abs(W2) + np.abs(b2)
    assert np.all(np.abs(y[at] - ref) <= 5e-5 * (m @ np.abs(W3) + np.abs(b3)))


@pytest.mark.parametrize("gather", [False, True])
def test_gradient_of_a_large_batch(env, gather):
    """FP32 sums over the rows: 3 sqrt(10300) 2^-24 = 1.8e-5."""
    torch, ctx = env
    from oracle import mlp
    n = 10300
    x, t, shape = _tables(ctx, n, 5)
    idx = np.random.default_rng(1).permutation(n).astype(np.int32)
    print(f"[gpu-case] gradient of {n} rows, gather {gather}", flush=True)
    loss, g = ctx.mlp_loss_grad(torch.from_numpy(x).cuda(), torch.from_numpy(t).cuda(), n,
                                idx=torch.from_numpy(idx).cuda() if gather else None)
    loss_o, g_o = mlp.loss_grad(ctx.mlp_get_params().astype(np.float64), x.astype(np.float64),
                                t.astype(np.float64), shape)
    assert abs(loss - loss_o) <= 1.8e-5 * loss_o
    assert np.linalg.norm(g - g_o) <= 1.8e-5 * np.linalg.norm(g_o)
