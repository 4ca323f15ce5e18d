"""The network products and the density of states at the edges of their tiles:
batches around the 16-row tiles and the splits of K, energies around the tile of
512, and what each does with an index or an energy outside its range."""

import ctypes

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
    s = synth.config_diamond64()
    ctx.build_tb(s)
    ctx.mlp_init(seed=3)
    yield torch, ma, ctx, s
    ctx.close()


# the sums are FP32 over at most 1,000 rows or 256 inputs in three layers:
# 3 sqrt(1000) 2^-24 = 6e-6
@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 65, 1000])
def test_gradient_at_tile_edges(env, n):
    torch, ma, ctx, s = env
    from oracle import mlp
    sh = ctx.mlp_shape()
    rng = np.random.default_rng(n)
    X = rng.normal(size=(n, sh["n_in"])).astype(np.float32)
    T = (rng.normal(size=(n, sh["n_out"])) * 0.1).astype(np.float32)
    loss, g = ctx.mlp_loss_grad(torch.from_numpy(X).cuda(), torch.from_numpy(T).cuda(), n)
    loss_o, g_o = mlp.loss_grad(ctx.mlp_get_params().astype(np.float64), X.astype(np.float64),
                                T.astype(np.float64), (sh["n_in"], sh["n_hidden"], sh["n_out"]))
    print(f"[gpu-case] n {n}: loss {abs(loss - loss_o) / loss_o:.1e} "
          f"gradient {np.linalg.norm(g - g_o) / np.linalg.norm(g_o):.1e}", flush=True)
    assert abs(loss - loss_o) <= 1e-5 * loss_o
    assert np.linalg.norm(g - g_o) <= 1e-5 * np.linalg.norm(g_o)


@pytest.mark.parametrize("n", [1, 15, 17, 64, 100])
def test_inference_rows_are_independent(env, n):
    torch, ma, ctx, s = env
    sh = ctx.mlp_shape()
    rng = np.random.default_rng(7)
    X = torch.from_numpy(rng.normal(size=(100, sh["n_in"])).astype(np.float32)).cuda()
    full = torch.zeros(100, sh["n_out"], dtype=torch.float32, device="cuda")
    ctx.mlp_forward(X, 100, full, bf16=True)
    part = torch.full((101, sh["n_out"]), 7.0, dtype=torch.float32, device="cuda")
    ctx.mlp_forward(X[100 - n:].contiguous(), n, part, bf16=True)
    assert torch.equal(part[:n], full[100 - n:])
    assert bool((part[n:] == 7.0).all())


def test_an_index_outside_the_table_makes_no_update(env):
    torch, ma, ctx, s = env
    sh = ctx.mlp_shape()
    X = torch.randn(20, sh["n_in"], device="cuda")
    T = torch.randn(20, sh["n_out"], device="cuda")
    before = ctx.mlp_get_params()
    good = torch.arange(16, dtype=torch.int32, device="cuda")
    for bad in (-1, 20):
        idx = good.clone()
        idx[5] = bad
        with pytest.raises(Exception, match="outside the table"):
            ctx.mlp_train_step(X, T, 16, 1e-3, idx=idx)
        assert np.array_equal(ctx.mlp_get_params(), before)
        # nor has a caller's gradient buffer been written by a call that fails
        g = np.full(sh["n_params"], 3.0, np.float32)
        loss = ctypes.c_double(5.0)
        st = ctx._lib.ma_mlp_loss_grad(ctx._h, X.data_ptr(), T.data_ptr(), 20, idx.data_ptr(), 16,
                                       ctypes.byref(loss), g.ctypes.data)
        assert st != 0 and loss.value == 5.0 and np.all(g == 3.0)
    # the step counter has not moved either: as from a fresh optimizer
    ctx.mlp_train_step(X, T, 16, 1e-3, idx=good)
    got = ctx.mlp_get_params()
    ctx.mlp_init(seed=3)
    ctx.mlp_train_step(X, T, 16, 1e-3, idx=good)
    assert np.array_equal(ctx.mlp_get_params(), got)
    ctx.mlp_init(seed=3)


@pytest.mark.parametrize("nE,eta", [(1, 0.1), (15, 1e-3), (511, 0.1), (513, 1.0), (1025, 0.05)])
def test_dos_at_tile_edges(env, nE, eta):
    torch, ma, ctx, s = env
    import oracle
    o = s.n_orb
    rho = torch.zeros(s.nblk * o * o, dtype=torch.float64, device="cuda")
    ctx.solve_columns(None, s.p, s.q, kT=s.kT, rho=rho)
    E = np.linspace(-30.0, 25.0, nE)
    got = ctx.dos(E, eta=eta)
    ref = oracle.dos(oracle.solve_raw(s), E, eta=eta)
    # a Ritz value off by 1e-12 moves a Lorentzian by at most 1e-12 / eta of its height
    assert np.abs(got - ref).max() <= (1e-10 + 1e-11 / eta) * ref.max()
    # far away and at infinity the density vanishes; the other energies are as before
    E2 = E.copy()
    E2[-1] = np.inf
    got2 = ctx.dos(E2, eta=eta)
    assert got2[-1] == 0.0
    assert np.abs(got2[:-1] - got[:-1]).max(initial=0.0) <= 1e-14 * max(got.max(), 1e-300)
    E2[-1] = 1e170
    assert ctx.dos(E2, eta=eta)[-1] == 0.0
