"""The reduced eigenproblem at the edges of its kernels' widths (16, 32, 48 and 64
columns; nu = 1 and 2, where no reduction to tridiagonal form is needed), with
given and with bisected chemical potential.

The subspaces are well conditioned (q = 0 where nu nears the dimension), so the
solve differs from the oracle by rounding only: 1e-10 on rho and pi and 1e-9 on
the Ritz values (norm of the pencils about 10, 1e6 ulp)."""

import math

import numpy as np
import pytest

from paper_1202_0098_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p,q", [(1, 0), (1, 1), (2, 1), (8, 7), (8, 8), (9, 8), (16, 15), (16, 16),
                                 (17, 16), (25, 20), (47, 0), (48, 0), (49, 0), (63, 0), (64, 0)])
@pytest.mark.parametrize("bisect", [False, True])
def test_widths(p, q, bisect):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle
    import paper_1202_0098_amd as ma
    s = synth.random_pencil(24, 4, seed=31)
    nu, mu = p + q, math.nan if bisect else 0.2
    ctx = ma.Context(0)
    ctx.build_tb(s)
    cols = np.arange(5, 29, dtype=np.int32)
    n_target = 0.5 * len(cols)
    print(f"[gpu-case] pencil n={s.M} p={p} q={q} bisect={bisect}", flush=True)
    rho = torch.zeros(s.nblk * 16, dtype=torch.float64, device="cuda")
    pi = torch.zeros_like(rho)
    eps = torch.zeros(len(cols) * nu, dtype=torch.float64, device="cuda")
    r = ctx.solve_columns(cols, p, q, mu=mu, kT=0.25, rho=rho, pi=pi, eps=eps,
                          opts=ma.default_opts(n_target=n_target))
    raw = oracle.solve_raw(s, cols=cols, p=p, q=q)
    if bisect:
        mu = oracle.find_mu(raw, 0.25, n_target)
        assert abs(r.mu - mu) <= 1e-9 * max(1.0, abs(mu))
    rho_o, pi_o, E, N = oracle.outputs(s, raw, mu, 0.25)
    got = [x.cpu().numpy().reshape(s.nblk, 4, 4) for x in (rho, pi)]
    assert np.abs(eps.cpu().numpy().reshape(-1, nu) - raw["eps"]).max() <= 1e-9
    assert np.abs(got[0] - oracle.scatter_slots(s, cols, rho_o)).max() <= 1e-10
    assert np.abs(got[1] - oracle.scatter_slots(s, cols, pi_o)).max() <= 1e-10 * np.abs(pi_o).max()
    assert abs(r.energy - 2 * E.sum()) <= 1e-10 * abs(E).sum()
    ctx.close()


@pytest.mark.parametrize("nu", [1, 2, 3, 31, 32, 33, 64])
def test_stored_fp32_amplitudes(nu):
    """The kernel of the mixed modes with mu bisected (two lanes per column up to
    32 columns).  The operator is rounded to FP32: 6e-8 of a norm of about 10
    moves an occupation by 6e-7 / 4 kT and a Ritz value by 6e-7; an order of
    magnitude for the subspace."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle
    import paper_1202_0098_amd as ma
    s = synth.random_pencil(24, 4, seed=31)
    ctx = ma.Context(0)
    ctx.build_tb(s)
    cols = np.arange(5, 29, dtype=np.int32)
    print(f"[gpu-case] pencil n={s.M} nu={nu} mixed_f64acc", flush=True)
    rho = torch.zeros(s.nblk * 16, dtype=torch.float64, device="cuda")
    r = ctx.solve_columns(cols, nu, 0, kT=0.25, rho=rho,
                          opts=ma.default_opts(n_target=12.0, precision="mixed_f64acc"))
    raw = oracle.solve_raw(s, cols=cols, p=nu, q=0)
    rho_o = oracle.outputs(s, raw, r.mu, 0.25)[0]
    assert abs(r.mu - oracle.find_mu(raw, 0.25, 12.0)) <= 1e-5
    assert np.abs(rho.cpu().numpy().reshape(s.nblk, 4, 4) - oracle.scatter_slots(s, cols, rho_o)).max() <= 1e-5
    ctx.close()
