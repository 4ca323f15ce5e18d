"""The automatic kernel for FP64 solves of spd cells: the atom kernel where most
columns of enough atoms are asked for and its workspaces fit, the workspace
kernel otherwise; the same results on every route."""

import math

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
    s = synth.config_fcc_spd(5, cells=(4, 4, 5))
    ctx.build_tb(s)
    yield torch, ma, ctx, s
    ctx.set_workspace(None)
    ctx.close()


def _solve(torch, ma, ctx, s, cols, p, q, kernel="auto", **kw):
    o = s.n_orb
    rho = torch.zeros(s.nblk * o * o, dtype=torch.float64, device="cuda")
    r = ctx.solve_columns(cols, p, q, mu=0.3, kT=s.kT, rho=rho, **kw,
                          opts=ma.default_opts(basis_kernel=kernel))
    torch.cuda.synchronize()
    return rho.cpu().numpy(), r


# all columns; 8 of 9; the least that takes the atom kernel (7 of 9); below it;
# columns out of order; too few atoms
@pytest.mark.parametrize("which", ["all", "eight", "seven", "six", "shuffled", "half"])
@pytest.mark.parametrize("p,q", [(1, 0), (4, 3)])
def test_every_selection_of_columns_agrees(env, which, p, q):
    torch, ma, ctx, s = env
    assert s.n_atoms > 256 and s.n_orb == 9
    per = {"eight": 8, "seven": 7, "six": 6}.get(which, 9)
    cols = np.array([9 * a + i for a in range(s.n_atoms) for i in range(per)], np.int32)
    if which == "shuffled":
        cols = np.random.default_rng(1).permutation(cols).astype(np.int32)
    if which == "half":
        cols = cols[:9 * 100]
    a, _ = _solve(torch, ma, ctx, s, cols, p, q)
    b, _ = _solve(torch, ma, ctx, s, cols, p, q, "workspace")
    # the bound of the parity tests between kernels
    assert np.abs(a - b).max() <= 1e-10


def test_a_small_workspace_takes_the_workspace_kernel(env):
    torch, ma, ctx, s = env
    cols = np.arange(s.M, dtype=np.int32)
    ref, _ = _solve(torch, ma, ctx, s, cols, 4, 3, "workspace")
    kw = dict(mu=0.3, opts=ma.default_opts())
    full = ctx.workspace_size(cols, 4, 3, **kw)
    small = ctx.workspace_size(cols, 4, 3, mu=0.3, opts=ma.default_opts(basis_kernel="workspace"))
    assert small < full
    for n in (full, small):
        buf = torch.empty(n, dtype=torch.uint8, device="cuda")
        ctx.set_workspace(buf)
        try:
            got, _ = _solve(torch, ma, ctx, s, cols, 4, 3)
        finally:
            ctx.set_workspace(None)
        assert np.abs(got - ref).max() <= 1e-10
    buf = torch.empty(small // 2, dtype=torch.uint8, device="cuda")
    ctx.set_workspace(buf)
    try:
        with pytest.raises(Exception, match="workspace"):
            _solve(torch, ma, ctx, s, cols, 4, 3)
    finally:
        ctx.set_workspace(None)
    # the allocation-free entry point, whatever its scratch holds
    got, _ = _solve(torch, ma, ctx, s, cols, 4, 3, noalloc=True)
    assert np.abs(got - ref).max() <= 1e-10
