"""The force kernels alone, on every route: one launch (o <= 4, up to 16,384 blocks),
and block sums first, with 16 lanes and a wavefront per atom, for several o.

Random blocks against extended precision.  Sums of products whose additions lose
nothing have the products' roundings, about 0.4 u of each term (u = 2^-53), and the
result's own: 0.6 u of the result in the 2-norm; one u is asserted."""

import numpy as np
import pytest

from paper_1202_0098_amd import synth

pytestmark = pytest.mark.gpu
U = 2.0 ** -53


@pytest.fixture(scope="module")
def env():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1202_0098_amd as ma
    yield torch, ma


def _diamond(n, region):
    s = synth.build_tb(synth.diamond_positions(n, n, n, 5.43), np.full(3, 5.43 * n), synth.SP3_PARAMS)
    s.region_mode, s.region_nrp = "nearest", np.full(s.n_atoms, region, np.int32)
    return s


SYSTEMS = {
    "sp3 64 atoms": lambda: _diamond(2, 20),
    "sp3 5,832 atoms": lambda: _diamond(9, 8),
    "o = 4, 160 neighbours": lambda: synth.random_pencil(160, 4, seed=1, s_scale=0.01),
    "o = 1": lambda: synth.random_pencil(40, 1, seed=2),
    "o = 2": lambda: synth.random_pencil(170, 2, seed=3, s_scale=0.01),
    "o = 5": lambda: synth.random_pencil(12, 5, seed=4),
    "spd 108 atoms": lambda: synth.config_fcc_spd(5, cells=(3, 3, 3)),
}


def _blocks(s, seed):
    rng = np.random.default_rng(seed)
    o = s.n_orb
    return [rng.normal(size=n) for n in (s.nblk * o * o, s.nblk * o * o, 3 * s.nblk * o * o,
                                         3 * s.nblk * o * o)]


def _reference(s, rho, pi, dH, dS):
    L, oo = np.longdouble, s.n_orb ** 2
    row = np.repeat(np.arange(s.n_atoms), np.diff(s.blk_ptr))
    g = (rho.reshape(-1, 1, oo).astype(L) * dH.reshape(-1, 3, oo)
         - pi.reshape(-1, 1, oo).astype(L) * dS.reshape(-1, 3, oo)).sum(2)
    g[row == s.blk_col] = 0
    F = np.zeros((s.n_atoms, 3), L)
    np.add.at(F, s.blk_col, -2 * g)
    np.add.at(F, row, 2 * g)
    return F


def _forces(torch, ctx, s, *host):
    F = torch.full((3 * s.n_atoms + 1,), 7.0, dtype=torch.float64, device="cuda")
    rho, pi, dH, dS = (torch.from_numpy(x).cuda() for x in host)
    ctx.forces(dH, dS, rho, pi, F)
    F = F.cpu().numpy()
    assert F[-1] == 7.0
    return F[:-1].reshape(-1, 3)


@pytest.mark.parametrize("name", SYSTEMS)
def test_precision(env, name):
    torch, ma = env
    s = SYSTEMS[name]()
    ctx = ma.Context(0)
    ctx.build_tb(s)
    host = _blocks(s, 3)
    ref = _reference(s, *host)
    F = _forces(torch, ctx, s, *host)
    err = float(np.sqrt(((F - ref) ** 2).sum() / (ref ** 2).sum()))
    print(f"[gpu-case] {name}, {s.nblk} blocks: {err / U:.2f} u", flush=True)
    assert err <= U
    ctx.close()


@pytest.mark.parametrize("name", ["sp3 64 atoms", "sp3 5,832 atoms", "spd 108 atoms"])
def test_infinite_values_stay_where_they_are(env, name):
    """An infinite rho in one block makes the forces of its two atoms infinite (not
    NaN), and no other; NaN on the atom-diagonal blocks, which are not used, nothing."""
    torch, ma = env
    s = SYSTEMS[name]()
    oo = s.n_orb ** 2
    ctx = ma.Context(0)
    ctx.build_tb(s)
    rho, pi, dH, dS = _blocks(s, 4)
    before = _forces(torch, ctx, s, rho, pi, dH, dS)
    row = np.repeat(np.arange(s.n_atoms), np.diff(s.blk_ptr))
    rho.reshape(-1, oo)[row == s.blk_col] = np.nan
    k = int(np.nonzero(row != s.blk_col)[0][7])
    rho[k * oo + oo - 1] = np.inf
    dH.reshape(-1, 3, oo)[k, :, oo - 1] = [1.0, 2.0, 0.5]
    got = _forces(torch, ctx, s, rho, pi, dH, dS)
    assert np.all(got[row[k]] == np.inf) and np.all(got[s.blk_col[k]] == -np.inf)
    rest = np.setdiff1d(np.arange(s.n_atoms), [row[k], s.blk_col[k]])
    assert np.array_equal(got[rest], before[rest])
    ctx.close()
