"""The on-chip kernel's register form (FP64, o = 4) at the edges of its shapes:
regions of exactly, one under and one over 256 and 512 orbitals, p + q at 16 and
32 and just past them, q above p (the chain outlasts block 1), no block 2 and
one vector, spaces that run out, several columns per workgroup.

Against the oracle with the FP64 bounds of the parity tests: max-abs rho 1e-10,
pi 1e-10 of its largest entry, effective sizes equal."""

import numpy as np
import pytest

from paper_1202_0098_amd import synth

pytestmark = pytest.mark.gpu


def _check(s, p, q, cols, mu, kT, **opt):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle
    import paper_1202_0098_amd as ma
    o = s.n_orb
    print(f"[gpu-case] {s.name} p={p} q={q} {opt}", flush=True)
    ctx = ma.Context(0)
    ctx.build_tb(s)
    rho = torch.zeros(s.nblk * o * o, dtype=torch.float64, device="cuda")
    pi = torch.zeros_like(rho)
    st = torch.zeros(s.M * ma.STATS, dtype=torch.int32, device="cuda")
    ctx.solve_columns(None, p, q, mu=mu, kT=kT, rho=rho, pi=pi, col_stats=st,
                      opts=ma.default_opts(**opt))
    st = st.cpu().numpy().reshape(s.M, ma.STATS)[cols]
    raw = oracle.solve_raw(s, cols=cols, p=p, q=q)
    rho_o, pi_o, _, _ = oracle.outputs(s, raw, mu, kT)
    atoms = np.unique(cols // o)
    rows = np.repeat(np.arange(s.n_atoms), np.diff(s.blk_ptr))
    full = np.isin(rows, atoms)   # every column of these atoms is in cols
    got = [x.cpu().numpy().reshape(s.nblk, o, o)[full] for x in (rho, pi)]
    want = [oracle.scatter_slots(s, cols, x)[full] for x in (rho_o, pi_o)]
    assert np.array_equal(st[:, 0], raw["nu_eff"])
    assert np.all(st[:, 3] == 0)
    assert np.abs(got[0] - want[0]).max() <= 1e-10
    assert np.abs(got[1] - want[1]).max() <= 1e-10 * np.abs(want[1]).max()
    ctx.close()


@pytest.mark.parametrize("nrp,p,q", [(63, 8, 8), (64, 9, 8), (65, 16, 16), (127, 15, 16), (128, 17, 15),
                                     (128, 6, 11), (64, 5, 11), (120, 12, 0), (100, 1, 1), (129, 10, 10),
                                     (128, 20, 13)])
def test_regions(nrp, p, q):
    rng = np.random.default_rng(11)
    pos = synth.diamond_positions(4, 4, 4, 5.43)
    s = synth.build_tb(pos + rng.normal(0, 0.05, size=pos.shape), [4 * 5.43] * 3, synth.SP3_PARAMS,
                       name=f"diamond512/{nrp}")
    s.region_mode = "nearest"
    s.region_nrp = np.full(s.n_atoms, nrp, np.int32)
    atoms = np.sort(rng.choice(s.n_atoms, 8, replace=False))
    cols = (atoms[:, None] * 4 + np.arange(4)).ravel().astype(np.int32)
    _check(s, p, q, cols, 1.0, 0.1)


@pytest.mark.parametrize("n_atoms,seed,p,q", [(3, 1, 8, 4), (6, 7, 1, 9), (3, 2, 6, 12), (2, 6, 3, 8),
                                              (2, 11, 2, 20), (6, 3, 16, 16), (1, 4, 3, 2)])
@pytest.mark.parametrize("kernel", ["auto", "onchip"])
def test_spaces_that_run_out(n_atoms, seed, p, q, kernel):
    if kernel == "onchip" and q > (8 if p + q <= 16 else 16):
        pytest.skip("refused by the on-chip kernel's shape rule")
    s = synth.random_pencil(n_atoms, 4, seed=seed)
    _check(s, p, q, np.arange(s.M, dtype=np.int32), 0.2, 0.25, basis_kernel=kernel)


def test_uneven_regions():
    """Rows with more blocks than are held in registers, regions of 8 to 128 atoms."""
    s = synth.config_disordered8000(3009, n_atoms=220)
    rng = np.random.default_rng(5)
    need = np.diff(s.blk_ptr) + 6
    s.region_nrp = np.maximum(rng.integers(8, 129, size=s.n_atoms), need).astype(np.int32)
    atoms = np.sort(rng.choice(s.n_atoms, 10, replace=False))
    cols = (atoms[:, None] * 4 + np.arange(4)).ravel().astype(np.int32)
    _check(s, 7, 6, cols, 0.4, 0.1)
