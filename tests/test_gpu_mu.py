"""The chemical-potential search against the same K-section (14 passes of 15 trial
potentials, the first that reaches the target) done directly in numpy on the
returned Ritz values and weights: from kT so small that the bracket never falls
below kT / 8 (no series) to kT above the spectrum's width, and from an almost
empty to an almost full count.

N(mu) is summed to about 1e-15 of the total weight on both sides, so that mu
agrees to that over dN/dmu; asserted to 1e-12 of the weight over the local slope,
and never looser than 1e-6 kT."""

import math

import numpy as np
import pytest

from paper_1202_0098_amd import synth

pytestmark = pytest.mark.gpu


def _count(mu, e, w, kT):
    x = (e[None, :] - np.atleast_1d(mu)[:, None]) / kT
    t = np.exp(-np.abs(x))
    return (np.where(x <= 0, 1.0, t) / (1.0 + t)) @ w


@pytest.mark.parametrize("kT", [1e-9, 1e-4, 0.1, 0.7, 40.0])
@pytest.mark.parametrize("fill", [0.02, 0.5, 0.97])
def test_mu(kT, fill):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1202_0098_amd as ma
    s = synth.config_diamond64()
    nu, target = s.p + s.q, fill * s.M
    print(f"[gpu-case] diamond64 kT={kT} fill={fill}", flush=True)
    ctx = ma.Context(0)
    ctx.build_tb(s)
    eps = torch.zeros(s.M * nu, dtype=torch.float64, device="cuda")
    wts = torch.zeros_like(eps)
    r = ctx.solve_columns(None, s.p, s.q, kT=kT, eps=eps, wts=wts, opts=ma.default_opts(n_target=target))
    e, w = eps.cpu().numpy(), wts.cpu().numpy()
    lo, hi = e.min() - 50 * kT, e.max() + 50 * kT
    for _ in range(14):
        mus = lo + (hi - lo) * np.arange(1, 16) / 16
        reach = np.nonzero(_count(mus, e, w, kT) >= target)[0]
        first = reach[0] if len(reach) else 15
        lo, hi = (mus[first - 1] if first > 0 else lo), (mus[first] if first < 15 else hi)
    mu = 0.5 * (lo + hi)
    d = 1e-3 * kT
    slope = float(np.diff(_count([mu - d, mu + d], e, w, kT))[0] / (2 * d))
    assert abs(r.mu - mu) <= max(4e-16 * abs(mu), min(1e-12 * s.M / max(slope, 1e-300), 1e-6 * kT))
    # the same search again on the kept data, at another temperature and back
    ctx.find_mu(target, 2 * kT)
    assert ctx.find_mu(target, kT).mu == r.mu
    ctx.close()


@pytest.mark.parametrize("kT", [1e-7, 1e-5, 0.1])
def test_density_at_the_found_mu(kT):
    """The density and the sums belong to the mu that is returned, also where the
    search needs more passes than are launched at once (small kT)."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1202_0098_amd as ma
    s = synth.config_diamond64()
    o = s.n_orb
    ctx = ma.Context(0)
    ctx.build_tb(s)
    rho, again, ref = (torch.zeros(s.nblk * o * o, dtype=torch.float64, device="cuda") for _ in range(3))
    # a filling at which no level is partly occupied: mu lies in a gap
    r = ctx.solve_columns(None, s.p, s.q, kT=kT, rho=rho)
    f = ctx.find_mu(0.5 * s.M, kT, rho=again)
    g = ctx.solve_columns(None, s.p, s.q, mu=r.mu, kT=kT, rho=ref)
    torch.cuda.synchronize()
    # an occupation moves by at most dmu / 4 kT; mu is exact to a few ulp of 1 eV
    tol = 1e-10 + 1e-15 / kT
    print(f"[gpu-case] kT={kT}: d rho {float((rho - ref).abs().max()):.1e} dN {abs(r.n_elec - g.n_elec):.1e}", flush=True)
    assert float((rho - ref).abs().max()) <= tol
    assert abs(r.n_elec - g.n_elec) <= tol * s.M and abs(r.energy - g.energy) <= tol * s.M * 10
    assert f.mu == r.mu and float((again - ref).abs().max()) <= tol
    ctx.close()


@pytest.mark.parametrize("kind", ["sp3", "spd"])
@pytest.mark.parametrize("precision,p,q", [("fp64", 1, 0), ("fp64", 2, 1), ("fp64", 15, 15),
                                           ("fp64", 32, 32), ("mixed_f64acc", 9, 8)])
def test_stored_amplitudes_give_the_density_of_a_given_mu(kind, precision, p, q):
    """rho and pi of a bisected solve (amplitudes stored, then weighted) against
    the same columns at that mu (weighted before they are stored): 20 and up to
    390 rows, stages of 128, 64 and fewer rows."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1202_0098_amd as ma
    s = synth.config_diamond64() if kind == "sp3" else synth.config_fcc_spd(5, cells=(4, 4, 4))
    cols = np.arange(0, s.M, 1 if kind == "sp3" else 7, dtype=np.int32)
    o = s.n_orb
    print(f"[gpu-case] {kind} {precision} p={p} q={q}", flush=True)
    ctx = ma.Context(0)
    ctx.build_tb(s)
    out = [torch.zeros(s.nblk * o * o, dtype=torch.float64, device="cuda") for _ in range(4)]
    opts = ma.default_opts(precision=precision)
    r = ctx.solve_columns(cols, p, q, kT=s.kT, rho=out[0], pi=out[1], opts=opts)
    g = ctx.solve_columns(cols, p, q, mu=r.mu, kT=s.kT, rho=out[2], pi=out[3], opts=opts)
    torch.cuda.synchronize()
    # FP64: rounding of sums of at most 64 terms of order one (eps up to 30 for
    # pi); FP32 amplitudes: an ulp of each, 64 * 6e-8
    tol = 1e-10 if precision == "fp64" else 4e-6
    assert float((out[0] - out[2]).abs().max()) <= tol
    assert float((out[1] - out[3]).abs().max()) <= 30 * tol
    assert abs(r.energy - g.energy) <= 30 * tol * len(cols)
    assert abs(r.n_elec - g.n_elec) <= tol * len(cols)
    ctx.close()
