"""Which basis kernel a solve takes.  The caller workspace that a solve needs tells
them apart: the on-chip kernel has no basis workspace, the workspace kernel one
column's per workgroup, the atom kernel a whole atom's."""

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
    yield torch, ma


def _sp3(cells, region, rcut=None):
    prm = synth.SP3_PARAMS if rcut is None else dict(synth.SP3_PARAMS, rcut=rcut)
    pos = synth.diamond_positions(*cells, 5.43)
    pos = pos + np.random.default_rng(2).normal(0, 0.05, size=pos.shape)
    s = synth.build_tb(pos, np.array(cells) * 5.43, prm, name="sp3")
    s.region_mode, s.kT = "nearest", 0.1
    s.region_nrp = np.full(s.n_atoms, region, np.int32)
    return s


def _size(ma, ctx, cols, p, q, kernel):
    return ctx.workspace_size(cols, p, q, mu=0.9, opts=ma.default_opts(basis_kernel=kernel, pipeline=0))


def _solve(torch, ma, ctx, s, p, q, kernel, cols=None):
    rho = torch.zeros(s.nblk * 16, dtype=torch.float64, device="cuda")
    ctx.solve_columns(cols, p, q, mu=0.9, kT=s.kT, rho=rho, opts=ma.default_opts(basis_kernel=kernel))
    torch.cuda.synchronize()
    return rho.cpu().numpy()


# (cutoff: operator blocks per row of the largest region)
@pytest.mark.parametrize("rcut,rows,onchip", [(None, (3, 8), True), (4.2, (8, 18), False),
                                              (5.6, (18, 40), False)])
def test_dense_operators_leave_the_register_form(env, rcut, rows, onchip):
    """Up to 8 blocks per row the automatic kernel is the on-chip one, past that the
    workspace kernel; the named on-chip kernel goes back to its LDS form past 18."""
    torch, ma = env
    import oracle
    s = _sp3((4, 4, 4), 100, rcut)
    ctx = ma.Context(0)
    ctx.build_tb(s)
    na, lb = ctx.region_sizes(s.n_atoms)
    assert rows[0] < lb.max() / na.max() <= rows[1]
    cols = np.sort(np.random.default_rng(3).choice(s.n_atoms, 6, replace=False))
    cols = (4 * cols[:, None] + np.arange(4)).ravel().astype(np.int32)
    auto, on, work = (_size(ma, ctx, cols, 6, 5, k) for k in ("auto", "onchip", "workspace"))
    assert on < work and auto == (on if onchip else work)
    raw = oracle.solve_raw(s, cols=cols, p=6, q=5)
    want = oracle.scatter_slots(s, cols, oracle.outputs(s, raw, 0.9, s.kT)[0])
    for kernel in ("auto", "onchip"):
        print(f"[gpu-case] cutoff {rcut} {kernel}", flush=True)
        got = _solve(torch, ma, ctx, s, 6, 5, kernel, cols).reshape(-1, 4, 4)
        assert np.abs(got - want).max() <= 1e-10     # the parity tests' FP64 bound
    ctx.close()


@pytest.mark.parametrize("p,q", [(5, 11), (15, 17), (10, 18)])
def test_tuner_tries_what_runs_untuned(env, p, q):
    """Shapes that the on-chip kernel holds in its register form alone: the tuner tries
    the automatic choice (whatever an earlier tuning says), and a solve with the tuning
    it finds takes it, as an untuned one does.  By name the kernel stays refused."""
    torch, ma = env
    import oracle
    s = _sp3((4, 4, 4), 100)
    ctx = ma.Context(0)
    ctx.build_tb(s)
    untuned = _size(ma, ctx, None, p, q, "auto")
    assert untuned < _size(ma, ctx, None, p, q, "workspace")
    with pytest.raises(ma.MarnoldiError) as ei:
        _size(ma, ctx, None, p, q, "onchip")
    assert ei.value.status == ma.MA_EINVAL
    ctx.set_tuning(p, q, "fp64", 1, "lpt", "workspace", 0)
    print(f"[gpu-case] autotune p={p} q={q}", flush=True)
    t = ctx.autotune(None, p, q, mu=0.9, kT=s.kT, reps=2)
    assert {k for _, _, _, k in t["tried"]} >= {"auto", "workspace"}
    # (1.2 to 1.9 times the workspace kernel's speed)
    assert t["basis_kernel"] == "auto"
    assert _size(ma, ctx, None, p, q, "auto") == untuned
    got = _solve(torch, ma, ctx, s, p, q, "auto").reshape(-1, 4, 4)
    cols = np.arange(8, dtype=np.int32)
    raw = oracle.solve_raw(s, cols=cols, p=p, q=q)
    want = oracle.scatter_slots(s, cols, oracle.outputs(s, raw, 0.9, s.kT)[0])
    assert np.abs(got[:s.blk_ptr[2]] - want[:s.blk_ptr[2]]).max() <= 1e-10
    ctx.close()


def test_tuner_names_the_kernels_that_have_one(env):
    torch, ma = env
    s = _sp3((3, 3, 3), 60)
    ctx = ma.Context(0)
    ctx.build_tb(s)
    t = ctx.autotune(None, 6, 5, mu=0.9, kT=s.kT, reps=1)
    assert "onchip" in {k for _, _, _, k in t["tried"]} and "auto" not in {k for _, _, _, k in t["tried"]}
    ctx.close()


# 256 and 512 orbitals, 16 and 32 vectors, one more of each; chains that LDS does not hold
@pytest.mark.parametrize("atoms,p,q,onchip", [
    (64, 8, 8, True), (64, 9, 8, True), (65, 8, 8, True), (64, 16, 16, True), (64, 1, 31, True),
    (64, 17, 16, False), (128, 16, 16, True), (128, 8, 8, True), (128, 17, 16, False),
    (129, 8, 8, False), (128, 8, 24, True), (128, 1, 31, False)])
def test_shapes_of_the_register_form(env, atoms, p, q, onchip):
    torch, ma = env
    s = _sp3((4, 4, 4), atoms)
    ctx = ma.Context(0)
    ctx.build_tb(s)
    # (without a basis workspace: less than the workspace kernel by all of its own, of
    # which a workgroup's is 3 nu + q vectors)
    auto, work = (_size(ma, ctx, None, p, q, k) for k in ("auto", "workspace"))
    if onchip:
        assert auto <= work - 256 * (3 * (p + q) + q) * 4 * atoms * 8
    else:
        assert auto == work
    ctx.close()


@pytest.mark.parametrize("which,kernel", [("all", "atom"), ("eight", "atom"), ("seven", "atom"),
                                          ("shuffled", "atom"), ("six", "workspace"),
                                          ("255 atoms", "workspace"), ("256 atoms", "atom")])
def test_columns_that_take_the_atom_kernel(env, which, kernel):
    """FP64 spd: at least 256 atoms and on average 7 columns of each."""
    torch, ma = env
    assert torch.cuda.get_device_properties(0).multi_processor_count == 256
    s = synth.config_fcc_spd(5, cells=(4, 4, 5))
    per = {"eight": 8, "seven": 7, "six": 6}.get(which, 9)
    cols = np.array([9 * a + i for a in range(s.n_atoms) for i in range(per)], np.int32)
    if which == "shuffled":
        cols = np.random.default_rng(1).permutation(cols).astype(np.int32)
    if which.endswith("atoms"):
        cols = cols[:9 * int(which.split()[0])]
    ctx = ma.Context(0)
    ctx.build_tb(s)
    size = {k: _size(ma, ctx, cols, 4, 3, k) for k in ("auto", "atom", "workspace")}
    assert size["atom"] > size["workspace"] and size["auto"] == size[kernel]
    # not where the caller chose, nor in the mixed modes
    for kw in (dict(basis_kernel="workspace"), dict(precision="mixed_f64acc")):
        a, b = (ctx.workspace_size(cols, 4, 3, mu=0.3, opts=ma.default_opts(pipeline=0, **{**kw, **x}))
                for x in ({}, dict(basis_kernel="workspace")))
        assert a == b
    ctx.close()


def test_dense_operators_without_room_for_the_workspace_kernel(env):
    """The register form needs no basis workspace: it still runs where a caller's
    workspace does not hold the workspace kernel's."""
    torch, ma = env
    import oracle
    s = _sp3((4, 4, 4), 100, 4.2)
    ctx = ma.Context(0)
    ctx.build_tb(s)
    p, q = 6, 5
    buf = torch.empty(_size(ma, ctx, None, p, q, "onchip"), dtype=torch.uint8, device="cuda")
    assert buf.numel() < _size(ma, ctx, None, p, q, "workspace")
    ctx.set_workspace(buf)
    got = _solve(torch, ma, ctx, s, p, q, "auto").reshape(-1, 4, 4)
    ctx.set_workspace(None)
    cols = np.arange(8, dtype=np.int32)
    raw = oracle.solve_raw(s, cols=cols, p=p, q=q)
    want = oracle.scatter_slots(s, cols, oracle.outputs(s, raw, 0.9, s.kT)[0])
    assert np.abs(got[:s.blk_ptr[2]] - want[:s.blk_ptr[2]]).max() <= 1e-10
    ctx.close()
