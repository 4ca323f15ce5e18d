"""Calls on a card whose memory is mostly held by the caller: the automatic kernel
falls back to the one that fits, the forces to one launch without block sums, the density
of states to fewer partial sums."""

import ctypes

import numpy as np
import pytest

from paper_1202_0098_amd import synth

pytestmark = pytest.mark.gpu

MB = 1 << 20


@pytest.fixture(scope="module")
def env():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1202_0098_amd as ma
    yield torch, ma


def _hold_about(torch, leave):
    """Device memory of the caller's, so that about `leave` bytes are free (to within a
    GB: what the runtime says is free is not just what it gives)."""
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    held = []
    for _ in range(3):
        more = torch.cuda.mem_get_info()[0] - leave
        if more > 64 * MB:
            held.append(torch.empty(more, dtype=torch.uint8, device="cuda"))
    return held


class _HoldAll:
    """All that the runtime gives but `leave` bytes, a few MB, without torch's allocator
    and its larger pieces."""

    def __init__(self, torch, leave):
        self.hip = ctypes.CDLL("libamdhip64.so")
        self.hip.hipMalloc.argtypes = [ctypes.POINTER(ctypes.c_void_p), ctypes.c_size_t]
        self.hip.hipFree.argtypes = [ctypes.c_void_p]
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        room, size, self.held = self._take(leave), torch.cuda.mem_get_info()[0], []
        while size >= 2 * MB:
            ptr = self._take(size)
            if ptr:
                self.held.append(ptr)
            else:
                size = size // 2 // (2 * MB) * (2 * MB)
        self.hip.hipFree(room)

    def _take(self, size):
        ptr = ctypes.c_void_p()
        if self.hip.hipMalloc(ctypes.byref(ptr), size) == 0:
            return ptr
        self.hip.hipGetLastError()
        return None

    def release(self):
        for ptr in self.held:
            self.hip.hipFree(ptr)


def test_automatic_kernel_where_its_other_buffers_do_not_fit(env):
    """The atom kernel's workspaces fit half of the free memory, but not all of the
    solve's buffers beside them; the workspace kernel's do."""
    torch, ma = env
    s = synth.config_fcc_spd(5, cells=(8, 8, 12))
    p, q, n = 28, 20, s.nblk * 81
    opts = {k: ma.default_opts(basis_kernel=k, pipeline=0, slots_per_cu=1) for k in ("auto", "atom", "workspace")}
    rho, ref, by_atoms = (torch.zeros(n, dtype=torch.float64, device="cuda") for _ in range(3))
    ctx = ma.Context(0)
    ctx.build_tb(s)
    ctx.solve_columns(None, p, q, kT=s.kT, rho=by_atoms, opts=opts["atom"])
    want = ctx.solve_columns(None, p, q, kT=s.kT, rho=ref, opts=opts["workspace"])
    ctx.close()
    ctx = ma.Context(0)
    ctx.build_tb(s)
    auto, atom, work = (ctx.workspace_size(None, p, q, opts=opts[k]) for k in ("auto", "atom", "workspace"))
    leave = (atom + work) // 2
    assert auto == atom and atom - work >= 2000 * MB
    held = _hold_about(torch, leave)
    try:
        print(f"[gpu-case] {leave / MB:.0f} MB free, atom {atom / MB:.0f}, workspace {work / MB:.0f}",
              flush=True)
        rho.zero_()
        got = ctx.solve_columns(None, p, q, kT=s.kT, rho=rho, opts=opts["auto"])
    finally:
        del held
        torch.cuda.empty_cache()
    assert torch.equal(rho, ref) and got.mu == want.mu and got.energy == want.energy
    # with the memory back, the atom kernel again
    ctx.solve_columns(None, p, q, kT=s.kT, rho=rho, opts=opts["auto"])
    assert torch.equal(rho, by_atoms) and not torch.equal(rho, ref)
    ctx.close()


@pytest.mark.parametrize("kind", ["sp3", "spd"])
def test_forces_without_memory_for_the_block_sums(env, kind):
    """One launch instead of two; both carry the rounding of their sums, so that they
    agree to the rounding of the result (2^-53 of the largest, twice)."""
    torch, ma = env
    if kind == "sp3":
        s = synth.build_tb(synth.diamond_positions(22, 22, 22, 5.43), np.full(3, 5.43 * 22), synth.SP3_PARAMS)
        s.region_mode, s.region_nrp = "nearest", np.full(s.n_atoms, 5, np.int32)
    else:
        s = synth.config_fcc_spd(5, cells=(12, 12, 12))
    g = torch.Generator(device="cuda").manual_seed(1)
    rho, pi = (torch.randn(s.nblk * s.n_orb ** 2, dtype=torch.float64, device="cuda", generator=g)
               for _ in range(2))
    dH, dS = (torch.randn(3 * s.nblk * s.n_orb ** 2, dtype=torch.float64, device="cuda", generator=g)
              for _ in range(2))
    F, ref = (torch.zeros(3 * s.n_atoms, dtype=torch.float64, device="cuda") for _ in range(2))
    for out in (ref, F):
        ctx = ma.Context(0)
        ctx.build_tb(s)
        held = None
        if out is F:   # the sums take 48 bytes per block
            held = _HoldAll(torch, 4 * MB)
            assert 48 * s.nblk > 8 * MB
        print(f"[gpu-case] forces, {s.nblk} blocks, {torch.cuda.mem_get_info()[0] / MB:.0f} MB free", flush=True)
        try:
            ctx.forces(dH, dS, rho, pi, out)
        finally:
            if held:
                held.release()
        ctx.close()
    assert float((F - ref).abs().max()) <= 2 ** -52 * float(ref.abs().max())


def test_dos_without_memory_for_its_partial_sums(env):
    """8,192 energies and 245,760 Ritz pairs in 240 chunks take 15.7 MB of partial sums, in
    30 chunks 2.  The two groupings agree to the rounding of sums of 245,760
    positive terms (their weights are: an orthonormal basis), each of which is at
    most 8,192 long before it is added: 8192 x 2^-53 = 1e-12."""
    torch, ma = env
    s = synth.config_diamond4096()
    ctx = ma.Context(0)
    ctx.build_tb(s)
    ctx.solve_columns(None, 10, 5, mu=0.9, kT=s.kT)
    E = np.linspace(-16.0, 14.0, 8192)
    ref = ma.Context(0)
    ref.build_tb(s)
    ref.solve_columns(None, 10, 5, mu=0.9, kT=s.kT)
    want = ref.dos(E, 0.1)
    ref.close()
    held = _HoldAll(torch, 10 * MB)
    try:
        print(f"[gpu-case] dos, {torch.cuda.mem_get_info()[0] / MB:.0f} MB free", flush=True)
        got = ctx.dos(E, 0.1)
    finally:
        held.release()
    assert np.abs(got - want).max() <= 1e-12 * want.max()
    ctx.close()


def test_chunk_buffer_of_the_default(env):
    """43,200 columns of 64 vectors fill 11 GB of chunk buffer; by default a solve keeps
    at most 8 GiB of it, whatever is free, and gives the same as one long chunk."""
    torch, ma = env
    s = synth.config_fcc_spd(5, cells=(10, 10, 12))
    p = q = 32
    rho, ref = (torch.zeros(s.nblk * 81, dtype=torch.float64, device="cuda") for _ in range(2))
    ctx = ma.Context(0)
    ctx.build_tb(s)
    # (basis workspaces, lists and a chunk buffer of 4 GiB)
    size = ctx.workspace_size(None, p, q, mu=0.3, opts=ma.default_opts())
    assert size == ctx.workspace_size(None, p, q, mu=0.3, opts=ma.default_opts(basis_kernel="atom", pipeline=0))
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    print(f"[gpu-case] {s.M} columns, p = q = 32", flush=True)
    a = ctx.solve_columns(None, p, q, mu=0.3, kT=s.kT, rho=rho)
    grown = before - torch.cuda.mem_get_info()[0]
    b = ctx.solve_columns(None, p, q, mu=0.3, kT=s.kT, rho=ref, opts=ma.default_opts(pipeline=0))
    print(f"[gpu-case] {grown / MB:.0f} MB, in a workspace {size / MB:.0f}", flush=True)
    # (1 GiB for what the runtime keeps for itself)
    assert grown <= size + 5 * 1024 * MB
    assert torch.equal(rho, ref) and a.energy == b.energy
    ctx.close()
