"""The density of states where a workgroup takes several stages of Ritz pairs (many
energies), with a short last stage and with a workgroup that divides because one of
its energies is not finite; against the same energies in a short list, for which
every workgroup takes one stage.  The sums of 4,000 terms are grouped otherwise:
4,000 x 2^-53 = 4.4e-13 of the largest."""

import numpy as np
import pytest

from paper_1202_0098_amd import synth

pytestmark = pytest.mark.gpu


def test_several_stages_per_workgroup():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1202_0098_amd as ma
    s = synth.config_diamond64()
    ctx = ma.Context(0)
    ctx.build_tb(s)
    # 250 columns of 16 vectors: 4,000 pairs, four stages of which the last has 928
    ctx.solve_columns(np.arange(250, dtype=np.int32), 8, 8, mu=0.9, kT=s.kT)
    # 4 stages x 2,149 tiles of 512 energies = 8,596: four stages per workgroup
    E = np.linspace(-30.0, 25.0, 1100000)
    E[1234] = np.inf
    print("[gpu-case] dos of 1,100,000 energies", flush=True)
    got = ctx.dos(E, 0.1)
    at = np.unique(np.concatenate([np.arange(1000, 1600), np.arange(len(E) - 300, len(E)),
                                   np.arange(0, len(E), 99991)]))
    want = ctx.dos(E[at], 0.1)
    assert got[1234] == 0.0
    assert np.abs(got[at] - want).max() <= 4.4e-13 * want.max()
    ctx.close()
