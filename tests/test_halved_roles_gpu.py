"""phi == psi on the cubes' kernels: both roles of the plane-inverse pass, one launch.

Block sizes that leave a ragged last block and orbitals fewer than a sum group's
share, for every form of the pass (the staged ones run a role per launch).  Held to
the FP64 oracle at the precision's tolerance (1e-10 FP64, 1e-5 FP32); with one sum
group the result is independent of the block size, bitwise, since each target's
terms are added in ascending order whatever launch they arrive in.
"""
import numpy as np
import pytest

import oracle
import synth
from tests.gpu_util import rel_err, dev, host, say

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-10, "fp32acc64": 1e-5, "fp32": 1e-5}


@pytest.mark.parametrize("n,N", [(24, 1), (24, 5), (48, 5), (72, 3), (96, 3)])
def test_roles(n, N, monkeypatch):
    from paper_1905_01348_amd import Context

    n3, L3 = (n,) * 3, (5.0, 4.0, 6.0)
    psi = synth.random_grid_vectors(72, n3, N)
    ref = oracle.apply_vx(psi, psi, n3, L3, "hse", 0.3)
    ctx, P = Context(0), dev(psi)
    monkeypatch.setenv("FX_VX_HALVE", "1")
    for prec in TOL:
        for var in ("1", "2", "3", "4", "5"):
            monkeypatch.setenv("FX_VX_C_VAR", var)
            got = {}
            for split in ("1", "4"):
                monkeypatch.setenv("FX_VX_C_SPLIT", split)
                for nj in ("1", "2", "8"):
                    say("roles", n, prec, var, split, nj)
                    monkeypatch.setenv("FX_VX_NJ", nj)
                    out = host(ctx.apply_vx(P, n=n3, L=L3, kernel="hse", omega=0.3, prec=prec))
                    assert rel_err(out, ref) <= TOL[prec], (prec, var, split, nj)
                    assert np.array_equal(got.setdefault(split, out), out), (prec, var, split, nj)
    ctx.close()
