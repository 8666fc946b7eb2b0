"""K_ACE for few right-hand sides: the wave-per-32-rows kernel against the tiled one.

A right-hand side's bits must not depend on how many share the call, so blocks
of 1, 16, 17 and 32 columns (one and two column tiles of the narrow kernel,
full and ragged) are held bitwise to the same columns of a block of 33, which
takes the tiled kernel; that block is held to the FP64 form at each
precision's tolerance.  Row counts that are not multiples of 32, fewer steps
than the narrow kernel reads ahead, and padded columns.
"""
import numpy as np
import pytest

import synth
from tests.gpu_util import dev, host, rel_err, say

pytestmark = pytest.mark.gpu

TOL = {"ace_fp32r": 1e-5, "ace_bf16r": 3e-5, "ace_fp16r": 1e-5, "ace_fp32": 1e-5, "ace_bf16": 2e-2, "ace_fp16": 3e-3}


@pytest.fixture(scope="module")
def ctx():
    from paper_1905_01348_amd import Context

    c = Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("n3,N", [((3, 4, 2), 2), ((9, 8, 6), 33), ((24, 18, 16), 70)])
@pytest.mark.parametrize("dtype", ["complex64", "complex128"])
def test_few_columns_match_the_tiled_kernel(ctx, n3, N, dtype):
    import torch

    L3 = (6.0, 5.0, 4.0)
    ace = ctx.build_ace(dev(synth.make_orbitals(6, n3, L3, N, ecut=1e4)), n=n3, L=L3, kernel="hse", omega=0.4)
    phi = dev(synth.random_grid_vectors(7, n3, 33).astype(dtype))
    ref = host(ace.apply(phi, prec="ace_fp64"))
    for prec, tol in TOL.items():
        say("few columns", n3, N, dtype, prec)
        wide = host(ace.apply(phi, prec=prec))
        assert rel_err(wide, ref) <= tol
        for first, count in ((0, 1), (5, 16), (16, 17), (1, 32)):
            got = host(ace.apply(phi[first:first + count], prec=prec))
            assert np.array_equal(got, wide[first:first + count]), (prec, count)
    torch.cuda.synchronize()
    ace.free()
