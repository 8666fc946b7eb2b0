"""K_ACE for blocks of right-hand sides in the 2-byte precisions: the paired-tile kernel.

Factor counts on both sides of a row tile (128) and of a wave's half of it, blocks
on both sides of a column tile (64 right-hand sides) and of a wave's half, grids
whose rows end inside a tile.  Held to the FP64 form at each precision's tolerance,
and a column's bits must not depend on the size of its block.
"""
import numpy as np
import pytest

import synth
from tests.gpu_util import dev, host, rel_err, say

pytestmark = pytest.mark.gpu

TOL = {"ace_bf16r": 3e-5, "ace_fp16r": 1e-5, "ace_bf16": 2e-2, "ace_fp16": 3e-3}


@pytest.mark.parametrize("n3,N", [((3, 4, 4), 1), ((9, 8, 6), 64), ((12, 9, 16), 128), ((12, 9, 16), 129),
                                  ((18, 16, 16), 200)])
@pytest.mark.parametrize("dtype", ["complex64", "complex128"])
def test_blocks(n3, N, dtype):
    from paper_1905_01348_amd import Context

    ctx, L3 = Context(0), (6.0, 5.0, 4.0)
    ace = ctx.build_ace(dev(synth.make_orbitals(8, n3, L3, N, ecut=1e4)), n=n3, L=L3, kernel="hse", omega=0.4)
    phi = dev(synth.random_grid_vectors(9, n3, 130).astype(dtype))
    ref = host(ace.apply(phi, prec="ace_fp64"))
    for prec, tol in TOL.items():
        say("blocks", n3, N, dtype, prec)
        wide = host(ace.apply(phi, prec=prec))
        if N > 1:  # (one factor's coefficients are sums that may cancel: no bound relative to the result)
            assert rel_err(wide, ref) <= tol, prec
        for first, count in ((0, 33), (1, 64), (3, 65), (30, 97)):
            got = host(ace.apply(phi[first:first + count], prec=prec))
            assert np.array_equal(got, wide[first:first + count]), (prec, count)
    ace.free()
    ctx.close()
