"""FP64 products of the ACE apply at the edges of the GEMM's tiles.

y = -xi (xi^H phi) in FP64 against numpy on the exported factors, for orbital
and right-hand-side counts around the 16-wide matrix tiles, the 32- and
64-wide workgroup tiles and the block of right-hand sides that shares one set
of split partial sums.  Both products sum at most N_r + N terms of rounding
2^-53 each: 1e-12 leaves two orders of magnitude.
"""
import numpy as np
import pytest

import synth
from tests.gpu_util import dev, host, rel_err, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1905_01348_amd import Context

    c = Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("N,R", [(1, 1), (15, 17), (16, 64), (33, 300), (65, 129), (129, 7), (140, 31)])
def test_fp64_apply_at_tile_edges(ctx, N, R):
    import torch

    n3, L3 = (16, 12, 18), (7.0, 5.5, 8.0)
    say("fp64 apply", N, R)
    ace = ctx.build_ace(dev(synth.make_orbitals(3, n3, L3, N, ecut=1e4)), n=n3, L=L3, kernel="hse", omega=0.4)
    xi = host(ace.export()[0])
    phi = synth.random_grid_vectors(4, n3, R)
    got = host(ace.apply(dev(phi)))
    c = phi.reshape(R, -1) @ xi.conj().T
    assert rel_err(got, -(c @ xi)) <= 1e-12
    # a right-hand side's bits do not depend on how many share the call
    one = host(ace.apply(dev(phi[R - 1:])))
    assert np.array_equal(one[0], got[R - 1])
    torch.cuda.synchronize()
    ace.free()


@pytest.mark.parametrize("N", [1, 63, 64, 65, 129, 192, 300])
def test_cholesky_qr_at_block_edges(ctx, N):
    """Blocks of 64 columns, joined in pairs by level: below, at and above one block, a level whose last
    pair is short, three levels.  Against numpy's Cholesky factor; the overlap of random vectors has a
    condition number below 100, so N eps cond stays under 1e-11."""
    import torch

    n3 = (16, 12, 18)
    psi = synth.random_grid_vectors(5, n3, N)
    say("cholesky-qr", N)
    p = psi.reshape(N, -1)
    low = np.linalg.cholesky(p.conj() @ p.T)
    ref = np.linalg.solve(low.conj(), p)
    got = host(ctx.orthonormalize(dev(psi))).reshape(N, -1)
    torch.cuda.synchronize()
    assert rel_err(got, ref) <= 1e-11
    # a zero column (pivot exactly 0) is found, and the block is left as it was
    psi[N - 1] = 0.0
    q = dev(psi)
    with pytest.raises(Exception, match=f"pivot {N} of {N}"):
        ctx.orthonormalize(q)
    assert np.array_equal(host(q), psi)
