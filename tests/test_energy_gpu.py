"""E_X of a phi == psi application, against the FP64 sum over the returned columns.

Grids of one span per column, ragged spans and the largest count of spans, every
input and output type, and the form without allocations.  Both sides add the same
FP64 products, so they agree to 1e-13 of the sum of the magnitudes (nr * N < 4e6
terms added pairwise or in short chains of a few hundred).
"""
import numpy as np
import pytest
import torch

import synth
from tests.gpu_util import dev, host, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n3,N", [((4, 4, 4), 1), ((8, 9, 6), 300), ((24, 24, 24), 5), ((27, 16, 18), 3),
                                  ((72, 54, 48), 2)])
def test_energy_is_half_the_trace(n3, N):
    from paper_1905_01348_amd import Context

    ctx, L3 = Context(0), (5.0, 4.0, 6.0)
    P = dev(synth.random_grid_vectors(73, n3, N))
    for prec in ("fp64", "fp32acc64", "fp32"):
        for tin in (torch.complex128, torch.complex64):
            for tout in (torch.complex128, torch.complex64):
                say("energy", n3, N, prec, tin, tout)
                psi = P.to(tin)
                kw = dict(n=n3, L=L3, kernel="coulomb", prec=prec)
                out, ex = ctx.apply_vx(psi, out_dtype=tout, energy=True, **kw)
                prods = (host(psi).astype(np.complex128).conj() * host(out).astype(np.complex128)).real
                bound = 1e-13 * np.abs(prods).sum()
                assert abs(float(ex) - 0.5 * prods.sum()) <= bound
                if (tin == torch.complex128) != (prec == "fp64"):
                    continue  # the form without allocations converts no inputs
                o2, e2 = torch.empty_like(out), torch.empty((), dtype=torch.float64, device="cuda")
                ctx.apply_vx_noalloc(psi, out=o2, energy_out=e2, **kw)
                prods = (host(psi).astype(np.complex128).conj() * host(o2).astype(np.complex128)).real
                assert abs(float(e2) - 0.5 * prods.sum()) <= bound
    ctx.close()
