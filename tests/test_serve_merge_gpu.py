"""A served request for all orbitals gives the same bits alone (phi == psi) and merged, off the specialised grids."""
import numpy as np
import pytest
import torch

import oracle
import synth
from paper_1905_01348_amd import Context, Server
from tests.gpu_util import dev, host, rel_err, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,tol", [("fp64", 1e-10), ("fp32", 1e-5), ("fp32acc64", 1e-5)])
def test_all_orbitals_alone_and_merged(prec, tol):
    n3, L3, N = (96, 64, 36), (41.0, 27.0, 15.0), 16  # enough planes for the halved form of a plain call
    dt, npd = (torch.complex128, np.complex128) if prec == "fp64" else (torch.complex64, np.complex64)
    psi = synth.random_grid_vectors(90, n3, N).astype(npd)
    ctx = Context(0)
    srv = Server(ctx, max_slots=1, n_streams=1, max_batch_pairs=1 << 16)
    P = dev(psi)
    srv.register(0, P, n=n3, L=L3, kernel="hse", omega=0.106, vx_prec=prec, ace_prec="ace_fp64")

    def req(first, count):
        return dict(traj=0, op=0, first=first, count=count, t=0.0,
                    out=torch.zeros((count,) + n3[::-1], dtype=dt, device="cuda"))

    alone = req(0, N)
    st, _, rep = srv.serve([alone])
    assert st == [0] and rep["n_batches"] == 1
    merged = [req(0, N), req(3, 2)]
    st, _, rep = srv.serve(merged)
    torch.cuda.synchronize()
    say("merged", prec, rep["n_batches"])
    assert st == [0, 0] and rep["n_batches"] == 1
    assert np.array_equal(host(torch.view_as_real(merged[0]["out"])), host(torch.view_as_real(alone["out"])))
    assert np.array_equal(host(merged[1]["out"]), host(alone["out"])[3:5])
    p = psi[[0, N - 1]].astype(np.complex128)
    ref = oracle.apply_vx(psi.astype(np.complex128), p, n3, L3, "hse", 0.106)
    assert rel_err(host(alone["out"])[[0, N - 1]], ref) <= tol
    srv.close()
    ctx.close()
