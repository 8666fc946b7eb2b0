"""Pair passes on grids off the workload edges, against the FP64 oracle.

The phi == psi form, halved (each unordered pair solved once: the FP64 and FP32
forms of large grids) or not, is independent of the batch (bitwise); the two
agree to rounding and both with the oracle to the precision's tolerance (1e-10
FP64, 1e-5 FP32).  Sum
groups, and first x radices that leave more butterflies than one per thread of
the plane-inverse pass, are held to the same tolerances.
"""
import numpy as np
import pytest

import oracle
import synth
from tests.gpu_util import rel_err, dev, host, say

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-10, "fp32acc64": 1e-5, "fp32": 1e-5}
CLOSE = {"fp64": 1e-12, "fp32acc64": 2e-6, "fp32": 5e-6}


@pytest.fixture(scope="module")
def ctx():
    from paper_1905_01348_amd import Context

    c = Context(0)
    yield c
    c.close()


# one-, two- and mixed-stage axes, odd edges (no row padding), tiles that are whole rows and that are not
@pytest.mark.parametrize("n3", [(2, 3, 4), (9, 8, 48), (27, 16, 18), (81, 4, 96), (96, 3, 72), (64, 54, 3)])
def test_square_form_and_groups(ctx, n3, monkeypatch):
    L3, N, Nt = (5.0, 4.0, 6.0), 7, 3
    psi, phi = synth.random_grid_vectors(70, n3, N), synth.random_grid_vectors(71, n3, Nt)
    P, Q = dev(psi), dev(phi)
    sq, rect = oracle.apply_vx(psi, psi, n3, L3, "hse", 0.3), oracle.apply_vx(psi, phi, n3, L3, "hse", 0.3)
    kw = dict(n=n3, L=L3, kernel="hse", omega=0.3)
    for prec in TOL:
        say("square", n3, prec)
        forms = []
        for halve in ("0", "1"):
            monkeypatch.setenv("FX_VX_HALVE", halve)
            got = host(ctx.apply_vx(P, prec=prec, **kw))
            assert rel_err(got, sq) <= TOL[prec], halve
            for nj in ("1", "2", "3"):
                monkeypatch.setenv("FX_VX_NJ", nj)
                assert np.array_equal(host(ctx.apply_vx(P, prec=prec, **kw)), got), (halve, nj)
            monkeypatch.delenv("FX_VX_NJ")
            forms.append(got)
        monkeypatch.delenv("FX_VX_HALVE")
        assert rel_err(forms[1], forms[0]) <= CLOSE[prec]
        for s in (1, 2, 8):
            monkeypatch.setenv("FX_VX_C_SPLIT", str(s))
            r = host(ctx.apply_vx(P, Q, prec=prec, **kw))
            assert rel_err(r, rect) <= TOL[prec], s
            # a target's bits do not depend on its neighbours in the launch or on the batch
            monkeypatch.setenv("FX_VX_NJ", "2")
            assert np.array_equal(host(ctx.apply_vx(P, Q[1:2], prec=prec, **kw))[0], r[1]), s
            monkeypatch.delenv("FX_VX_NJ")
        monkeypatch.delenv("FX_VX_C_SPLIT")


@pytest.mark.parametrize("n3,radix", [((96, 72, 2), [2, 6, 8]), ((96, 72, 2), [3, 4, 8]), ((96, 72, 2), [4, 3, 8]),
                                      ((96, 72, 2), [6, 2, 8]), ((96, 72, 2), [8, 12]), ((81, 96, 2), [9, 9])],
                         ids=lambda v: str(v).replace(" ", ""))
def test_several_butterflies_per_thread(ctx, n3, radix):
    L3, N = (20.0, 15.0, 1.0), 3
    psi = synth.random_grid_vectors(72, n3, N)
    ref = oracle.apply_vx(psi, psi, n3, L3, "coulomb")
    for prec in TOL:
        say("radix", n3, radix, prec)
        ctx.set_vx_config({"kernels": 2, "radix": [radix]}, n=n3, prec=prec, phi_is_psi=True)
        got = host(ctx.apply_vx(dev(psi), n=n3, L=L3, kernel="coulomb", prec=prec))
        ctx.set_vx_config(None, n=n3, prec=prec, phi_is_psi=True)
        assert rel_err(got, ref) <= TOL[prec]


# x axes of one stage, a thread per plane value: one, two and three values per thread (FP64), the largest plane of
# both precisions, and planes just past it
@pytest.mark.parametrize("n3", [(12, 36, 3), (12, 48, 2), (12, 96, 2), (9, 12, 4), (12, 9, 8), (12, 12, 3), (8, 16, 3)])
def test_one_stage_x_axes(ctx, n3, monkeypatch):
    test_square_form_and_groups(ctx, n3, monkeypatch)


@pytest.mark.parametrize("prec", ["fp64", "fp32acc64"])
def test_z_tiles_too_large_are_refused(ctx, prec):
    """A z-pass tile of more than 18 points per thread (a whole row of 96 pencils of 96 points need not fit the
    LDS) is FX_ERR_UNSUPPORTED before anything is launched, and the tuner passes over it."""
    from paper_1905_01348_amd import FockError

    n3, L3, N = (96, 2, 96), (30.0, 1.0, 30.0), 3
    psi = synth.random_grid_vectors(74, n3, N)
    ref = oracle.apply_vx(psi, psi, n3, L3, "hse", 0.3)
    cdt = np.complex128 if prec == "fp64" else np.complex64
    P, kw = dev(psi.astype(cdt)), dict(n=n3, L=L3, kernel="hse", omega=0.3, prec=prec)
    for cfg in ({"kernels": 2, "b_xtile": 96}, {"kernels": 2, "b_xtile": 49}, {"kernels": 2, "b_threads": 128}):
        say("refused", prec, cfg)
        ctx.set_vx_config(cfg, n=n3, prec=prec, phi_is_psi=True)
        with pytest.raises(FockError) as ei:
            ctx.apply_vx(P, **kw)
        assert ei.value.status == -2, cfg
    ctx.set_vx_config({"kernels": 2, "b_xtile": 48}, n=n3, prec=prec, phi_is_psi=True)
    assert rel_err(host(ctx.apply_vx(P, **kw)), ref) <= TOL[prec]
    say("tune", prec)
    cfg, _ = ctx.vx_autotune(n=n3, L=L3, n_psi=N, n_phi=N, phi_is_psi=True, prec=prec)
    assert cfg["b_xtile"] <= 48
    assert rel_err(host(ctx.apply_vx(P, **kw)), ref) <= TOL[prec]
    ctx.set_vx_config(None, n=n3, prec=prec, phi_is_psi=True)


@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp32acc64"])
def test_automatic_halving(ctx, prec, monkeypatch):
    """phi == psi off the specialised grids: FP64 and FP32 solve each unordered pair once from 512 planes of targets
    on (8 to 12 waves per plane here), FP32 with FP64 sums never; bitwise what asking for it gives."""
    n3, L3 = (96, 64, 36), (41.0, 27.0, 15.0)
    for N, halved in ((14, False), (15, prec != "fp32acc64")):
        psi = dev(synth.random_grid_vectors(75, n3, N).astype(np.complex128 if prec == "fp64" else np.complex64))
        call = lambda: host(ctx.apply_vx(psi, n=n3, L=L3, kernel="hse", omega=0.3, prec=prec))
        auto = call()
        for h in (False, True):
            monkeypatch.setenv("FX_VX_HALVE", str(int(h)))
            assert np.array_equal(call(), auto) == (h == halved), (N, h)
            monkeypatch.delenv("FX_VX_HALVE")
