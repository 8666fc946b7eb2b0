"""The automatic sum groups of V_X (phi != psi): order and bits that depend on the grid and n_psi only.

For each grid the number of groups the rule takes is pinned by asking for it
explicitly (bitwise equal), the result is held to the oracle (1e-10 FP64, 1e-5
the FP32 forms), and its bits stay the same for one target and for many, for
budgets that shrink the blocks or run the groups one after the other, through
the replay cache and under capture in such a budget.
"""
import numpy as np
import pytest
import torch

import oracle
import synth
from paper_1905_01348_amd import Context
from tests.gpu_util import dev, host, rel_err, say

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-10, "fp32acc64": 1e-5, "fp32": 1e-5}


def _bits(t):
    return host(torch.view_as_real(t))


# (grid, orbitals, targets, groups): as many as fill the chip, few orbitals, the most groups, two where eight
# targets are a little more than the resident workgroups, and a block large enough for the groups in rounds
@pytest.mark.parametrize("n3,N,R,groups", [((32, 36, 24), 27, 11, 4), ((24, 24, 24), 16, 9, 4), ((24, 24, 24), 7, 3, 1),
                                           ((9, 8, 27), 33, 70, 8), ((96, 64, 36), 32, 2, 2), ((24, 24, 24), 18, 40, 4)])
@pytest.mark.parametrize("prec", ["fp64", "fp32acc64", "fp32"])
def test_automatic_groups(n3, N, R, groups, prec, monkeypatch):
    L3 = tuple(0.43 * n for n in n3)
    psi, phi = synth.random_grid_vectors(80, n3, N), synth.random_grid_vectors(81, n3, R)
    cdt = np.complex128 if prec == "fp64" else np.complex64
    P, Q = dev(psi.astype(cdt)), dev(phi.astype(cdt))
    kw = dict(n=n3, L=L3, kernel="hse", omega=0.3, prec=prec)
    nr = n3[0] * n3[1] * n3[2]
    pair, asum = nr * (16 if prec == "fp64" else 8), nr * (8 if prec == "fp32" else 16)
    ctx = Context(0)
    got = ctx.apply_vx(P, Q, **kw)
    few = [0, R - 1]
    assert rel_err(host(got)[few], oracle.apply_vx(psi, phi[few], n3, L3, "hse", 0.3)) <= TOL[prec]
    for s in (1, 2, 4, 8):
        if 2 * s > N:  # groups of one term add up like one running sum where the product is rounded first
            continue
        monkeypatch.setenv("FX_VX_C_SPLIT", str(s))
        same = np.array_equal(_bits(ctx.apply_vx(P, Q, **kw)), _bits(got))
        assert same == (s == groups), s
    monkeypatch.delenv("FX_VX_C_SPLIT")
    for k in few:
        assert np.array_equal(_bits(ctx.apply_vx(P, Q[k:k + 1], **kw))[0], _bits(got)[k]), k
    # the other output type holds the same sums, rounded or widened
    other = torch.complex64 if prec != "fp32" else torch.complex128
    assert torch.equal(ctx.apply_vx(P, Q, out_dtype=other, **kw), got.to(other))
    ctx.close()
    # budgets: blocks of one or two targets; less than the groups' sums (with room for tables)
    tables = 8 * (n3[0] // 2 + 1) * (n3[1] // 2 + 1) * (n3[2] // 2 + 1) + (64 << 10)
    for what, budget in (("small blocks", 4 * 2 * (groups * asum + 3 * pair) + tables),
                         ("groups in turn", pair + 2 * asum + tables)):
        say("groups", n3, prec, what, budget)
        small = Context(0, hbm_budget_bytes=budget)
        assert np.array_equal(_bits(small.apply_vx(P, Q, **kw)), _bits(got)), what
        if groups > 1:  # (one running sum needs its own n_phi columns where out is of another type)
            assert torch.equal(small.apply_vx(P, Q, out_dtype=other, **kw), got.to(other)), what
        # captured in this budget (after the eager calls above), and through the replay cache
        out, s, g = torch.empty_like(got), torch.cuda.Stream(), torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            small.apply_vx(P, Q, out=out, **kw)
        for _ in range(3):
            out.zero_()
            g.replay()
            torch.cuda.synchronize()
            assert np.array_equal(_bits(out), _bits(got)), what
            small.apply_vx(P, Q, **kw)  # the same shape: the workspace stays
            torch.cuda.synchronize()
        del g
        small.graph_cache(2)
        for _ in range(2):
            out.zero_()
            small.apply_vx(P, Q, out=out, **kw)
            assert np.array_equal(_bits(out), _bits(got)), what
        assert small.graph_cache_stats()[:2] == (1, 1), what
        small.close()


@pytest.mark.parametrize("c_variant", [1, 2, 3, 5])
@pytest.mark.parametrize("prec", ["fp64", "fp32acc64", "fp32"])
def test_groups_in_rounds_by_variant(c_variant, prec):
    """24^3: the groups of a block of 40 targets one after the other in registers (the staged form 3: in memory)
    and those of a few targets in memory give a target the same bits, for a count of orbitals that the groups
    do not divide."""
    n3, L3, N, R = (24, 24, 24), (10.26,) * 3, 11, 40
    cdt = np.complex128 if prec == "fp64" else np.complex64
    P, Q = dev(synth.random_grid_vectors(82, n3, N).astype(cdt)), dev(synth.random_grid_vectors(83, n3, R).astype(cdt))
    ctx, kw = Context(0), dict(n=n3, L=L3, kernel="coulomb", prec=prec)
    for s in (2, 4, 8):
        ctx.set_vx_config({"kernels": 1, "c_variant": c_variant, "c_split": s}, n=n3, prec=prec)
        say("rounds", prec, c_variant, s)
        block, some = ctx.apply_vx(P, Q, **kw), ctx.apply_vx(P, Q[7:12], **kw)
        assert np.array_equal(_bits(block)[7:12], _bits(some)), s
    ref = oracle.apply_vx(host(P), host(Q[7:9]), n3, L3, "coulomb")
    assert rel_err(host(block[7:9]), ref) <= TOL[prec]
    ctx.close()
