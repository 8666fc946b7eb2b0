"""Sum groups in tuned and stored launch configurations.

The tuner names the number of groups it measured (one running sum among the
candidates), on the specialised and the run-time-plan kernels.  In a file, a
configuration saved when automatic meant one running sum (0, or a line older than
the field) still means that; automatic is written as -1.
"""
import numpy as np
import pytest

import synth
from paper_1905_01348_amd import Context
from tests.gpu_util import dev, host, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n3,N,R,prec", [((24, 24, 24), 16, 200, "fp64"), ((18, 16, 12), 24, 4, "fp32acc64")])
def test_tuner_names_the_groups(n3, N, R, prec):
    ctx = Context(0)
    cfg, _ = ctx.vx_autotune(n=n3, L=tuple(0.43 * n for n in n3), n_psi=N, n_phi=R, prec=prec)
    say(n3, prec, cfg)
    assert cfg["c_split"] in (1, 2, 4, 8)
    ctx.close()


def test_stored_automatic_groups(tmp_path, monkeypatch):
    n3, L3, path = (18, 16, 12), (7.0, 6.0, 5.0), str(tmp_path / "cfg.txt")
    psi, phi = (dev(synth.random_grid_vectors(84 + i, n3, k)) for i, k in enumerate((24, 3)))
    kw = dict(n=n3, L=L3, kernel="hse", omega=0.3, prec="fp64")
    ctx = Context(0)
    ctx.set_vx_config({"kernels": 2, "b_xtile": 9}, n=n3, prec="fp64")
    auto = host(ctx.apply_vx(psi, phi, **kw))
    ctx.set_vx_config({"kernels": 2, "b_xtile": 9, "c_split": 1}, n=n3, prec="fp64")
    one = host(ctx.apply_vx(psi, phi, **kw))
    assert not np.array_equal(auto, one)
    ctx.set_vx_config({"kernels": 2, "b_xtile": 9}, n=n3, prec="fp64")
    ctx.save_configs(path)
    ctx.close()
    lines = open(path).read().splitlines()
    assert lines[-1].startswith("fxcfg gfx950/") and lines[-1].endswith(" -1")
    for end, want, split in ((" -1", auto, 0), (" 0", one, 1), ("", one, 1), (" 1", one, 1)):
        with open(path, "w") as f:
            f.write(lines[-1][:-len(" -1")] + end + "\n")
        ctx = Context(0)
        assert ctx.load_configs(path) == 1
        assert ctx.get_vx_config(n=n3, prec="fp64")[0]["c_split"] == split, end
        assert np.array_equal(host(ctx.apply_vx(psi, phi, **kw)), want), end
        ctx.close()
