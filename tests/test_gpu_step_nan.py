"""A monomer loop whose charges turn into NaN reports that it has not
converged, on every route of a monomer step: the one-wave solver
(waters), orbital rotations and the eigensolver (FX_OV=0)."""

import os

import pytest

import workloads as w

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["waters", "anthracene"])
@pytest.mark.parametrize("ov", ["1", "0"])
def test_nan_step_is_no_convergence(kind, ov):
    from paper_2606_28022_amd import FmoXtb
    s = w.water_cluster_cube(n=4, seed=1) if kind == "waters" else w.anthracene_crystal(reps=(1, 1, 1), sigma=0.05, seed=1)
    env = dict(FX_FUSED_BETA="nan", FX_OV=ov)
    old = {k: os.environ.get(k) for k in env}
    os.environ.update(env)
    try:
        c = FmoXtb()
    finally:
        for k, v in old.items():
            os.environ.pop(k) if v is None else os.environ.__setitem__(k, v)
    c.set_system(s.Z, s.xyz, s.frag, s.frag_charge)
    c.set_options(max_macro=12, max_iter=20, want_gradient=0, scc_retry=0, cutoff_bohr=0.0)
    r = c.run(allow_noconv=True)
    assert not r["converged"]
    assert r["macro_iter"] == 12
    c.close()
