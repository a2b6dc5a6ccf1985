"""Systems that leave the rotation route while they are solved: the limits of
the route narrowed, or the monomer steps made to overshoot, so that a residual
or a rotation exceeds them in the middle of a loop; against the eigensolver
throughout (FX_OV=0).  Both sides converge the charges to 1e-10; the energies
are stationary in them, the gradient is first order in the density."""

import os

import numpy as np
import pytest

import workloads as w

pytestmark = pytest.mark.gpu


def _system(kind):
    if kind == "waters":  # monomers of 36 AOs, pairs of 72
        return w.water_droplet(n=24, radius=5.55, seed=3).grouped(6)
    if kind == "two":
        return w.water_droplet(n=12, radius=4.4, seed=3).grouped(6)
    return w.anthracene_crystal(reps=(1, 1, 2), sigma=0.05, seed=1)


def _run(s, options, **env):
    from paper_2606_28022_amd import FmoXtb
    old = {k: os.environ.get(k) for k in env}
    os.environ.update(env)
    try:
        c = FmoXtb()
    finally:
        for k, v in old.items():
            os.environ.pop(k) if v is None else os.environ.__setitem__(k, v)
    c.set_system(s.Z, s.xyz, s.frag, s.frag_charge)
    c.set_options(**options)
    if options.get("guess"):
        from paper_2606_28022_amd.binding import trained_guess_model
        c.mlp_load(trained_guess_model()[0])
    r = c.run(allow_noconv=True)
    out = r, c.charges(), c.gradient()
    c.close()
    return out


# beta: factor of the monomer steps (above 2 the first ones overshoot); the
# residual then rises past the limit after every monomer had come to rotate
@pytest.mark.parametrize("kind,beta,errmax", [("waters", "6", "0.1"), ("waters", "6", "1e-2"), ("anthracene", "3", "1e-2"),
                                              ("anthracene", "6", "1e-2"), ("anthracene", "1", "1e-4")])
def test_monomer_leaves_the_route_mid_loop(kind, beta, errmax):
    s = _system(kind)
    r, q, g = _run(s, dict(max_macro=60), FX_FUSED_BETA=beta, FX_OV_ERRMAX=errmax)
    r0, q0, g0 = _run(s, dict(max_macro=60), FX_OV="0")
    assert r["converged"] and r0["converged"]
    assert abs(r["e_total"] - r0["e_total"]) < 1e-9
    assert np.abs(q - q0).max() < 1e-9
    assert np.abs(g - g0).max() < 5e-9


# Narrow rotation limits send a system back to the eigensolver every few
# iterations, so that in the device-driven schedule, whose host looks at counts a
# few iterations old, systems wait for an eigensolver launch again and again.
@pytest.mark.parametrize("kind,xmax,max_iter", [("waters", "3e-4", 16), ("waters", "1e-4", 16), ("two", "3e-4", 10),
                                                ("two", "1e-4", 12), ("anthracene", "3e-4", 10),
                                                ("anthracene", "3e-4", 15), ("waters", "1e-6", 5), ("two", "1e-3", 200)])
def test_schedules_agree_at_the_iteration_limit(kind, xmax, max_iter):
    from paper_2606_28022_amd.binding import FX_BATCHED, FX_BATCHED_HOST_SYNC
    s = _system(kind)
    out = [_run(s, dict(schedule=k, max_iter=max_iter, scc_retry=0), FX_OV_XMAX=xmax)
           for k in (FX_BATCHED, FX_BATCHED_HOST_SYNC)]
    (r, q, g), (r0, q0, g0) = out
    for k in ("converged", "macro_iter", "iters_mono", "iters_dimer", "e_total"):
        assert r[k] == r0[k], k
    assert np.array_equal(q, q0) and np.array_equal(g, g0)


# The learned guess falls back after its first solve's guess_max_iter own
# iterations, however many launches these took.
@pytest.mark.parametrize("guess_max_iter", [3, 4, 5, 6])
def test_schedules_agree_on_the_guess_fallback(guess_max_iter):
    from paper_2606_28022_amd.binding import FX_BATCHED, FX_BATCHED_HOST_SYNC, FX_GUESS_LEARNED
    s = _system("waters")
    a, b = [_run(s, dict(schedule=k, guess=FX_GUESS_LEARNED, guess_max_iter=guess_max_iter, scc_tol=1e-9),
                 FX_OV_XMAX="1e-6") for k in (FX_BATCHED, FX_BATCHED_HOST_SYNC)]
    for k in ("guess_fallbacks", "iters_mono", "macro_iter", "e_total"):
        assert a[0][k] == b[0][k], k
    assert np.array_equal(a[1], b[1])
