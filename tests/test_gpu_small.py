"""One-wave SCC solves (systems of up to 32 AOs) against the batched kernels
(FX_SMALL=0): fragments of one to four waters (8 to 32 AOs, pairs of 16 that
stay on the route and of 24 to 64, some beyond it), charged and odd-electron
fragments, tight iteration caps.  Both sides converge the charges to 1e-10;
energies are stationary in them, the gradient is first order."""

import os

import numpy as np
import pytest

import workloads as w

pytestmark = pytest.mark.gpu


def _run(s, charge=None, env=None, **opt):
    from paper_2606_28022_amd import FmoXtb
    old = {k: os.environ.get(k) for k in (env or {})}
    os.environ.update(env or {})
    try:
        c = FmoXtb()
    finally:
        for k, v in old.items():
            os.environ.pop(k) if v is None else os.environ.__setitem__(k, v)
    c.set_system(s.Z, s.xyz, s.frag, s.frag_charge if charge is None else charge)
    c.set_options(**opt)
    r = c.run(allow_noconv=True)
    out = r, c.energies(), c.charges(), c.gradient() if opt.get("want_gradient", 1) else None
    c.close()
    return out


def _compare(a, b, tol=1e-9):
    assert abs(a[0]["e_total"] - b[0]["e_total"]) < tol
    for x, y in zip(a[1], b[1]):
        assert x.size == 0 or np.abs(x - y).max() < tol
    assert np.abs(a[2] - b[2]).max() < tol
    if a[3] is not None:
        assert np.abs(a[3] - b[3]).max() < 5 * tol


@pytest.mark.parametrize("group", [1, 2, 3, 4])
@pytest.mark.parametrize("order", [2, 3])
def test_one_wave_solves_match_batched(group, order):
    s = w.water_cluster_cube(n=8, seed=5)
    s = s.grouped(group) if group > 1 else s
    _compare(_run(s, order=order), _run(s, env={"FX_SMALL": "0"}, order=order))


def test_charged_and_odd_fragments():
    s = w.ion_pair_cluster()
    _compare(_run(s), _run(s, env={"FX_SMALL": "0"}))
    s = w.water_cluster_cube(n=4, seed=2)
    q = np.array([1, 0, 0, 0], np.int32)  # an odd electron: no response
    _compare(_run(s, q, want_gradient=0), _run(s, q, env={"FX_SMALL": "0"}, want_gradient=0))


def test_iteration_caps_and_retry():
    s = w.water_cluster_cube(n=8, seed=5)
    full = _run(s)
    short = _run(s, max_iter=4)  # pairs go through the automatic retry
    assert short[0]["scc_retries"] > 0 and short[0]["converged"]
    _compare(full, short, 1e-8)
    assert not _run(s, max_iter=4, scc_retry=0)[0]["converged"]


def test_learned_guess_fallback():
    from paper_2606_28022_amd import FmoXtb
    from paper_2606_28022_amd.binding import trained_guess_model
    s = w.water_cluster_cube(n=8, seed=5)
    full = _run(s)
    blob, _ = trained_guess_model()
    c = FmoXtb()
    c.mlp_load(blob)
    c.set_system(s.Z, s.xyz, s.frag, s.frag_charge)
    # every monomer restarts after its first iteration; those left after three
    c.set_options(guess=1, guess_tau=1e-12, guess_max_iter=3)
    r = c.run()
    assert r["guess_fallbacks"] == 8 and abs(r["e_total"] - full[0]["e_total"]) < 1e-9
    c.close()
