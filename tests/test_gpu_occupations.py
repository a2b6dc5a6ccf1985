"""Occupations of single fragments: gapped levels (Newton root), odd electron
counts and closing gaps (bisection), against the FP64 oracle."""

import numpy as np
import pytest

import workloads as w
from oracle import xtb as X

pytestmark = pytest.mark.gpu
A2B = w.ANGSTROM_TO_BOHR


def _fragment(kind):
    if kind.startswith("h2"):  # the gap closes with the distance
        return np.array([1, 1], np.int32), np.array([[0.0, 0, 0], [float(kind[3:]), 0, 0]]), 0
    s = w.water_cluster_cube().subset([0])
    if kind == "oh":
        return s.Z[:2], s.xyz[:2], 0
    if kind == "pentacene":
        s = w.pentacene_crystal((1, 1, 1)).subset([0])
    return s.Z, s.xyz, 1 if kind == "water+" else 0


@pytest.mark.parametrize("kind", ["water", "water+", "oh", "h2:1.4", "h2:5.0", "h2:6.0", "h2:9.0", "h2:12.0", "pentacene"])
def test_single_fragment_matches_oracle(kind, params):
    from paper_2606_28022_amd import FmoXtb
    Z, xyz, charge = _fragment(kind)
    cn = X.coordination_numbers(params, Z, xyz)
    sm = X.XtbSystem(params, Z, xyz, cn, charge)
    ro = X.scc(sm, tol=1e-11, etol=1e-12, maxiter=2000, beta=0.2)
    assert ro.converged
    c = FmoXtb()
    c.set_system(Z, xyz, np.zeros(len(Z), np.int32), np.array([charge], np.int32))
    c.set_options(want_gradient=0)
    r = c.run()
    # the SCC stops at 1e-10 in the charges; the energy is stationary in them
    assert abs(r["e_total"] - ro.e_int) < 1e-9
    assert np.abs(c.charges() - ro.q).max() < 2e-9
    c.close()
