"""The occupation cases of test_gpu_occupations.py by the batched kernels
(FX_SMALL=0): all but one of their fragments have at most 32 AOs and go to the
one-wave solver by default, which has its own Fermi level.  In addition larger
fragments whose gap closes, for the bisection of an even electron number."""

import os

import numpy as np
import pytest

import workloads as w
from oracle import xtb as X
from test_gpu_occupations import _fragment
from workloads.geometry import acene

pytestmark = pytest.mark.gpu
A2B = w.ANGSTROM_TO_BOHR


def _large(kind):
    if kind.startswith("stretched"):  # naphthalene, an H pulled off
        Z, xyz = acene(2)
        xyz = xyz.copy()
        h = int(np.argmax(Z == 1))
        c = int(np.argmin(np.where(Z == 6, np.linalg.norm(xyz - xyz[h], axis=1), 1e9)))
        u = (xyz[h] - xyz[c]) / np.linalg.norm(xyz[h] - xyz[c])
        xyz[h] = xyz[c] + float(kind[9:]) * u
        return Z.astype(np.int32), xyz * A2B, 0
    return _fragment(kind)


@pytest.mark.parametrize("kind", ["water", "water+", "oh", "h2:1.4", "h2:5.0", "h2:6.0", "h2:9.0", "h2:12.0",
                                  "stretched1.6", "stretched3.0", "stretched5.0"])
def test_batched_fragment_matches_oracle(kind, params):
    from paper_2606_28022_amd import FmoXtb
    Z, xyz, charge = _large(kind)
    cn = X.coordination_numbers(params, Z, xyz)
    sm = X.XtbSystem(params, Z, xyz, cn, charge)
    ro = X.scc(sm, tol=1e-11, etol=1e-12, maxiter=4000, beta=0.1)
    assert ro.converged
    old = os.environ.get("FX_SMALL")
    os.environ["FX_SMALL"] = "0"
    try:
        c = FmoXtb()
    finally:
        os.environ.pop("FX_SMALL") if old is None else os.environ.__setitem__("FX_SMALL", old)
    c.set_system(Z, xyz, np.zeros(len(Z), np.int32), np.array([charge], np.int32))
    c.set_options(want_gradient=0)
    r = c.run()
    # the SCC stops at 1e-10 in the charges; the energy is stationary in them
    assert abs(r["e_total"] - ro.e_int) < 1e-9
    assert np.abs(c.charges() - ro.q).max() < 2e-9
    c.close()
