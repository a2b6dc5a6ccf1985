"""The monomer susceptibility M by the matrix-core kernel, one work-group per
system and a block per wave, against the kernel without matrix instructions,
through the charges' preconditioner and the gradient's response.  Monomers of 24
to 120 shells: two to eight 16-shell blocks, and one batch of uneven ones.
M enters a converged result through the response only: both sides converge the
charges to 1e-10, the gradient is first order in them."""

import os

import numpy as np
import pytest

import workloads as w
from workloads.geometry import acene

pytestmark = pytest.mark.gpu
A2B = w.ANGSTROM_TO_BOHR


def _run(rings, form):
    from paper_2606_28022_amd import FmoXtb
    Z, xyz, frag = [], [], []
    for f, r in enumerate(rings):
        z, x = acene(r)
        Z.append(z)
        xyz.append(x + [0.3 * f, 0.2 * f, 3.6 * f])
        frag.append(np.full(len(z), f))
    xyz = np.concatenate(xyz)
    xyz = (xyz + np.random.default_rng(sum(rings)).normal(0.0, 0.02, xyz.shape)) * A2B
    old = os.environ.get("FX_RESP_M")
    os.environ["FX_RESP_M"] = str(form)
    try:
        c = FmoXtb()
    finally:
        os.environ.pop("FX_RESP_M") if old is None else os.environ.__setitem__("FX_RESP_M", old)
    c.set_system(np.concatenate(Z).astype(np.int32), xyz, np.concatenate(frag).astype(np.int32),
                 np.zeros(len(rings), np.int32))
    c.set_options(cutoff_bohr=0.0)  # monomers only
    r = c.run()
    out = r, c.charges(), c.gradient()
    c.close()
    return out


# shells: 12 rings + 12 (benzene 24, naphthalene 36, ..., nonacene 120)
@pytest.mark.parametrize("rings", [(1, 1), (2, 2, 2), (3, 3), (4, 4), (5, 5, 5), (6, 6), (7, 7), (8, 8), (9, 9), (9, 1, 4)])
def test_forms_of_the_susceptibility(rings):
    r0, q0, g0 = _run(rings, 0)
    for form in (1, 2):
        r, q, g = _run(rings, form)
        assert r["converged"] and r0["converged"]
        assert abs(r["e_total"] - r0["e_total"]) < 1e-9
        assert np.abs(q - q0).max() < 1e-9
        assert np.abs(g - g0).max() < 5e-9
