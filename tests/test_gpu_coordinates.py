"""New coordinates for a system against the same system set afresh, and the
contact check of the coordinates on both sides of its limit (0.3 bohr), inside
a cell of 2 bohr and across its faces, edges and corners, at negative and at
large coordinates.  Both ways run the same kernels on the same tables: equal
to the last bit."""

import numpy as np
import pytest

import workloads as w

pytestmark = pytest.mark.gpu


def _results(c):
    r = c.run()
    return [np.array([r["e_total"], r["iters_mono"], r["iters_dimer"]]), *c.energies(), c.charges(), c.gradient()]


@pytest.mark.parametrize("cutoff", [4.0, 9.0])
def test_new_coordinates_equal_new_system(cutoff):
    from paper_2606_28022_amd import FmoXtb
    s = w.water_cluster_cube(n=8, seed=5)
    xyz = np.asarray(s.xyz).reshape(-1, 3)
    other = xyz * 1.05 + np.random.default_rng(1).normal(0, 0.05, xyz.shape)  # (other pair lists as well)
    a, b = FmoXtb(), FmoXtb()
    a.set_system(s.Z, s.xyz, s.frag, s.frag_charge)
    a.set_options(cutoff_bohr=cutoff)
    _results(a)
    a.set_coordinates(other)
    b.set_system(s.Z, other, s.frag, s.frag_charge)
    b.set_options(cutoff_bohr=cutoff)
    for x, y in zip(_results(a), _results(b)):
        assert np.array_equal(x, y)
    a.close()
    b.close()


@pytest.mark.parametrize("origin", [(0.9, 0.9, 0.9), (2.0, 1.0, 1.0), (-2.0, 4.0, 1.0), (6.0, -4.0, 0.0),
                                    (-1e6, 1e6 + 2, 3e5)])
def test_contact_limit(origin):
    from paper_2606_28022_amd import FmoXtb
    from paper_2606_28022_amd.binding import FxError
    rng = np.random.default_rng(3)
    d = rng.normal(size=3)
    d /= np.linalg.norm(d)
    c = FmoXtb()
    for dist, ok in ((0.2999, False), (0.3001, True)):
        far = np.array([[5.0, 5, 5], [-5, -5, -5.0]])
        xyz = np.array(origin) + np.concatenate([[-0.5 * dist * d, 0.5 * dist * d], far])
        Z, frag, q = np.ones(4, np.int32), np.array([0, 0, 1, 1], np.int32), np.zeros(2, np.int32)
        if ok:
            c.set_system(Z, xyz, frag, q)
            c.set_coordinates(xyz)
        else:
            with pytest.raises(FxError):
                c.set_system(Z, xyz, frag, q)
            c.set_system(Z, xyz + np.outer([0, 1, 0, 0], 3 * d), frag, q)
            with pytest.raises(FxError):
                c.set_coordinates(xyz)
            with pytest.raises(FxError):  # refused coordinates leave no system
                c.set_coordinates(xyz + np.outer([0, 1, 0, 0], 3 * d))
    c.close()
