"""Overlap and core Hamiltonian from the table of primitive pairs against the
oracle: all elements of the parameters in one system (fewer atoms than the
four-lane form's limit), systems with some of them only and in another order
(the table holds the elements present), and a fragment with more pairs than a
pass of a work-group.  The oracle sums the same at most 36 terms, each below
1, in another order: 1e-12."""

import numpy as np
import pytest

import workloads as w
from oracle import xtb as X

pytestmark = pytest.mark.gpu
A2B = w.ANGSTROM_TO_BOHR


@pytest.mark.parametrize("symbols", [(1, 1), (6, 1), (8, 1, 1), (7, 6, 8, 1), (1, 8, 7, 6, 6, 1), (6, 7, 1, 8) * 10])
def test_matrices_from_table(params, symbols):
    from paper_2606_28022_amd import FmoXtb
    rng = np.random.default_rng(len(symbols))
    n = len(symbols)
    grid = np.stack(np.meshgrid(*[np.arange(4)] * 3), -1).reshape(-1, 3)[:n] * 1.5
    xyz = (grid + rng.normal(0.0, 0.1, (n, 3))) * A2B
    Z = np.array(symbols, np.int32)
    c = FmoXtb()
    # another system first: its table is replaced
    c.set_system(np.array([8, 1, 1], np.int32), np.array([[0, 0, 0], [0, 0, 1.8], [0, 1.8, 0.0]]), np.zeros(3, np.int32),
                 np.zeros(1, np.int32))
    c.set_system(Z, xyz, np.zeros(n, np.int32), np.zeros(1, np.int32))
    S, H = c.cluster_matrices((0,))
    ref = X.XtbSystem(params, Z, xyz, X.coordination_numbers(params, Z, xyz))
    assert np.abs(S - ref.S).max() < 1e-12
    assert np.abs(H - ref.H0).max() < 1e-12
    c.close()
