"""Anderson mixing on nearly dependent residuals: radical anthracenes, whose first
SCC takes about a hundred iterations, and a monomer loop started from solves cut
short.  Counted are the iterations: the mixers' coefficients come from a Gram
system whose condition exceeds 1e12, so a less accurate solution of it costs
iterations long before it shows in a result.  (Gaussian elimination on one
thread: 3,435 iterations and a loop of 18 steps; Gauss-Jordan by a wave 4,116
and no convergence in 200.)"""

import numpy as np
import pytest

import workloads as w

pytestmark = pytest.mark.gpu


def _run(seed, charge, **options):
    from paper_2606_28022_amd import FmoXtb
    s = w.anthracene_crystal(reps=(1, 1, 2), sigma=0.05, seed=seed)
    q = np.zeros(s.n_frag, np.int32)
    q[0] = charge
    c = FmoXtb()
    c.set_system(s.Z, s.xyz, s.frag, q)
    c.set_options(want_gradient=0, **options)
    r = c.run(allow_noconv=True)
    c.close()
    return r


def test_radical_iterations():
    runs = [_run(seed, charge) for charge in (1, -1) for seed in range(4)]
    assert all(r["converged"] for r in runs)
    assert sum(r["iters_mono"] for r in runs) < 3800


@pytest.mark.parametrize("seed,charge", [(2, 1), (0, 1), (1, -1), (3, -1)])
def test_loop_after_short_solves(seed, charge):
    r = _run(seed, charge, cutoff_bohr=0.0, max_iter=12)
    assert r["macro_iter"] < 100
