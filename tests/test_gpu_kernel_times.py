"""A run's kernel statistics are its own: component calls before it on the same
context add nothing to them."""

import numpy as np
import pytest

import workloads as w

pytestmark = pytest.mark.gpu


def test_component_calls_leave_no_launches_behind():
    from paper_2606_28022_amd import FmoXtb
    s = w.water_droplet(n=24, radius=5.55, seed=3).grouped(6)
    m = np.diag(np.arange(64.0)) + 0.01
    launches = []
    for calls in (0, 30):
        c = FmoXtb()
        c.set_system(s.Z, s.xyz, s.frag, s.frag_charge)
        c.run()
        for _ in range(calls):
            c.embedding_field(np.zeros(c.n_shells))
            c.eigh_batched([m, m])
        launches.append({k["name"]: k["launches"] for k in c.run()["kernels"]})
        c.close()
    a, b = launches
    assert {k: a[k] for k in a if k in b} == {k: b[k] for k in b if k in a}
