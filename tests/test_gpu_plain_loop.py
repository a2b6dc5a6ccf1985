"""One system at a time (FX_PLAIN_LOOP): the same bits as the batched schedules,
gradient and warm-started clusters included.  Sizes: pairs of at most 32 AOs
(one wave per system), pairs and trimers with the FP64 and with the FP32
factor of the initial basis."""

import numpy as np
import pytest

import workloads as w

pytestmark = pytest.mark.gpu


def _system(kind):
    if kind == "water":
        return w.water_cluster_cube(n=8, seed=1)
    if kind == "grouped":
        return w.water_droplet(n=24, radius=5.55, seed=3).grouped(6)
    if kind == "anthracene":
        return w.anthracene_crystal(reps=(1, 1, 2), sigma=0.05, seed=1)
    return w.pentacene_crystal(reps=(1, 1, 2), sigma=0.05, seed=1)


@pytest.mark.parametrize("kind,order", [("water", 2), ("water", 3), ("grouped", 2), ("anthracene", 2), ("anthracene", 3),
                                        ("pentacene", 2)])
def test_plain_loop_gradient(kind, order):
    from paper_2606_28022_amd import FmoXtb
    from paper_2606_28022_amd.binding import FX_BATCHED, FX_PLAIN_LOOP
    s = _system(kind)
    moved = s.xyz + np.random.default_rng(2).normal(0.0, 0.01, s.xyz.shape)
    out = []
    for schedule in (FX_PLAIN_LOOP, FX_BATCHED):
        c = FmoXtb()
        c.set_system(s.Z, s.xyz, s.frag, s.frag_charge)
        c.set_options(schedule=schedule, order=order, warm_clusters=1)
        steps = []
        for xyz in (None, moved):
            if xyz is not None:
                c.set_coordinates(xyz)
            r = c.run()
            steps.append((r["e_total"], r["iters_dimer"], r["warm_dimers"], c.charges(), c.gradient()))
        out.append(steps)
        c.close()
    for a, b in zip(*out):
        assert a[:3] == b[:3]
        assert np.array_equal(a[3], b[3]) and np.array_equal(a[4], b[4])
