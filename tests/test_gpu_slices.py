"""Small batches whose systems are spread over several work-groups against one
work-group per system (FX_SLICES=1), and the pair rules against their
definition.

Sizes: basis sizes on both sides of 32, 64 and 128 AOs (one, two, four and
eight slices), shell counts on both sides of 64 (the susceptibility kernel's
two block counts); fragments of 1 to 70 atoms for the contacts.  The slices
change the order of a few sums only, so the SCC takes the same steps: 1e-10;
contacts are decided exactly."""

import os

import numpy as np
import pytest

import workloads as w
from workloads.geometry import acene

pytestmark = pytest.mark.gpu
A2B = w.ANGSTROM_TO_BOHR


def _run(s, **env):
    from paper_2606_28022_amd import FmoXtb
    old = {k: os.environ.get(k) for k in env}
    os.environ.update(env)
    try:
        c = FmoXtb()
    finally:
        for k, v in old.items():
            os.environ.pop(k) if v is None else os.environ.__setitem__(k, v)
    Z, xyz, frag = s
    c.set_system(Z, xyz, frag, np.zeros(frag.max() + 1, np.int32))
    r = c.run()
    out = r, c.energies(), c.charges(), c.gradient()
    c.close()
    return out


def _stack(rings, copies):
    Z, X = acene(rings)
    rng = np.random.default_rng(rings)
    xyz = np.concatenate([X + [0.3 * k, 0.2 * k, 3.5 * k] for k in range(copies)])
    return (np.tile(Z, copies).astype(np.int32), (xyz + rng.normal(0, 0.02, xyz.shape)) * A2B,
            np.repeat(np.arange(copies), len(Z)).astype(np.int32))


@pytest.mark.parametrize("rings,copies", [(1, 2), (2, 3), (3, 2), (5, 2), (6, 2)])
def test_sliced_systems_match_whole(rings, copies):
    s = _stack(rings, copies)
    a, b = _run(s), _run(s, FX_SLICES="1")
    assert abs(a[0]["e_total"] - b[0]["e_total"]) < 1e-10
    for x, y in zip(a[1], b[1]):
        assert x.size == 0 or np.abs(x - y).max() < 1e-10
    assert np.abs(a[2] - b[2]).max() < 1e-10
    assert np.abs(a[3] - b[3]).max() < 1e-9


@pytest.mark.parametrize("sizes", [(1, 1, 2), (3, 3, 3, 3), (1, 5, 16, 2), (17, 64, 3), (70, 1, 33, 65)])
def test_pair_contacts_by_definition(sizes):
    from paper_2606_28022_amd import FmoXtb
    rng = np.random.default_rng(sum(sizes))
    xyz, frag = [], []
    for f, n in enumerate(sizes):
        g = np.stack(np.meshgrid(*[np.arange(5)] * 3), -1).reshape(-1, 3)[:n] * 1.6
        xyz.append(g + rng.normal(0, 0.05, (n, 3)) + rng.uniform(0, 12, 3) + [11.0 * f, 0, 0])
        frag += [f] * n
    xyz = np.concatenate(xyz)
    frag = np.array(frag, np.int32)
    Z = np.ones(len(frag), np.int32)
    charge = np.array([n % 2 for n in sizes], np.int32)
    d2 = ((xyz[:, None] - xyz[None]) ** 2).sum(-1)
    F = len(sizes)
    dmin = {(i, j): d2[np.ix_(frag == i, frag == j)].min() for i in range(F) for j in range(i + 1, F)}
    c = FmoXtb()
    c.set_system(Z, xyz, frag, charge)
    for cut in sorted(np.sqrt(list(dmin.values())) * 1.0001)[:3]:
        c.set_options(cutoff_bohr=float(cut))
        scc = {tuple(p) for p in np.sort(c.build_lists()[0], axis=1).tolist()}
        assert scc == {p for p, d in dmin.items() if d < cut * cut}
    c.close()
