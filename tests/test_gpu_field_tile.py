"""The allocation-free field's pass over super-block pairs (512 atoms a side)
against the allocating field: fewer atoms than a 64-atom block, one super-block
exactly and one atom more or less, several with a ragged end, more pairs than one
launch's scratch holds, fragments across block borders.  Both sum the same FP64
terms in another order: 1e-12 of the sum of magnitudes bounds far more than
their rounding."""

import os

import numpy as np
import pytest
import torch

import workloads as w

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nmol,group", [(7, 1), (170, 1), (171, 1), (256, 2), (512, 1), (400, 40), (1500, 3), (5800, 1)])
def test_field_tile(nmol, group):
    from paper_2606_28022_amd import FmoXtb
    s = w.water_droplet(nmol, radius=12.5 * (nmol / 256) ** (1 / 3) + 2.0, seed=nmol)
    s = s.grouped(group) if group > 1 else s
    names = "FX_FIELD_WAVE_MAX", "FX_FIELD_TILE_MIN"
    old = {k: os.environ.get(k) for k in names}
    os.environ.update({k: "0" for k in names})
    try:
        c = FmoXtb(device=0)
    finally:
        for k, v in old.items():
            os.environ.pop(k) if v is None else os.environ.__setitem__(k, v)
    c.set_system(s.Z, s.xyz, s.frag, s.frag_charge)
    q = np.random.default_rng(nmol).normal(0.0, 0.3, c.n_shells)
    ref, scale = c.embedding_field(q), c.embedding_field(np.abs(q))
    dq = torch.tensor(q, dtype=torch.float64, device="cuda:0")
    phi = torch.full_like(dq, float("nan"))
    for _ in range(2):
        c.embedding_field_noalloc(dq, phi)
        torch.cuda.synchronize()
        assert np.all(np.abs(phi.cpu().numpy() - ref) <= 1e-12 * np.maximum(scale, 1e-300) + 1e-300)
    c.close()
