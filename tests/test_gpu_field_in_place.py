"""The allocation-free field with charges and result in the same or in
overlapping memory: the call has always read every charge before it wrote a
result.  Sizes: the wave form's range, the chunked form's and the one where the
passes over super-block pairs take several launches.  Both sides sum the same
FP64 terms in another order: 1e-12 of the sum of magnitudes bounds far more
than their rounding."""

import numpy as np
import pytest
import torch

import workloads as w

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shift", [0, 1, -1, 7])
@pytest.mark.parametrize("nmol", [3, 700, 2500, 5600])
def test_result_over_the_charges(nmol, shift):
    from paper_2606_28022_amd import FmoXtb
    s = w.water_droplet(nmol, radius=12.5 * (nmol / 256) ** (1 / 3) + 2.0, seed=nmol)
    c = FmoXtb(device=0)
    c.set_system(s.Z, s.xyz, s.frag, s.frag_charge)
    n, pad = c.n_shells, abs(shift)
    q = np.random.default_rng(nmol).normal(0.0, 0.3, n)
    ref, scale = c.embedding_field(q), c.embedding_field(np.abs(q))
    buf = torch.zeros(n + 2 * pad, dtype=torch.float64, device="cuda:0")
    dq, phi = buf[pad:pad + n], buf[pad + shift:pad + shift + n]
    for _ in range(3):
        dq.copy_(torch.tensor(q))
        c.embedding_field_noalloc(dq, phi)
        torch.cuda.synchronize()
        assert np.all(np.abs(phi.cpu().numpy() - ref) <= 1e-12 * np.maximum(scale, 1e-300) + 1e-300)
    c.close()
