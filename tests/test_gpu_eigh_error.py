"""Errors of the batched eigensolver on a ragged batch, in units of n times the
rounding unit times the norm, the size of a backward-stable solver's: the
thousands of rotations of a cold solve must not add up beyond it."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("largest", [60, 130, 232, 256])
@pytest.mark.parametrize("seed", [0, 1])
def test_rotations_do_not_add_up(largest, seed):
    from paper_2606_28022_amd import FmoXtb
    rng = np.random.default_rng(seed)
    mats = []
    for n in np.linspace(12, largest, 24).astype(int):
        a = rng.normal(0.0, 0.05, (n, n))
        mats.append((a + a.T) / 2 + np.diag(rng.uniform(-1.2, 0.8, n)))
    c = FmoXtb()
    unit = largest * np.finfo(float).eps
    for m, (w, V) in zip(mats, c.eigh_batched(mats)):
        ref = np.linalg.eigvalsh(m)
        norm = np.abs(ref).max()
        assert np.abs(V @ V.T - np.eye(len(m))).max() < unit
        assert np.abs(np.sort(w) - ref).max() < unit * norm
        assert np.abs(V @ m - w[:, None] * V).max() < 10 * unit * norm
    c.close()
