"""The batched eigensolver's cold solve by logged passes: one batch per case
with sizes around the 64-column tiles and the FP64 / FP32 working matrices,
uneven sizes together, sizes beyond the split form, and spectra at its ends (a
unit matrix, a diagonal one, fully degenerate and nearly degenerate levels,
couplings as large as the levels).  Tolerance: rotations are applied to V in
FP64 and the last one ends on a sweep below 1e-12 of the scale, so vectors are
orthonormal to n rounding errors and residuals stay below 1e-9 of the norm."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _matrix(n, kind, rng):
    a = rng.normal(0.0, 0.05, (n, n))
    a = (a + a.T) / 2
    if kind == "levels":
        return a + np.diag(rng.uniform(-1.2, 0.8, n))
    if kind == "dense":
        return 20 * a
    if kind == "unit":
        return np.eye(n)
    if kind == "diagonal":
        return np.diag(rng.normal(size=n))
    q, _ = np.linalg.qr(rng.normal(size=(n, n)))
    w = np.repeat(rng.normal(size=(n + 3) // 4), 4)[:n] + 1e-9 * rng.normal(size=n) * (kind == "near")
    return (q * w) @ q.T


@pytest.mark.parametrize("kind", ["levels", "dense", "unit", "diagonal", "degenerate", "near"])
@pytest.mark.parametrize("sizes", [(8, 9, 31, 33), (63, 64, 65, 12), (127, 128, 130), (161, 8, 232), (255, 256), (300, 20)])
def test_cold_passes(sizes, kind):
    from paper_2606_28022_amd import FmoXtb
    rng = np.random.default_rng(sum(sizes))
    mats = [_matrix(n, kind, rng) for n in sizes]
    mats = [(m + m.T) / 2 for m in mats]
    c = FmoXtb()
    for m, (w, V) in zip(mats, c.eigh_batched(mats)):
        n = len(m)
        norm = np.abs(np.linalg.eigvalsh(m)).max()
        assert np.abs(V @ V.T - np.eye(n)).max() < 1e-11
        assert np.abs(V @ m - w[:, None] * V).max() < 1e-9 * norm
        assert np.abs(np.sort(w) - np.linalg.eigvalsh(m)).max() < 1e-9 * norm
    c.close()
