"""guess_max_iter 1 means no fallback by iterations, whatever kernel solves the
monomers (a fallback after the first iteration would throw away every guess):
the one-wave solver and the batched kernels (FX_SMALL=0) agree."""

import os

import pytest

import workloads as w

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("small", ["1", "0"])
@pytest.mark.parametrize("limit,fallbacks", [(0, 0), (1, 0), (2, 8)])
def test_guess_limit(small, limit, fallbacks):
    from paper_2606_28022_amd import FmoXtb
    from paper_2606_28022_amd.binding import FX_GUESS_LEARNED, trained_guess_model
    s = w.water_cluster_cube(n=8, seed=1)
    old = os.environ.get("FX_SMALL")
    os.environ["FX_SMALL"] = small
    try:
        c = FmoXtb()
    finally:
        os.environ.pop("FX_SMALL") if old is None else os.environ.__setitem__("FX_SMALL", old)
    c.mlp_load(trained_guess_model()[0])
    c.set_system(s.Z, s.xyz, s.frag, s.frag_charge)
    # (no monomer converges to 1e-10 in two iterations)
    c.set_options(guess=FX_GUESS_LEARNED, guess_max_iter=limit, want_gradient=0)
    assert c.run()["guess_fallbacks"] == fallbacks
    c.close()
