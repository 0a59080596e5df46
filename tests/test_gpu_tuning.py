"""What the tuner may choose: only between shapes that differ."""
import numpy as np
import pytest

import synth
from tests.gpu_util import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
def test_one_shape_is_no_choice(prec):
    """A call of 24 atoms runs its AEV kernels with four waves per centre
    whatever the sites say: they keep their defaults, so that larger calls of
    the same model do not run a shape that was picked by chance.  float32
    dense layers have two shapes, 16-row (64) and 128-row tiles (128)."""
    from paper_2207_14276_amd import NNPModel
    m = NNPModel(synth.make_model(0), prec)
    tuned = m.autotune(*to_dev(synth.make_batch([synth.config0()])))
    assert tuned and "aev_fwd_waves" not in tuned and "aev_bwd_waves" not in tuned, tuned
    if prec == "fp32":
        assert all(v in (64, 128) for k, v in tuned.items() if k.startswith("gemm")), tuned
    tuned = m.autotune(*to_dev(synth.ragged_solutes(160, seed=64)))
    assert "aev_fwd_waves" in tuned and "aev_bwd_waves" in tuned, tuned
    m.close()


def _solutes(n, count):
    rng = np.random.default_rng(n)
    return synth.make_batch([synth.random_solute(rng, n, 2.0 * n ** (1 / 3), synth.CONFIG2_PROBS) for _ in range(count)])


# (batch, neighbour capacity, several waves per centre in the forward, in the backward)
FORMS = {
    "400 solutes of 10": (lambda: _solutes(10, 400), 256, False, False),
    "80 solutes of 20": (lambda: _solutes(20, 80), 256, True, False),
    "40 solutes of 100": (lambda: _solutes(100, 40), 256, True, True),
    "water, 6,000 atoms": (lambda: synth.make_batch([synth.water_box(2000, seed=1)]), 304, False, False),
    "water, 6,000 atoms, long lists": (lambda: synth.make_batch([synth.water_box(2000, seed=1)]), 640, True, True),
}


@pytest.mark.parametrize("name", list(FORMS))
def test_waves_per_centre(name):
    """Several waves per centre only where they do not cost more than they
    give: many small molecules, and large boxes at capacities a little above
    the default, keep one wave in the backward.  (The tuner records a site
    where the call leaves it a choice.)"""
    from paper_2207_14276_amd import NNPModel
    batch, capacity, fwd, bwd = FORMS[name]
    b = batch()
    m = NNPModel(synth.make_model(0), "bf16")
    m.reserve(b.n_atoms, b.n_systems, capacity)
    tuned = m.autotune(*to_dev(b))
    assert ("aev_fwd_waves" not in tuned, "aev_bwd_waves" not in tuned) == (fwd, bwd), tuned
    m.close()
