"""What the tuner may choose: only between shapes that differ."""
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
