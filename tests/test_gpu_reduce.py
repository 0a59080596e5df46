"""Per-system sums at the edges of their passes (256, 1,024 and 4,096 atoms),
with and without virials."""
import numpy as np
import pytest

import synth
from tests.gpu_util import FP32_F, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 255, 256, 257, 1023, 1025, 4095, 4096, 4097])
@pytest.mark.parametrize("kind", ["aev", "dp"])
def test_sums_and_virial_switch(kind, n):
    """The energy is the float64 sum of the atomic energies (n additions round
    by at most n * 2^-53 of the sum of magnitudes each way), it and the forces
    do not depend on the virial being asked for, and every force is written."""
    from paper_2207_14276_amd import NNPModel
    rng = np.random.default_rng(n)
    batch = synth.make_batch([synth.random_solute(rng, 3, 3.0, synth.CONFIG2_PROBS),
                              synth.random_solute(rng, n, 2.4 * n ** (1.0 / 3.0), synth.CONFIG2_PROBS)])
    m = NNPModel(synth.make_model(0) if kind == "aev" else synth.make_dp_model(0), "fp32")
    m.reserve(batch.n_atoms, 2, 304)
    a, b = run_gpu(m, batch), run_gpu(m, batch, virial=False)
    for k in range(2):
        e = a["e_atom"][int(batch.offsets[k]):int(batch.offsets[k + 1])]
        assert abs(a["energy"][k] - e.sum()) <= 2 * len(e) * 2.0 ** -53 * np.abs(e).sum()
    assert np.array_equal(a["energy"], b["energy"])
    if kind == "aev":  # (DeepPot forces add up by float atomics, in no fixed order)
        assert np.array_equal(a["forces"], b["forces"])
    else:
        assert np.abs(a["forces"] - b["forces"]).max() <= FP32_F
    assert np.isfinite(a["forces"]).all() and np.isfinite(a["virial"]).all()
    alone = run_gpu(m, synth.make_batch([batch.systems[1]]))
    assert np.array_equal(alone["energy"][0], a["energy"][1])
    assert kind == "dp" or np.array_equal(alone["virial"][0], a["virial"][1])
    m.close()
