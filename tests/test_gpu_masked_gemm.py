"""The dense layers on tiles whose rows have few of the AEV's 16-column halves:
live halves are gathered side by side, so tiles of one, of some and of all
species together give the same results, whatever else the call holds."""
import numpy as np
import pytest

import synth
from tests.gpu_util import run_gpu

pytestmark = pytest.mark.gpu


def _of_species(n, species, seed):
    rng = np.random.default_rng(seed)
    s = synth.random_solute(rng, n, 2.2 * n ** (1.0 / 3.0), synth.CONFIG2_PROBS)
    return synth.System(s.coords, rng.choice(species, n).astype(np.int32), s.box)


# one species: 1 + 2 halves; two: 2 + 6; four: 4 + 20; seven: 63
SETS = {"one": [3], "two": [0, 3], "four": [0, 1, 2, 6], "all": list(range(7)), "last": [6]}


@pytest.mark.parametrize("prec,members", [("bf16", 1), ("bf16", 8), ("fp32", 1), ("fp32", 8)])
@pytest.mark.parametrize("n", [1, 2, 130])
def test_live_halves(prec, members, n):
    """Each system alone (its tiles hold its own halves only) and all of them
    in one call (the tiles hold the halves of all): the same bits."""
    from paper_2207_14276_amd import NNPModel
    systems = [_of_species(n, sp, 7 * n + k) for k, sp in enumerate(SETS.values())]
    m = NNPModel(synth.make_model(0, n_ensemble=members), prec)
    both = synth.make_batch(systems + [_of_species(400, range(7), 99)] * 12)
    m.reserve(both.n_atoms, both.n_systems, 400)
    whole = run_gpu(m, both)
    for k, s in enumerate(systems):
        a, e = int(both.offsets[k]), int(both.offsets[k + 1])
        alone = run_gpu(m, synth.make_batch([s]))
        assert np.array_equal(alone["e_atom"], whole["e_atom"][a:e])
        assert np.array_equal(alone["forces"], whole["forces"][a:e])
        assert np.isfinite(alone["forces"]).all()
    m.close()
