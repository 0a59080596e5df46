"""First layer and dense layers of the smallest float32 calls, whose tiles
take two chunks of columns per step: a system alone gives the energies and
forces it has in a batch of the wide tiles, bit for bit, for odd and even
numbers of chunks, one chunk and none (every output sums its products in the
same order in all forms)."""
import numpy as np
import pytest

import synth
from tests.gpu_util import run_gpu

pytestmark = pytest.mark.gpu


def _chain(species, gap):
    n = len(species)
    c = np.zeros((n, 3), np.float32)
    c[:, 0] = gap * np.arange(n)
    c[:, 1] = 0.4 * (np.arange(n) % 2)
    return synth.System(c, np.array(species, np.int32), np.zeros(3, np.float32))


@pytest.mark.parametrize("hidden", [None, (64, 96, 64, 32, 32)], ids=["default", "layer_by_layer"])
def test_alone_equals_batch(hidden):
    from paper_2207_14276_amd import NNPModel
    kw = {} if hidden is None else {"hidden": {s: hidden for s in range(7)}}
    m = NNPModel(synth.make_model(4, **kw), "fp32")
    small = [_chain([0], 1.0)]                                       # no neighbour
    small += [_chain([0, 1], 4.5)]                                   # radial columns only
    small += [_chain(list(range(k)) * 2, 1.1) for k in range(1, 8)]  # 1 to 7 species
    b = synth.make_batch(small + synth.ragged_solutes(400, seed=54).systems)
    whole = run_gpu(m, b, virial=False)
    for k in range(len(small)):
        a, e = int(b.offsets[k]), int(b.offsets[k + 1])
        alone = run_gpu(m, synth.make_batch([small[k]]), virial=False)
        assert np.array_equal(alone["e_atom"], whole["e_atom"][a:e]), k
        assert np.array_equal(alone["forces"], whole["forces"][a:e]), k
    m.close()
