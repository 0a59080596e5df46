"""The AEV kernels' forms with several waves per centre (few centres, or long
lists) against the one-wave form: the same sums in the same order, so the same
energies, forces and virials bit for bit."""
import numpy as np
import pytest

import synth
from tests.gpu_util import run_gpu

pytestmark = pytest.mark.gpu


def _same(a, b, sl):
    assert np.array_equal(a["energy"], b["energy"][sl[0]:sl[0] + 1])
    assert np.array_equal(a["e_atom"], b["e_atom"][sl[1]:sl[2]])
    assert np.array_equal(a["forces"], b["forces"][sl[1]:sl[2]])
    assert np.array_equal(a["virial"], b["virial"][sl[0]:sl[0] + 1])


# atoms of a solute without a list: one to two 64-entry chunks, their edges,
# and more chunks than waves
@pytest.mark.parametrize("n", [1, 2, 9, 64, 65, 66, 129, 300])
@pytest.mark.parametrize("prec", ["fp32", "bf16"])
def test_alone_equals_large_batch(prec, n):
    from paper_2207_14276_amd import NNPModel
    rng = np.random.default_rng(n)
    one = synth.random_solute(rng, n, 1.2 * n ** (1.0 / 3.0), synth.CONFIG2_PROBS)
    batch = synth.make_batch(synth.ragged_solutes(70, seed=61).systems + [one])  # above 4,096 atoms: a wave per centre
    m = NNPModel(synth.make_model(0), prec)
    m.reserve(batch.n_atoms, batch.n_systems, 304)
    k = batch.n_systems - 1
    _same(run_gpu(m, synth.make_batch([one])), run_gpu(m, batch), (k, int(batch.offsets[k]), int(batch.offsets[k + 1])))
    m.close()


@pytest.mark.parametrize("n_mol,copies", [(60, 8), (341, 2)])
def test_lists_alone_and_at_a_large_capacity(n_mol, copies):
    """Periodic boxes (neighbour lists): alone (at most 1,024 atoms), several
    in one call, and at a capacity whose lists take four waves per centre."""
    from paper_2207_14276_amd import NNPModel
    boxes = [synth.water_box(n_mol, seed=70 + k) for k in range(copies)]
    b = synth.make_batch(boxes)
    m = NNPModel(synth.make_model(0), "fp32")
    m.reserve(b.n_atoms, copies, 128)
    whole = run_gpu(m, b)
    alone = run_gpu(m, synth.make_batch(boxes[-1:]))
    k = copies - 1
    _same(alone, whole, (k, int(b.offsets[k]), int(b.offsets[k + 1])))
    m.reserve(b.n_atoms, copies, 640)
    wide = run_gpu(m, b)
    for key in ("energy", "e_atom", "forces", "virial"):
        assert np.array_equal(wide[key], whole[key])
    m.close()
