"""AEV kernels: species-sorted lists and the stream of pair blocks at their
edges: rows of up to 64, 128 (kept in registers) and more entries, one to
seven species (four byte counters a word), a list and none, blocks that end
inside, at the end of and past a pass of 64 pairs; against the float64 oracle."""
import numpy as np
import pytest

import synth
from tests.gpu_util import FP32_E_ATOM, FP32_F, run_gpu, to_dev

pytestmark = pytest.mark.gpu


def _dense(n, n_species, seed):
    rng = np.random.default_rng(seed)
    s = synth.random_solute(rng, n, 2.0 * n ** (1.0 / 3.0), synth.CONFIG2_PROBS, dmin=0.9)
    return synth.System(s.coords, rng.integers(0, n_species, n).astype(np.int32), s.box)


@pytest.mark.parametrize("n_species", [1, 4, 5, 7])
@pytest.mark.parametrize("n", [2, 3, 9, 12, 64, 65, 66, 128, 129, 130, 200])
def test_lists_and_streams(oracle_lib, n, n_species):
    """Features |dG| <= 2e-5 (1 + |G|); energies and forces to the float32
    bars, relative to the largest value where that is above one; the same
    forces with and without a list (the entries come in the same order)."""
    from paper_2207_14276_amd import NNPModel
    spec = synth.make_model(0)
    s = _dense(n, n_species, 100 * n + n_species)
    b = synth.make_batch([s])
    m = NNPModel(spec, "fp32")
    m.reserve(b.n_atoms, 1, 256)
    want = oracle_lib.aev(s.coords, s.species, s.box, spec.aev)
    got = m.aev(*to_dev(b)).cpu().numpy().astype(np.float64)
    assert (np.abs(got - want) <= 2e-5 * (1 + np.abs(want))).all()
    ora = oracle_lib.batch_energy_forces(b, oracle_lib.OracleModel(spec))
    plain = run_gpu(m, b)
    e, f = np.abs(ora["e_atom"][0]).max(), np.abs(ora["forces"][0]).max()
    assert np.abs(plain["e_atom"] - ora["e_atom"][0]).max() <= FP32_E_ATOM * max(e, 1.0)
    assert np.abs(plain["forces"] - ora["forces"][0]).max() <= FP32_F * max(f, 1.0)
    m.reserve(b.n_atoms, 1, n - 1 if n > 2 else 1)  # the least capacity that needs no list
    bare = run_gpu(m, b)
    assert np.array_equal(bare["forces"], plain["forces"]) and np.array_equal(bare["e_atom"], plain["e_atom"])
    m.close()
