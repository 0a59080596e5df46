"""Calls of 65,536 centres and more deal them to the XCDs in runs of 256: every
centre is still taken once, at the edge of the rule and with a last run that
is not whole."""
import numpy as np
import pytest

import synth
from tests.gpu_util import run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("extra", [0, 1, 40, 2048 * 9 + 255])
def test_every_centre_once(extra):
    """65,520 + extra atoms (the rule's line is at 65,536): the same energies
    and forces as in calls of a part of the systems each."""
    from paper_2207_14276_amd import NNPModel
    rng = np.random.default_rng(extra)
    kinds = [synth.random_solute(rng, 40, 7.5, synth.CONFIG2_PROBS) for _ in range(13)]
    sizes = [40] * (extra // 40) + ([extra % 40] if extra % 40 else [])
    tail = [synth.System(kinds[k % 13].coords[:n], kinds[k % 13].species[:n], kinds[0].box) for k, n in enumerate(sizes)]
    b = synth.make_batch([kinds[k % 13] for k in range(1638)] + tail)
    assert b.n_atoms == 65520 + extra
    m = NNPModel(synth.make_model(0), "bf16")
    m.reserve(b.n_atoms, b.n_systems, 64)
    whole = run_gpu(m, b)
    part = run_gpu(m, synth.make_batch(kinds + tail[-1:]))
    o = b.offsets
    for k in range(b.n_systems):
        if k < 1638 or len(b.systems[k].species) == 40:
            j = k % 13 if k < 1638 else (k - 1638) % 13
            assert whole["energy"][k] == part["energy"][j]
            assert np.array_equal(whole["forces"][o[k]:o[k + 1]], part["forces"][40 * j:40 * j + 40])
    if tail:
        assert whole["energy"][-1] == part["energy"][-1]
    m.close()
