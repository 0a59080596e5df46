"""A model may be used on any stream as soon as its creation returns."""
import numpy as np
import pytest
import torch

import synth
from tests.gpu_util import to_dev

pytestmark = pytest.mark.gpu

# one hidden layer; too wide for the fused chain; the chain
HIDDEN = [(64,), (288, 288), (256, 192, 160)]


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("hidden", HIDDEN, ids=str)
def test_first_call_on_a_stream_of_its_own(prec, hidden):
    """Eight networks are created and called at once on a stream that does not
    wait for the null stream: the bits of a later call."""
    from paper_2207_14276_amd import NNPModel
    b = synth.ragged_solutes(2, seed=66)
    c, s, bx, o = to_dev(b)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    for seed in range(3):
        spec = synth.make_model(seed, n_ensemble=8, hidden={q: hidden for q in range(7)})
        m = NNPModel(spec, prec)
        with torch.cuda.stream(side):
            first = m.energy_forces(c, s, bx, o, atom_energy=True)
        torch.cuda.synchronize()
        later = m.energy_forces(c, s, bx, o, atom_energy=True, check=True)
        for k in ("energy", "forces", "atom_energy"):
            assert np.array_equal(getattr(first, k).cpu().numpy(), getattr(later, k).cpu().numpy())
        m.close()
