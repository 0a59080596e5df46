"""NNPFunction.backward enqueues its work and returns, for one system and for
several."""
import pytest
import torch

import synth
from tests.gpu_util import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_sys", [1, 7])
def test_backward_does_not_wait_for_the_device(n_sys):
    from paper_2207_14276_amd import NNPFunction, NNPModel
    b = synth.ragged_solutes(n_sys, seed=63)
    m = NNPModel(synth.make_model(0), "fp32")
    c, s, bx, o = to_dev(b)
    w = torch.linspace(0.5, 1.5, n_sys, dtype=torch.float64, device=c.device)
    a = torch.randn(4096, 4096, device=c.device)
    want = None
    for turn in range(3):                         # the first turns allocate
        x = c.clone().requires_grad_(True)
        E = NNPFunction.apply(x, s, bx, o, m)
        torch.cuda.synchronize()
        for _ in range(60):                       # some 100 ms of work ahead of the backward
            a @ a
        ahead = torch.cuda.Event()
        ahead.record()
        E.backward(w)
        waited = ahead.query()
        torch.cuda.synchronize()
        if turn == 0:
            f = m.energy_forces(c, s, bx, o, check=True).forces
            atoms = torch.as_tensor(b.offsets[1:] - b.offsets[:-1], device=c.device)
            want = -torch.repeat_interleave(w.float(), atoms)[:, None] * f
        assert torch.equal(x.grad, want)
    assert not waited
    m.close()
