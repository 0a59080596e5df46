"""Device memory of a float32 model: each layer's weights in the layouts that a
call reads, and no others."""
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


def test_fused_layers_hold_no_second_set_of_parts():
    """Bytes per weight: 24 in the first layer (float32, its transpose and the
    dE/dG form, parts of two), 20 in the fused ones (float32, its transpose,
    the parts of both in fragment order).  Allocation adds up to 3 per weight
    of the fused layers here; another set of parts would add 12."""
    from paper_2207_14276_amd import NNPModel
    hidden, members = (64, 256, 256), 8
    spec = synth.make_model(0, n_ensemble=members, hidden={s: hidden for s in range(7)})
    NNPModel(spec, "fp32").close()
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    m = NNPModel(spec, "fp32")
    assert m.dense_form() == "parts+chain"
    used = free - torch.cuda.mem_get_info()[0]
    first = 7 * members * 1008 * hidden[0]
    fused = 7 * members * (hidden[0] * hidden[1] + hidden[1] * hidden[2])
    assert used <= 24 * first + 26 * fused, (used, first, fused)
    m.close()
