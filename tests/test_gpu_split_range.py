"""Magnitudes at the ends of what a float32 value's three bfloat16 parts hold:
networks whose values lie near 2^-122, where a part would fall below the
smallest bfloat16, keep every bit.

Every sum below that could lose bits has terms of one sign and size, so that a
lost bit shows whole: a value v (1 + 2^-12) without its last bit is off by
2.4e-4.  Bars: float32 rounding of sums of at most 64 terms over six layers,
6 (64 / 2 + 4) 2^-24 = 1.3e-5 of a sum of one sign where the layers round at
random (a rounding error each, none above half an ulp of the partial sum), so
2e-5 of the largest atomic energy and, with an AEV gradient (1e-5) behind it,
4e-5 of the largest force."""
import numpy as np
import pytest

import synth
from tests.gpu_util import log, run_gpu

pytestmark = pytest.mark.gpu

HIDDEN = {"chain": (64, 64, 32), "layers": (64, 64, 64, 32, 32)}
TINY = np.float32(2.0 ** -122 * (1 + 2.0 ** -12))


def tiny_network(where, hidden):
    """Networks with values of about 2^-122 that count: `where` says which."""
    spec = synth.make_model(3, hidden={s: hidden for s in range(7)})
    w = spec.weights.copy()
    last = len(hidden) - 1                        # the last hidden layer
    for _, _, l, ws, bs, n_out, n_in in spec.layer_slices():
        if where in ("weights", "activations") and l < 2:
            # h_0 = 2^122 and 64 weights of 2^-122 (1 + 2^-12) to each channel
            # of the next layer, or the other way round: h_1 = 64 (1 + 2^-12)
            big, small = np.float32(2.0 ** 122), TINY
            w[ws] = 0.0 if l == 0 else (small if where == "weights" else big)
            w[bs] = (big if where == "weights" else small) if l == 0 else 0.0
        elif where == "gradients" and l >= last:
            # h_last is 2^122 times as large, and w_out 2^-122: dE/dh_last
            if l == last:
                w[ws] *= np.float32(2.0 ** 122)
                w[bs] *= np.float32(2.0 ** 122)
            else:
                w[ws] = np.where(w[ws] < 0, -TINY, TINY)
        elif where != "gradients":
            w[ws] = np.abs(w[ws])                 # one sign
            w[bs] = 0.0
    spec.weights = w
    return spec


@pytest.mark.parametrize("hidden", list(HIDDEN))
@pytest.mark.parametrize("where", ["weights", "activations", "gradients"])
def test_values_near_the_smallest_float(oracle_lib, where, hidden):
    from paper_2207_14276_amd import NNPModel
    spec = tiny_network(where, HIDDEN[hidden])
    b = synth.make_batch([synth.config0()] + synth.ragged_solutes(3, seed=61).systems)
    m = NNPModel(spec, "fp32")
    out = run_gpu(m, b, virial=False)
    ref = oracle_lib.batch_energy_forces(b, oracle_lib.OracleModel(spec))
    e_ref, f_ref = np.concatenate(ref["e_atom"]), np.concatenate(ref["forces"])
    de = np.abs(out["e_atom"] - e_ref).max() / np.abs(e_ref).max()
    df = np.abs(out["forces"] - f_ref).max()
    log(f"[tiny] {where} {hidden}: |E_i| {np.abs(e_ref).max():.3g} error {de:.2e}; |F| {np.abs(f_ref).max():.3g} error {df:.2e}")
    if where == "gradients":
        assert df <= 4e-5 * np.abs(f_ref).max()
    else:
        assert de <= 2e-5
    m.close()
