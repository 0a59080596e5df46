"""CELU of the float32 dense layers, value by value: networks that hand one
feature of the descriptor, times a power of two (exact), through one CELU to
the atomic energy (alpha = 1: no rounding but CELU's own).

Bar: one unit in the last place.  The exponential takes three roundings of
which two are scaled down by at least a half (0.5 + 0.25 + 0.25), and its
series ends below 2^-30 of the value; float32 arithmetic carried out on the
host gives 0.88 at most."""
import numpy as np
import pytest
import torch

import synth
from tests.gpu_util import log, to_dev

pytestmark = pytest.mark.gpu


def one_value_model(feature, scale, layers):
    """E_i = CELU(-scale G_i[feature]); layers = 2: through the fused chain."""
    spec = synth.make_model(0, hidden={s: (32,) * layers for s in range(7)}, celu_alpha=1.0)
    w = np.zeros_like(spec.weights)
    for _, _, l, ws, _, n_out, n_in in spec.layer_slices():
        W = np.zeros((n_out, n_in), np.float32)
        if l == 0:
            W[0, feature] = -scale if layers == 1 else scale
        else:
            W[0, 0] = -1.0 if (layers == 2 and l == 1) else 1.0
        w[ws] = W.ravel()
    spec.weights = w
    return spec


@pytest.mark.parametrize("layers", [1, 2])
def test_celu_to_the_last_place(layers):
    from paper_2207_14276_amd import NNPModel
    b = synth.ragged_solutes(48, seed=62)
    c, s, bx, o = to_dev(b)
    worst, seen = 0.0, np.zeros(4, int)
    for feature in (3, 20):                       # radial, of H and C neighbours
        for k in (-6, -3, -1, 0, 1, 3):
            m = NNPModel(one_value_model(feature, np.float32(2.0 ** k), layers), "fp32")
            g = m.aev(c, s, bx, o)[:, feature].cpu().numpy().astype(np.float64)
            e = m.energy_forces(c, s, bx, o, forces=False, atom_energy=True, check=True).atom_energy.cpu().numpy()
            m.close()
            t = -np.ldexp(g, k)
            live = t < -1e-30
            ref = np.expm1(t[live])
            ulp = np.abs(e[live] - ref) / np.spacing(np.abs(ref).astype(np.float32)).astype(np.float64)
            worst = max(worst, float(ulp.max()))
            seen += np.histogram(-t[live], [0, 0.3466, 0.5, 1.0, 100.0])[0]
    log(f"[celu] {layers} layer(s): {worst:.3f} ulp at most over {seen.tolist()} values")
    assert (seen > 300).all()
    assert worst <= 1.0
