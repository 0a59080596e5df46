"""Magnitudes at the ends of what a float32 value's three bfloat16 parts hold.

Networks whose values lie near 2^-122, where a part would fall below the
smallest bfloat16, keep every bit: they run on float32 operands.  Every sum below that could lose bits has terms of one sign and size, so that a
lost bit shows whole: a value v (1 + 2^-12) without its last bit is off by
2.4e-4.  Bars: float32 rounding of sums of at most 64 terms over six layers,
6 (64 / 2 + 4) 2^-24 = 1.3e-5 of a sum of one sign where the layers round at
random (a rounding error each, none above half an ulp of the partial sum), so
2e-5 of the largest atomic energy and, with an AEV gradient (1e-5) behind it,
4e-5 of the largest force.

Networks with activations above the largest bfloat16, finite and infinite,
run on the parts, and such activations' products on float32 operands."""
import numpy as np
import pytest

import synth
from tests.gpu_util import FP32_E_ATOM, FP32_F, log, run_gpu

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


# systems and members: tiles of 16 rows, two chunks per step and one; of 128 rows
SIZES = {"few": (3, 1), "more": (60, 1), "members": (60, 8)}


def wide_network(hidden, members):
    """S: h_0 is 3.395e38 (finite, above the largest bfloat16) in every
    channel, and the next weights are multiples of 2^-126 that bring it back
    (a channel's of one sign, all later ones above zero: nothing cancels).
    F, Cl: one channel of h_0 is, in the first and in the second 32; it takes
    half of h_1 to infinity or close, and weights below zero take that back to
    CELU's limit -alpha."""
    spec = synth.make_model(3, n_ensemble=members, hidden={s: hidden for s in range(7)})
    w = spec.weights.copy()
    rng = np.random.default_rng(0)
    for _, s, l, ws, bs, n_out, n_in in spec.layer_slices():
        W, b = w[ws].reshape(n_out, n_in), w[bs]
        sign = np.where(np.arange(n_out) % 2 == 0, 1.0, -1.0)
        if s == synth.S and l == 0:
            b[:] = 3.395e38
        elif s == synth.S and l == 1:
            W[:] = np.ldexp(sign[:, None] * rng.integers(1, 4096, (n_out, n_in)), -126)
        elif s == synth.S:
            W[:] = np.abs(W)
        elif s in (synth.F, synth.CL) and l == 0:
            b[5 if s == synth.F else 40] = 3.395e38
        elif s in (synth.F, synth.CL) and l == 1:
            W[:, 5 if s == synth.F else 40] = sign * rng.uniform(0.25, 4.0, n_out)
        elif s in (synth.F, synth.CL) and l == 2:
            W[:] = -0.05 - np.abs(W)
    spec.weights = w
    return spec


def magnitude(spec, species):
    """Per atom of `species`, the sum of the magnitudes of all terms."""
    total = 0.0
    for _, s, l, ws, bs, n_out, n_in in spec.layer_slices():
        if s != species:
            continue
        W, b = np.abs(spec.weights[ws].astype(np.float64)).reshape(n_out, n_in), np.abs(spec.weights[bs].astype(np.float64))
        a = b if l == 0 else W @ a + b  # (a first layer's sum beside its bias is far below a rounding)
        if n_out == 1:
            total += a[0] / spec.n_ensemble
    return total


@pytest.mark.parametrize("size", list(SIZES))
@pytest.mark.parametrize("hidden", list(HIDDEN))
def test_values_above_the_largest_bfloat16(oracle_lib, hidden, size):
    """Energies and forces of every species against the oracle: S within
    float32's n 2^-24 of the magnitudes summed (n terms in a row over all
    layers), the others within the float32 bars."""
    from paper_2207_14276_amd import NNPModel
    n_sys, members = SIZES[size]
    spec = wide_network(HIDDEN[hidden], members)
    b = synth.ragged_solutes(n_sys, seed=65)
    b = synth.make_batch([synth.System(s.coords, np.where(np.arange(s.n) % 3 == 0, synth.S + np.arange(s.n) % 9 // 3,
                                                          s.species).astype(np.int32), s.box) for s in b.systems])
    m = NNPModel(spec, "fp32")
    assert m.dense_form() == ("parts+chain" if hidden == "chain" else "parts")
    out = run_gpu(m, b, virial=False)
    ref = oracle_lib.batch_energy_forces(b, oracle_lib.OracleModel(spec))
    e_ref, f_ref = np.concatenate(ref["e_atom"]), np.concatenate(ref["forces"])
    hot = b.species == synth.S
    assert hot.any() and (b.species == synth.F).any() and (b.species == synth.CL).any()
    de, df = np.abs(out["e_atom"] - e_ref), np.abs(out["forces"] - f_ref).max()
    bar = sum(HIDDEN[hidden]) * 2.0 ** -24 * magnitude(spec, synth.S)
    log(f"[wide] {hidden} {size} N={b.n_atoms}: S |E_i| {np.abs(e_ref[hot]).max():.3g} error {de[hot].max():.2e} (bar {bar:.2e}); "
        f"others {de[~hot].max():.2e}; |dF| {df:.2e}")
    assert de[hot].max() <= bar
    assert de[~hot].max() <= FP32_E_ATOM and df <= FP32_F
    m.close()
