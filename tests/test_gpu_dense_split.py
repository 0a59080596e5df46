"""Dense layers of the float32 model on the bfloat16 matrix cores (three-part
operands) and the fused hidden-layer chain, at the shapes where their tiles,
chunks and forms change, against the FP64 oracle.

Bars: the float32 ones of the parity tests, |dE_i| <= 1e-5 and |dF| <= 1e-3.
The products left out are below 2^-25 of the terms (about 2e-8 of a layer's
sum); what float32 accumulation of up to 1,008 terms leaves is ~1e-6."""
import numpy as np
import pytest
import torch

import synth
from tests.gpu_util import FP32_E_ATOM, FP32_F, log, run_gpu

pytestmark = pytest.mark.gpu

# hidden widths: chunk counts 1..8, one to two column blocks per wave and the
# odd ones; one and no layer after the first; more layers than the chain runs;
# widths with a partial chunk (the float32 kernels) beside them
HIDDEN = {
    "one_layer": (64,),
    "two_layers": (32, 32),
    "widths_odd_chunks": (96, 224, 160),
    "widest": (256, 256, 256, 256),
    "too_deep_for_chain": (64, 96, 64, 32, 32),
    "too_wide_for_chain": (288, 64),
    "partial_chunks": (40, 24, 16),
}


@pytest.mark.parametrize("members", [1, 3])
@pytest.mark.parametrize("name", list(HIDDEN))
def test_widths_match_oracle(oracle_lib, name, members):
    from paper_2207_14276_amd import NNPModel
    spec = synth.make_model(9, n_ensemble=members, hidden={s: HIDDEN[name] for s in range(7)})
    om = oracle_lib.OracleModel(spec)
    m = NNPModel(spec, "fp32")
    b = synth.make_batch([synth.config0(), synth.water_box(8, seed=5)] + synth.ragged_solutes(6, seed=51).systems)
    out = run_gpu(m, b, virial=False)
    ref = oracle_lib.batch_energy_forces(b, om)
    de = max(np.abs(out["e_atom"][b.offsets[k]:b.offsets[k + 1]] - ref["e_atom"][k]).max() for k in range(b.n_systems))
    df = max(np.abs(out["forces"][b.offsets[k]:b.offsets[k + 1]] - ref["forces"][k]).max() for k in range(b.n_systems))
    log(f"[split] {name} x{members}: |dE_i|={de:.2e} |dF|={df:.2e}")
    assert de <= FP32_E_ATOM and df <= FP32_F
    m.close()


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
def test_tile_forms_agree(prec):
    """Systems alone (16-row tiles, padding skipped) and in a batch large
    enough for the widest tiles give the same energies and forces bit for
    bit, whatever the tuned shape."""
    from paper_2207_14276_amd import NNPModel
    b = synth.ragged_solutes(400, seed=52)
    m = NNPModel(synth.make_model(0, n_ensemble=2), prec)
    whole = run_gpu(m, b, virial=False)
    for k in (0, 17, 399):
        a, e = int(b.offsets[k]), int(b.offsets[k + 1])
        alone = run_gpu(m, synth.make_batch([b.systems[k]]), virial=False)
        assert np.array_equal(alone["energy"][0], whole["energy"][k])
        assert np.array_equal(alone["e_atom"], whole["e_atom"][a:e])
        assert np.array_equal(alone["forces"], whole["forces"][a:e])
    m.close()


def test_values_without_a_finite_first_part(oracle_lib):
    """Activations within a rounding of the largest float (no finite bfloat16
    beside them) still give the oracle's energies; a layer that overflows
    float32 gives an infinite energy, as float32 sums do, and neither touches
    the other systems of the call."""
    from paper_2207_14276_amd import NNPModel
    hidden = {s: (64, 64, 32) for s in range(7)}
    spec = synth.make_model(3, hidden=hidden)
    w = spec.weights.copy()
    for m_, s, l, ws, bs, n_out, n_in in spec.layer_slices():
        if s == synth.S and l == 0:
            w[bs] = 3.395e38          # h_0 of the S network: above the largest bfloat16
        if s == synth.S and l == 1:
            w[ws] *= 1e-36
        if s == synth.F and l == 0:   # the F network overflows
            w[ws] = 3.0e38
            w[bs] = 3.0e38
        if s == synth.F and l > 0:
            w[ws] = np.abs(w[ws])
    spec.weights = w
    om = oracle_lib.OracleModel(spec)
    base = synth.ragged_solutes(3, seed=53).systems
    systems = []
    for k, s in enumerate(base):
        sp = s.species % 4
        if k:
            sp[:] = np.where(np.arange(s.n) % 5 == 0, (synth.S, synth.F)[k - 1], sp)
        systems.append(synth.System(s.coords, sp.astype(np.int32), s.box))
    b = synth.make_batch(systems)
    m = NNPModel(spec, "fp32")
    out = run_gpu(m, b, virial=False, forces=False)
    for k in range(2):
        a, e = int(b.offsets[k]), int(b.offsets[k + 1])
        ref = oracle_lib.energy_forces(b.coords[a:e], b.species[a:e], b.boxes[k], om, forces=False, virial=False)[1]
        err = np.abs(out["e_atom"][a:e] - ref) / np.maximum(1.0, np.abs(ref))
        log(f"[split huge] system {k}: max |E_i| {np.abs(ref).max():.3g}, relative error {err.max():.2e}")
        assert err.max() <= FP32_E_ATOM
    a, e = int(b.offsets[2]), int(b.offsets[3])
    hot = b.species[a:e] == synth.F
    assert np.all(np.isposinf(out["e_atom"][a:e][hot])) and np.all(np.isfinite(out["e_atom"][a:e][~hot]))
    m.close()
