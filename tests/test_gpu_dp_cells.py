"""DeepPot backward on grids whose reserved cells are mostly empty."""
import numpy as np
import pytest
import torch

import synth
from tests.gpu_util import FP32_E_ATOM, FP32_F, run_gpu, to_dev

pytestmark = pytest.mark.gpu


def _dense(n, side=1.2):
    return synth.random_solute(np.random.default_rng(n), n, side * n ** (1 / 3), synth.CONFIG2_PROBS)


# one cell of 130, 250 and 256 reserved; eight (more than 512 reserved); beside
# a second system, whose cells follow
SYSTEMS = {
    "520": lambda: [_dense(520)],
    "990": lambda: [_dense(990)],
    "1024 in one cell": lambda: [_dense(1024, 1.15)],
    "2100": lambda: [_dense(2100, 1.4)],
    "a box, 600, 7": lambda: [synth.water_box(216, seed=1), _dense(600), _dense(7)],
}


@pytest.mark.parametrize("name", list(SYSTEMS))
def test_crowded_cells(oracle_lib, name):
    """Forces, and virials from the shares of a cell: the oracle's."""
    from paper_2207_14276_amd import NNPModel
    b = synth.make_batch(SYSTEMS[name]())
    spec = synth.make_dp_model(0)
    m = NNPModel(spec, "fp32")
    m.reserve(b.n_atoms, b.n_systems, 1024)
    out = run_gpu(m, b)
    ref = oracle_lib.batch_energy_forces(b, oracle_lib.OracleModel(spec))
    f_ref = np.concatenate(ref["forces"])
    assert np.abs(out["e_atom"] - np.concatenate(ref["e_atom"])).max() <= FP32_E_ATOM
    assert np.abs(out["forces"] - f_ref).max() <= FP32_F * max(1.0, np.abs(f_ref).max() / 100)
    for k in range(b.n_systems):
        w = out["virial"][k]
        # the virial of a system without a box is the sum of r (x) F
        if not np.any(np.asarray(b.boxes[k]) > 0):
            a, e = int(b.offsets[k]), int(b.offsets[k + 1])
            x = b.coords[a:e].astype(np.float64)
            want = (x - x.mean(0)).T @ out["forces"][a:e]
            lever = np.abs(x - x.mean(0)).T @ np.abs(out["forces"][a:e])
            assert np.abs(w - want).max() <= 2e-5 * lever.max() + 1e-3
    m.close()


def test_one_crowded_cell_does_not_hold_the_call():
    """520 atoms in one cell: the backward takes less than the rest of the
    call (1.7 times as long when one workgroup took them all)."""
    from paper_2207_14276_amd import NNPModel
    b = synth.make_batch([_dense(520)])
    m = NNPModel(synth.make_dp_model(0), "bf16")
    m.reserve(b.n_atoms, 1, 512)
    d = to_dev(b)
    t = {}
    for forces in (False, True):
        out = m.energy_forces(*d, forces=forces, check=True)
        best = 1e9
        for _ in range(8):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            for _ in range(20):
                m.energy_forces(*d, forces=forces, out=out)
            end.record()
            torch.cuda.synchronize()
            best = min(best, start.elapsed_time(end))
        t[forces] = best
    assert t[True] < 2 * t[False], t
    m.close()
