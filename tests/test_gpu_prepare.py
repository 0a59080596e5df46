"""Small calls (at most 4,096 atoms, or as many per system): ingest, cells and
species buckets by one workgroup, against the same systems in a larger call,
which takes the separate kernels: the same lists and sums, so the same results
bit for bit.  (Batches of small systems without a box are searched by system,
in atom order, and others by cells: the larger call is one of the same kind.)"""
import numpy as np
import pytest
import torch

import synth
from tests.gpu_util import run_gpu, to_dev

pytestmark = pytest.mark.gpu

RC = 5.2


def _solute(n, seed):
    return synth.random_solute(np.random.default_rng(seed), n, 2.4 * n ** (1.0 / 3.0), synth.CONFIG2_PROBS)


def _gas(n, edge, seed):
    s = _solute(n, seed)
    box = np.full(3, edge, np.float32)
    return synth.System(s.coords - np.float32(0.3) * box, s.species, box)  # some atoms outside the box


# one system: one and four atoms per thread and their edges, without a box
# and in boxes of 1, 4,096 (the most prepared so) and 4,913 cells
ONE = {"n1_box": lambda: _gas(1, 7.0, 1), "n513": lambda: _solute(513, 2), "n1024": lambda: _solute(1024, 3),
       "n1025": lambda: _solute(1025, 4), "n4095": lambda: _solute(4095, 5), "n4096": lambda: _solute(4096, 6),
       "box_1_cell": lambda: _gas(65, 9.0, 7), "box_4096_cells": lambda: _gas(700, 16.2 * RC, 8),
       "box_4913_cells": lambda: _gas(700, 17.2 * RC, 9), "water": lambda: synth.water_box(512, seed=10)}


@pytest.fixture(scope="module")
def big():
    return _solute(4200, 11)


def _model(kind):
    from paper_2207_14276_amd import NNPModel
    m = NNPModel(synth.make_model(0) if kind == "aev" else synth.make_dp_model(0), "fp32")
    return m


def _check(m, systems, more, keys):
    b = synth.make_batch(systems)
    both = synth.make_batch(list(systems) + more)
    m.reserve(both.n_atoms, both.n_systems, 304)
    got, want = run_gpu(m, b), run_gpu(m, both)
    for key in keys:
        k = b.n_systems if key in ("energy", "virial") else b.n_atoms
        assert np.array_equal(got[key], want[key][:k]), key
    c, s, x, o = to_dev(b)
    cnt, ent = m.neighbors(c, s, x, o, 304)
    c, s, x, o = to_dev(both)
    cnt2, ent2 = m.neighbors(c, s, x, o, 304)
    assert torch.equal(cnt, cnt2[:b.n_atoms]) and torch.equal(ent, ent2[:b.n_atoms])


AEV_KEYS = ("energy", "e_atom", "forces", "virial")
DP_KEYS = ("energy", "e_atom")  # (DeepPot forces add up by float atomics, in no fixed order)


@pytest.mark.parametrize("case", list(ONE))
@pytest.mark.parametrize("kind", ["aev", "dp"])
def test_one_system(kind, case, big):
    m = _model(kind)
    _check(m, [ONE[case]()], [big], AEV_KEYS if kind == "aev" else DP_KEYS)
    m.close()


# several: all small without a box (1,024 systems and one more, empty ones
# among them; 4,096 atoms), and mixed with a box
@pytest.mark.parametrize("kind", ["aev", "dp"])
@pytest.mark.parametrize("case", ["few", "s1024", "s1025", "n4096", "mixed"])
def test_several_systems(kind, case, big):
    empty = synth.System(np.zeros((0, 3), np.float32), np.zeros(0, np.int32), np.zeros(3, np.float32))
    sizes = {"few": [1, 9, 130, 512], "s1024": [1, 5, 7, 2] * 255 + [2] * 4, "s1025": [1, 5, 7, 2] * 256 + [2],
             "n4096": [512] * 8, "mixed": [1, 600, 24]}[case]
    systems = [_solute(n, 20 + k) for k, n in enumerate(sizes)]
    systems[2:2] = [empty]
    if case in ("s1024", "s1025"):
        systems.pop()
    if case == "mixed":
        systems += [synth.water_box(216, seed=12), empty]
    m = _model(kind)
    more = [big] if case == "mixed" else [_solute(512, 40 + k) for k in range(9)]
    _check(m, systems, more, AEV_KEYS if kind == "aev" else DP_KEYS)
    m.close()


@pytest.mark.parametrize("kind", ["aev", "dp"])
def test_lists_of_few_and_many_cells(kind):
    """Sixteen waves per cell (one box) and four (a call of more than 512
    cells) build the same lists."""
    boxes = [synth.water_box(512, seed=50 + k) for k in range(9)]
    m = _model(kind)
    b, one = synth.make_batch(boxes), synth.make_batch(boxes[:1])
    m.reserve(b.n_atoms, len(boxes), 304)
    cnt, ent = m.neighbors(*to_dev(one), 304)
    cnt2, ent2 = m.neighbors(*to_dev(b), 304)
    assert torch.equal(cnt, cnt2[:one.n_atoms]) and torch.equal(ent, ent2[:one.n_atoms])
    m.close()


def test_persistent_lists(big):
    """Lists kept over calls: built, kept while no atom moves half the skin,
    and built again for the one system whose atom does; the same with the
    larger system in the call, and the builds counted alike."""
    from paper_2207_14276_amd import NeighborPool
    m = _model("aev")
    systems = [_solute(600, 30), synth.water_box(216, seed=31)]
    b, both = synth.make_batch(systems), synth.make_batch(systems + [big])
    n, n_big = b.n_atoms, both.n_atoms
    m.reserve(n_big, 3, 400)
    pools = NeighborPool(m, n, 400, 1.0), NeighborPool(m, n_big, 400, 1.0)
    shift = np.zeros((n, 3), np.float32)
    for step, builds in enumerate([(2, 3), (2, 3), (3, 4), (3, 4)]):
        if step == 1:
            shift[:] = np.random.default_rng(32).uniform(-0.2, 0.2, (n, 3))
        if step == 2:
            shift[700, 1] += 0.9
        res = []
        for batch, pool in ((b, pools[0]), (both, pools[1])):
            c, s, x, o = to_dev(batch)
            c[:n] += torch.as_tensor(shift, device="cuda")
            r = pool.energy_forces(c, s, x, o, o[:-1], virial=True, atom_energy=True)
            res.append(r)
        assert torch.equal(res[0].energy, res[1].energy[:2])
        assert torch.equal(res[0].forces, res[1].forces[:n])
        assert torch.equal(res[0].virial, res[1].virial[:2])
        assert (pools[0].builds(), pools[1].builds()) == builds
    for p in pools:
        p.close()
    m.close()
