"""DeepPot-style descriptor: the neighbour order at list lengths around the
64 entries of a pass and the 128 kept in registers, with few and many species,
and where distances tie exactly (a lattice; all ties go to the smaller index,
then the smaller image), against the float64 oracle."""
import numpy as np
import pytest

import synth
from tests.gpu_util import to_dev

pytestmark = pytest.mark.gpu

RC = 6.0


def _dense(n, n_species, seed):
    rng = np.random.default_rng(seed)
    s = synth.random_solute(rng, n, 1.15 * n ** (1.0 / 3.0), synth.CONFIG2_PROBS, dmin=0.6)
    return synth.System(s.coords, rng.integers(0, n_species, n).astype(np.int32), s.box)


def _lattice(k, a, box):
    g = (np.arange(k) * a).astype(np.float32)
    x = np.stack(np.meshgrid(g, g, g, indexing="ij"), -1).reshape(-1, 3)
    sp = np.random.default_rng(k).integers(0, 2, len(x)).astype(np.int32)
    return synth.System(x, sp, np.full(3, k * a if box else 0.0, np.float32))


def _frame_ok(s):
    """Centres whose two nearest neighbours are not near one line with them
    (a lattice's are at right angles or exactly on a line)."""
    n = len(s.species)
    if n < 3 or len(np.unique(s.coords)) < 6:
        return np.ones(n, bool)
    d = s.coords[None].astype(np.float64) - s.coords[:, None]
    r = np.sqrt((d * d).sum(-1)) + 1e9 * np.eye(n)
    near = np.argsort(r, axis=1)[:, :2]
    u = np.take_along_axis(d, near[..., None], axis=1)
    u /= np.linalg.norm(u, axis=-1, keepdims=True)
    return np.linalg.norm(np.cross(u[:, 0], u[:, 1]), axis=-1) >= 0.1


CASES = {f"n{n}_s{s}": (lambda n=n, s=s: _dense(n, s, 10 * n + s))
         for n in (2, 5, 64, 65, 66, 129, 130, 194) for s in (1, 2, 7)}
CASES["lattice"] = lambda: _lattice(5, 2.0, False)       # 125 atoms
CASES["lattice_box"] = lambda: _lattice(4, 2.5, True)    # own images tie as well


@pytest.mark.parametrize("name", list(CASES))
def test_order(oracle_lib, name):
    """Same slots filled, 1/R and x to float32 (|dG| <= 2e-5 (1 + |G|)), and y
    and z as well where the frame's neighbours are at least 0.1 rad from one
    line (nearer to it the float32 error of e_y grows as 1 / sin of the angle)."""
    from paper_2207_14276_amd import NNPModel
    spec = synth.make_dp_model(0)
    s = CASES[name]()
    b = synth.make_batch([s])
    m = NNPModel(spec, "fp32")
    m.reserve(b.n_atoms, 1, 256)
    got = m.aev(*to_dev(b)).cpu().numpy().astype(np.float64)
    want = oracle_lib.dp_descriptor(s.coords, s.species, s.box, spec.aev)
    assert np.array_equal(got[:, 0::4] != 0, want[:, 0::4] != 0)
    ok = np.abs(got - want) <= 2e-5 * (1 + np.abs(want))
    assert ok[:, 0::4].all() and ok[:, 1::4].all()
    assert ok[_frame_ok(s)].all()
    m.close()
