"""The distance screen and the walk behind it on states outside the ordinary.
The reference is the FP64 oracle.
"""
import numpy as np
import pytest

import ljsynth

pytestmark = pytest.mark.gpu


def _say(msg):
    print(f"[case] {msg}", flush=True)


def _system(n, box, **kw):
    from paper_0709_3225_amd import LJSystem

    return LJSystem(n, box, **kw)


def _dev(a):
    import torch

    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()


def rel_l2(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def _lattice_with_a_loner(m, box):
    """A jittered FCC lattice of 4 m^3 sites less those within 2.55 of the
    origin, and one atom there (the last): it has no partner within r_c."""
    x = ljsynth.jitter(ljsynth.fcc_positions(m, box), 0.05, 60 + m) % box
    d = x - box * np.round(x / box)
    x = x[(d * d).sum(-1) > 2.55 ** 2]
    pos4 = np.zeros((len(x) + 1, 4), np.float32)
    pos4[:-1, :3] = x
    pos4[pos4 >= box] = 0.0
    vel4 = np.zeros_like(pos4)
    vel4[:, :3] = np.random.default_rng(m).normal(scale=0.3, size=(len(pos4), 3))
    return pos4, vel4


# cells of 11..16, 17..21 and 22..32 atoms mostly: each layout of the matrix screen
GRIDS = [(9, 6), (10, 6), (9, 5)]


@pytest.mark.parametrize("waves,tile", [(1, 0), (4, 0), (1, 128)])
@pytest.mark.parametrize("m,nc", GRIDS)
def test_far_candidate_leaves_other_pairs_alone(m, nc, waves, tile, orc):
    """An atom that flies 64 box lengths a step (320 cell sides and more, past
    the range of 16 bits in the screen's units) between rebuilds: the run is
    flagged, and every other atom's forces are those of its own partners. The
    flight is exact in FP32 and ends each step where it began, in a hole of the
    lattice, so the oracle's run has the same forces. Velocities after three
    steps, the second of them on the cells of the first, within 1e-5: FP32
    round-off of the trajectory; a screen that drops the pairs of three other
    candidates per neighbourhood is off by more than 1e-4."""
    from paper_0709_3225_amd import _lib as L

    box = 16.0
    pos4, vel4 = _lattice_with_a_loner(m, box)
    vel4[-1, :3] = 0.0
    vel4[-1, 0] = 64 * box * 128
    _say(f"far candidate m={m} nc={nc} waves={waves} tile={tile}")
    s = _system(len(pos4), box, dt=1 / 128, cell_min=0.999 * box / nc, waves_per_cell=waves, tile_cap=tile)
    assert s.cells_per_dim == nc
    s.load(_dev(pos4), _dev(vel4))
    s.step_every(3, 3)
    _, vel = s.state()
    assert s.check(raise_on_error=False) == L.MD_DEV_SKIN
    _, v, _ = orc.run(orc.params(box, dt=1 / 128), pos4, vel4, 3)
    assert rel_l2(vel.cpu().numpy()[:-1, :3], v[:-1]) < 1e-5
