"""The distance screen and the walk behind it on states outside the ordinary.
The reference is the FP64 oracle.
"""
import numpy as np
import pytest

import ljsynth
from test_gpu_parity import _assert_rows

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


def _clear_of_cutoff(x, box, rc=2.5, band=1e-5):
    d = x[:, None] - x[None]
    d -= box * np.round(d / box)
    return not (np.abs(np.sqrt((d * d).sum(-1)) - rc) < band).any()


@pytest.mark.parametrize("k,waves,side", [(13, 1, 5.2), (16, 4, 6.0), (19, 1, 6.0), (21, 2, 5.2), (25, 1, 5.2),
                                          (32, 2, 6.0), (18, 1, 40.0)])
def test_matrix_screen_on_wide_cells(k, waves, side, orc):
    """Cells of more than two cutoffs, as WCA and dilute gases on cells sized by
    occupancy have, with k atoms in each: the accepted pairs are the oracle's."""
    rng = np.random.default_rng(k)
    cells = np.stack(np.meshgrid(*(np.arange(4),) * 3, indexing="ij"), -1).reshape(-1, 3)
    # k of 4^3 sites a cell, 1.3 to 1.5 apart, in the corner next to eight others
    sites = np.stack(np.meshgrid(*(np.arange(4),) * 3, indexing="ij"), -1).reshape(-1, 3) + 0.5
    at = min(side / 4, 1.5) * sites
    pts = []
    for c in cells:
        q = at[rng.choice(64, size=k, replace=False)]
        pts.append(c * side + np.where(c % 2 == 1, q, side - q))
    box = 4 * side
    for _ in range(100):
        pos4 = np.zeros((64 * k, 4), np.float32)
        pos4[:, :3] = np.concatenate(pts) + rng.uniform(-0.2, 0.2, (64 * k, 3))
        if _clear_of_cutoff(pos4[:, :3].astype(np.float64), box, band=2e-5):
            break
    _say(f"wide cells k={k} waves={waves} side={side}")
    counts_o, idx_o, guard = orc.neighbors(orc.params(box), pos4)
    assert guard == 0 and counts_o.mean() > 4
    s = _system(len(pos4), box, waves_per_cell=waves, cell_min=0.999 * side)
    assert s.cells_per_dim == 4
    s.load(_dev(pos4))
    counts, idx = s.neighbors(int(counts_o.max()) + 8)
    assert s.check() == 0
    _assert_rows(counts, idx, counts_o, idx_o)


@pytest.mark.parametrize("sign", [1, -1])
@pytest.mark.parametrize("nc,side,rho", [(4, 2.67, 0.8), (3, 3.2, 0.8), (3, 5.34, 0.17)])
def test_screen_of_atoms_outside_their_cells(nc, side, rho, sign, orc):
    """The step between rebuilds, with the whole state moving along a diagonal
    by 0.9 of what the cells allow: atoms at the faces lie outside their cells by
    0.52 of it on each axis. Truncated, unshifted force: a dropped pair at r_c
    would change a velocity by dt / 2 x 0.039 = 1.5e-4; FP32 round-off of these
    velocities and forces stays below 3e-5."""
    box, dt = nc * side, 1 / 128
    p = orc.params(box, dt=dt, shift_mode=1)
    for seed in range(100):
        rng = np.random.default_rng(seed)
        m = int(np.ceil((rho * box ** 3) ** (1 / 3)))
        g = np.stack(np.meshgrid(*(np.arange(m),) * 3, indexing="ij"), -1).reshape(-1, 3)
        pos4 = np.zeros((m ** 3, 4), np.float32)
        pos4[:, :3] = (g + 0.5) * (box / m) + rng.uniform(-0.06, 0.06, (m ** 3, 3))
        vel4 = np.zeros_like(pos4)
        vel4[:, :3] = sign * 0.9 * 0.5 * (side - 2.5) / dt / np.sqrt(3.0)
        path = [orc.run(p, pos4, vel4, k)[:2] for k in (1, 2, 3)]
        if all(_clear_of_cutoff(x, box) for x, _ in path) and _clear_of_cutoff(pos4[:, :3].astype(np.float64), box):
            break
    _say(f"outside cells nc={nc} side={side} sign={sign} n={len(pos4)}")
    s = _system(len(pos4), box, dt=dt, cell_min=0.999 * side, shift_mode=1)
    assert s.cells_per_dim == nc
    s.load(_dev(pos4), _dev(vel4))
    s.step_every(3, 3)
    _, vel = s.state()
    assert s.check() == 0
    assert np.abs(vel.cpu().numpy()[:, :3] - path[2][1]).max() < 3e-5
