"""Calls that follow one another on one workspace: what a call leaves behind for
the next one's cell builds.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _say(msg):
    print(f"[case] {msg}", flush=True)


@pytest.mark.parametrize("nc", [5, 33])
def test_calls_of_any_length_continue_each_other(nc):
    """A build counts atoms past a cell's bucket and (on grids up to 32^3) blocks
    of cells in one of two sets of counters in turn; calls of odd and even
    length leave one or the other set behind, a load the second. Steps of 2, 1,
    2, 3, 4 and 1 after a load, and calls with rebuilds every two steps among
    them, with 700 atoms in one cell (its bucket holds far fewer) and cells of 0
    to 9 around it, on both sides of 32^3 cells: after each call the cells are
    those of a counting sort, and the state is bit for bit that of one call."""
    import torch

    from paper_0709_3225_amd import LJSystem

    side, rng = 2.6, np.random.default_rng(nc)
    cells = np.stack(np.meshgrid(*(np.arange(nc),) * 3, indexing="ij"), -1).reshape(-1, 3)
    mid = np.flatnonzero((cells == nc // 2).all(1))[0]
    per = rng.integers(0, 10, nc ** 3)
    per[mid] = 700

    def sites(m):  # of m^3 in a cell, clear of its faces
        u = 0.15 + (np.arange(m) + 0.5) * (side - 0.3) / m
        return np.stack(np.meshgrid(u, u, u, indexing="ij"), -1).reshape(-1, 3)

    few, many = sites(3), sites(9)
    pts = [cells[c] * side + (many if c == mid else few)[rng.permutation(729 if c == mid else 27)[:per[c]]]
           for c in range(nc ** 3)]
    pos4 = np.zeros((per.sum(), 4), np.float32)
    pos4[:, :3] = np.concatenate(pts)
    perm = rng.permutation(len(pos4))
    pos4 = pos4[perm]
    c = np.repeat([a + nc * (b + nc * e) for a, b, e in cells], per)[perm]
    want_start = np.concatenate([[0], np.cumsum(np.bincount(c, minlength=nc ** 3))])
    want_order = np.lexsort((np.arange(len(c)), c))
    vel4 = np.zeros_like(pos4)
    vel4[:, :3] = rng.normal(size=(len(pos4), 3))
    x, v = torch.from_numpy(pos4).cuda(), torch.from_numpy(vel4).cuda()
    _say(f"calls nc={nc} n={len(pos4)}")

    def system():
        # (a step moves no atom by as much as the distance to its cell's face)
        s = LJSystem(len(pos4), nc * side, cell_min=0.999 * side, dt=1e-7, epsilon=1e-6)
        assert s.cells_per_dim == nc
        s.load(x, v)
        return s

    def cells_ok(s, what):
        start, order = s.cell_lists()
        assert s.check() == 0, what
        assert np.array_equal(start.cpu().numpy(), want_start), what
        assert np.array_equal(order.cpu().numpy(), want_order), what

    one = system()
    one.step(13)
    s = system()
    for n in (2, 1, 2, 3, 4, 1):
        s.step(n)
        cells_ok(s, n)
    for a, b in zip(s.state(), one.state()):
        assert torch.equal(a, b)
    for call in (lambda: s.step_every(4, 2), lambda: s.step(2), lambda: s.step_every(5, 2), lambda: s.step(3),
                 lambda: s.step_every(1, 2), lambda: s.step(4)):
        call()
        cells_ok(s, "mixed")
    s.load(x, v)
    s.step(13)
    for a, b in zip(s.state(), one.state()):
        assert torch.equal(a, b)
