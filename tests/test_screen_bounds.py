"""The 16-bit screen's bound on the host against the rounding that it has to
cover: a search for the pairs that rounding pushes out furthest.
"""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
RC = 2.5


@pytest.fixture(scope="module")
def bound(tmp_path_factory):
    d = tmp_path_factory.mktemp("bound")
    (d / "b.cpp").write_text('#include "screen_bounds.h"\n'
                             'extern "C" float bound16(double r, double s) '
                             "{ return mdlj::screen16_bound(r, s); }\n")
    csrc = os.path.join(ROOT, "paper_0709_3225_amd", "csrc")
    subprocess.run(["g++", "-O2", "-shared", "-fPIC", "-I", csrc, str(d / "b.cpp"), "-o", str(d / "b.so")], check=True)
    f = ctypes.CDLL(str(d / "b.so")).bound16
    f.restype, f.argtypes = ctypes.c_float, [ctypes.c_double] * 2
    return f


def _excess(xi, xj, s):
    """What the screen's value exceeds r^2 / s^2 by: operands rounded as the
    kernel rounds them (32-bit scaling, 16-bit operands), summed exactly."""
    f32, f16 = np.float32, np.float16
    inv = f32(1.0) / f32(s)
    xi, xj = xi.astype(f32), xj.astype(f32)
    v = xi * inv
    b = (f32(-2.0) * v).astype(f16).astype(np.float64)
    u = (xj.astype(np.float64) * inv - 0.5).astype(f32).astype(f16).astype(np.float64)
    w = ((xj * xj).sum(-1, dtype=f32) * (inv * inv)).astype(f16).astype(np.float64)
    c = ((v * v).sum(-1, dtype=f32) - v.sum(-1, dtype=f32)).astype(np.float64)
    d = xi.astype(np.float64) - xj
    return (b * u).sum(-1) + w + c - (d * d).sum(-1) / s ** 2


def _worst(s, r, d, rng):
    """The largest excess over pairs at distance r with the home atom within
    d s of its cell: random pairs, the best of them moved about."""
    def place(p):
        xi = np.clip(p[:, :3], -d, 1 + d) * s
        e = p[:, 3:] / np.linalg.norm(p[:, 3:], axis=1, keepdims=True)
        return xi, xi + r * e

    p = np.concatenate([rng.uniform(-d, 1 + d, (400000, 3)), rng.normal(size=(400000, 3))], 1)
    # near the far corner all three axes round coarsest
    p[:200000, :3] = (1 + d) - rng.exponential(0.1, (200000, 3)) * np.where(rng.random((200000, 3)) < 0.8, 1, 5)
    p[:200000, 3:] = np.abs(p[:200000, 3:])
    x = _excess(*place(p), s)
    p = np.repeat(p[np.argsort(x)[-400:]], 20, 0)
    best = _excess(*place(p), s)
    for k in range(120):
        q = p + rng.normal(size=p.shape) * 10.0 ** rng.uniform(-4, -1.5, (len(p), 1))
        y = _excess(*place(q), s)
        p[y > best] = q[y > best]
        best = np.maximum(best, y)
    return best.max()


@pytest.mark.parametrize("d", [0.0, 0.02, 0.05, 0.1, 0.17, 0.25, 0.33, 0.41, 0.49])
def test_margin_covers_the_rounding(d, bound):
    """Sides from r_c to 50 r_c, atoms as far out of their cells as a run may
    leave them, pairs at the cutoff: no pair needs more than the margin, and the
    pairs found need more than half of it (so the search would notice a margin
    cut to that)."""
    s = RC / (1 - 2 * d)
    margin = bound(RC, s) - (RC / s) ** 2
    worst = _worst(s, RC, d, np.random.default_rng(int(d * 1e4)))
    assert worst < margin
    assert worst > margin / 2


@pytest.mark.parametrize("d", [0.0, 0.03, 0.15, 0.3])
def test_margin_covers_the_list_radius(d, bound):
    """Words that are kept take the cell side as their radius, right after a
    rebuild (atoms in their cells)."""
    s = RC / (1 - 2 * d)
    margin = bound(s, s) - 1.0
    assert _worst(s, s, 0.0, np.random.default_rng(7 + int(d * 1e4))) < margin
