"""The staged spring kernels (k_spring_block) where a length or a position is not finite, and the
accuracy of their square root and quotient.

A spring of infinite rest length pulls without bound along its direction, as the quotient of the
library's division does; a vertex that no edge leaves has no force wherever it is."""
import math
from fractions import Fraction

import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_1506_07577_amd import ebbx
else:  # collected on a CPU host only to be deselected
    ebbx = None


def _ring(nv, reach=6):
    """Vertex i with the `reach` after it, cyclically, in both directions."""
    X = np.random.default_rng(1).uniform(0.0, 1.0, (nv, 3))
    i = np.arange(nv)
    pairs = [(i, (i + k) % nv) for k in range(1, reach + 1)]
    tail = np.concatenate([a for a, b in pairs] + [b for a, b in pairs])
    head = np.concatenate([b for a, b in pairs] + [a for a, b in pairs])
    return X, tail.astype(np.int32), head.astype(np.int32)


def _same(got, want):
    """Equal where not finite, 1e-12 normwise elsewhere (sums in another order)."""
    fin = np.isfinite(want)
    assert np.array_equal(got[~fin], want[~fin], equal_nan=True)
    assert np.abs(got[fin] - want[fin]).max() <= 1e-12 * max(np.abs(want[fin]).max(), 1.0)


def test_infinite_rest_length():
    X, tail, head = _ring(321)
    q = X + 0.01 * np.random.default_rng(2).uniform(-1, 1, X.shape)
    X = X.copy()
    X[100] = 1e200   # |X_h - X_v| overflows for its springs
    with np.errstate(all="ignore"):
        want = oracle.Springs(X, tail, head, np.ones(len(X)), 0.5).forces(q)
    assert np.isinf(want).any()
    sm = ebbx.SpringMesh(X, tail, head, 0.5)
    _same(sm.from_dev(sm.springs.forces(sm.to_dev(q))), want)


@pytest.mark.parametrize("value", [np.inf, np.nan])
@pytest.mark.parametrize("nv", [321, 70001])   # four and two lanes per vertex
def test_vertex_without_edges_at_no_finite_position(nv, value):
    X, tail, head = _ring(nv)
    lone = 200
    keep = (tail != lone) & (head != lone)
    tail, head = tail[keep], head[keep]
    q = X + 0.01 * np.random.default_rng(2).uniform(-1, 1, X.shape)
    q[lone] = value
    want = oracle.Springs(X, tail, head, np.ones(nv), 0.5).forces(q)
    assert not want[lone].any() and np.isfinite(want).all()
    sm = ebbx.SpringMesh(X, tail, head, 0.5)
    got = sm.from_dev(sm.springs.forces(sm.to_dev(q)))
    assert not got[lone].any()
    _same(got, want)
    # one step leaves its velocity as it is
    v0 = np.random.default_rng(3).uniform(-1, 1, X.shape)
    a, b = sm.to_dev(q), sm.to_dev(v0)
    sm.springs.run(sm.scalar_to_dev(np.ones(nv)), 1e-4, 2, a, b, torch.zeros_like(a))
    assert np.array_equal(sm.from_dev(b)[lone], v0[lone])


def _root(n2, bits=80):
    """sqrt(n2) as a fraction, to 2^-80."""
    return Fraction(math.isqrt(n2 << (2 * bits)), 1 << bits)


@pytest.mark.parametrize("exp2", [0, 100, -200, 440, -490])
def test_scale_of_a_spring(exp2):
    """len / sqrt(n2) of k_spring_block to one ulp.  Vertices in pairs, each with four springs to the
    other (so that the staged kernel takes them), by integer steps times a power of two: n2 is exact
    however it is contracted, the four forces add up exactly, and a - s a tells s to its last bits since
    s >= 1.  440 and -490: n2 on both sides of 1e280 and of 1e-280, the ends of the range of the kernel's
    own root."""
    rng = np.random.default_rng(40)
    nv = 4096
    step = rng.integers(1, 1 << 25, (nv // 2, 3)).astype(np.float64)
    rest = step * (1.0 + rng.uniform(0.0, 3.0, (nv // 2, 1)))
    unit = 2.0 ** exp2
    X, q = np.zeros((nv, 3)), np.zeros((nv, 3))
    X[1::2], q[1::2] = rest * unit, step * unit
    tail = np.repeat(np.arange(nv, dtype=np.int32), 4)
    sm = ebbx.SpringMesh(X, tail, tail ^ 1, 1.0)
    got = sm.from_dev(sm.springs.forces(sm.to_dev(q)))[0::2] / 4.0 / unit
    length = sm.springs.rest().cpu().numpy()[0::8] / unit
    n2 = ((step * unit) ** 2).sum(axis=1)
    if exp2 in (440, -490):
        edge = 1e280 if exp2 > 0 else 1e-280
        assert (n2 < edge).any() and (n2 > edge).any()
    worst = 0.0
    for a, f, ln in zip(step, got, length):
        s = Fraction(ln) / _root(sum(int(x) ** 2 for x in a))
        for x, y in zip(a, f):
            exact = Fraction(x) - s * Fraction(x)
            # one ulp of s, times x, and the rounding of the difference
            room = Fraction(np.spacing(float(s))) * Fraction(x) + Fraction(np.spacing(abs(y)))
            worst = max(worst, float(abs(Fraction(y) - exact) / room))
    assert worst <= 1.0
