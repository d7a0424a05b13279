"""The library's Gauss-Hermite nodes and weights for every kind of node count (CPU): those compiled
into the solver come from a table, all others from sign counts and Newton steps.

The reference is the same recurrence in 45 decimal digits, refined by Newton's method from the
library's nodes: a wrong or repeated node would give a repeated root or a broken order.  Nodes are
rounded from a Newton step whose last correction carries the rounding of h_Q over its slope, a few
units in the last place at the outer nodes; weights lose the digits that the recurrence loses, about
Q of them in units of 1e-16."""
from decimal import Decimal, getcontext

import numpy as np
import pytest

import paper_2211_16933_amd as elb

TABLE = [8, 12, 16, 20, 24, 32, 40, 48, 64, 96, 200]


def _reference(q, start):
    """Nodes x > 0 (or = 0) and weights from the given starting nodes, in 45 digits."""
    getcontext().prec = 45
    root = [Decimal(k).sqrt() for k in range(q + 1)]
    nodes, weights = [], []
    for x in (Decimal(float(v)) for v in start):
        for _ in range(4):
            a, b = Decimal(0), Decimal(1)       # h_{l-1}, h_l at l = 0
            total = Decimal(0)
            for l in range(q):
                total += b * b
                a, b = b, (x * b - root[l] * a) / root[l + 1]
            x -= b / (root[q] * a)
        nodes.append(x)
        weights.append(1 / total)
    return nodes, weights


@pytest.mark.parametrize("q", [1, 2, 3, 4, 5, 7, 9, 11, 31, 33, 97, 128, 199, 255, 256] + TABLE)
def test_nodes_and_weights(q):
    p, w = elb.quadrature(q)
    assert np.all(np.diff(p) > 0) and np.array_equal(p, -p[::-1]) and np.array_equal(w, w[::-1])
    if q % 2:
        assert p[q // 2] == 0.0
    nodes, weights = _reference(q, p[q // 2:])
    assert all(a < b for a, b in zip(nodes, nodes[1:]))     # q distinct roots of h_q: all of them
    ulp = np.spacing(np.maximum(p[q // 2:], 2.0 ** -2))
    assert max(abs(float(Decimal(float(a)) - b)) / u for a, b, u in zip(p[q // 2:], nodes, ulp)) <= 4.0
    assert max(abs(float(Decimal(float(a)) / b - 1)) for a, b in zip(w[q // 2:], weights)) <= (2 * q + 4) * 2.3e-16
    # moments of exp(-p^2/2) / sqrt(2 pi): 1, 0, 1, 0, 3, as far as q nodes are exact
    for power, want in ((0, 1.0), (2, 1.0), (4, 3.0), (6, 15.0)):
        if power < 2 * q:
            assert abs(np.sum(w * p ** power) - want) <= 4e-14 * want


@pytest.mark.parametrize("q", [0, -1, 257])
def test_other_counts_are_refused(q):
    buf = np.zeros(300)
    import ctypes
    ptr = buf.ctypes.data_as(ctypes.POINTER(ctypes.c_double))
    assert elb.lib().elb_quadrature(q, ptr, ptr) == elb.ELB_EINVAL and not buf.any()
