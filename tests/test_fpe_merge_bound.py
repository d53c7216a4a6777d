"""CPU test of the rule that lets a wavefront skip the merge of its lanes'
expansions (wave_fpe_merge_is_exact): wherever the rule holds, the merge tree
leaves no remainder, so skipping it changes neither the sum nor the escapes."""

import numpy as np
import pytest


def two_sum(a, b):
    r = a + b
    z = r - a
    return r, (a - (r - z)) + (b - z)


def accumulate(a, x):
    """Alg. 4 on arrays: a is a list of P arrays; returns the remainder."""
    for i in range(len(a)):
        a[i], x = two_sum(a[i], x)
    return x


def merge_remainders(a):
    """wave_fpe_merge of [P, 64]: number of nonzero remainders."""
    a = [v.copy() for v in a]
    esc = 0
    off = 32
    while off:
        b = [v[off:2 * off].copy() for v in a]
        c = [v[:off].copy() for v in a]
        for q in b:
            esc += int(np.count_nonzero(accumulate(c, q)))
        for i in range(len(a)):
            a[i][:off] = c[i]
        off //= 2
    return esc


def rule(a):
    e, lsb, top = [], 1 << 20, -(1 << 20)
    for v in a:
        ei = -(1 << 20)
        for x in v[v != 0.0]:
            m, ex = np.frexp(abs(x))
            ei = max(ei, int(ex) - 1)
            k = int(np.ldexp(m, 53))
            lsb = min(lsb, int(ex) - 53 + (k & -k).bit_length() - 1)
        e.append(ei)
        top = max(top, ei)
    p = top + 12 - 53
    for i in range(1, len(a)):
        p = max(e[i] + 1, p + 7) + 1 - 53
    return p < lsb


def lanes(rng, P, spread, nadd, bits):
    """Expansions as lanes have them after nadd accumulated products, or raw components."""
    a = [np.zeros(64) for _ in range(P)]
    for _ in range(nadd):
        x = np.ldexp(np.rint(np.ldexp(rng.random(64) + 0.5, bits)) / 2.0 ** bits, rng.integers(-spread, 1, 64)) * rng.choice([-1.0, 1.0], 64)
        accumulate(a, x)
    return a


@pytest.mark.parametrize("P", [1, 2, 3, 4, 8])
def test_rule_implies_no_remainder(P):
    rng = np.random.default_rng(P)
    held = 0
    for spread in (0, 3, 20, 40, 53, 80, 110, 160, 300):
        for bits in (4, 20, 52):
            for nadd in (1, 3, 9):
                a = lanes(rng, P, spread, nadd, bits)
                if rng.random() < 0.3:  # components of any size at any level
                    a = [np.ldexp(v, int(rng.integers(-10, 11))) for v in a]
                if rule(a):
                    held += 1
                    assert merge_remainders(a) == 0, (P, spread, bits, nadd)
    assert held > 5  # the rule is met by ordinary data


def test_rule_fails_where_remainders_occur():
    rng = np.random.default_rng(9)
    a = lanes(rng, 1, 60, 1, 52)
    assert merge_remainders(a) > 0 and not rule(a)
