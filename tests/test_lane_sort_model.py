"""The lane kernel's sorting network, step by step on the host: position i sits
in lane i % 64 of register i / 64, and every step compares a position with
i ^ m (m one bit, or all bits below a power of two), the larger value going to
the lower position."""
import numpy as np
import pytest


def steps(n):
    """The masks in the kernel's order: the mirrored half, then distances K/4 .. 1."""
    k = 2
    while k <= n:
        yield k - 1
        d = k // 4
        while d >= 1:
            yield d
            d //= 2
        k *= 2


def lane_xor_patterns(m):
    """The lane moves that lane i ^ m is composed of."""
    return {4: (7, 3), 8: (15, 7)}.get(m, (m,))


@pytest.mark.parametrize("regs", [1, 2, 4, 8])
def test_network_sorts(regs):
    n = 64 * regs
    i = np.arange(n)
    rng = np.random.Generator(np.random.PCG64(regs))
    for trial in range(200):
        kinds = rng.integers(2, 6 if trial % 2 else 1000)
        a = rng.integers(0, kinds, n)
        a[rng.random(n) < rng.random()] = 0        # empty positions, which sort last
        if trial % 5 == 0:                         # nearly in order
            a = np.sort(a)[::-1].copy()
            j = rng.integers(0, n, 4)
            a[j[:2]] = a[j[2:]]
        want = np.sort(a)[::-1]
        for m in steps(n):
            o = a[i ^ m]
            low = (i & (1 << (int(m).bit_length() - 1))) == 0
            a = np.where(low, np.maximum(a, o), np.minimum(a, o))
        assert np.array_equal(a, want)


def test_lane_moves_compose():
    lane = np.arange(64)
    for m in sorted(set(m for m in steps(64))):
        v = lane
        for p in lane_xor_patterns(m):
            v = v[lane ^ p]
        assert np.array_equal(v, lane ^ m), m
