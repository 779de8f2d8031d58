"""One iteration on complex bfloat16 storage against its definition: every part of c' is 2S/N - s c in binary64, rounded
once to bfloat16.  The states are such that S is exact in binary64 in any order, and that many parts of c' lie halfway
between two bfloat16 up to a distance that binary32 drops, so rounding through binary32 alone would give another value.
Bit for bit."""
from __future__ import annotations

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def round_bf16(d):
    """binary64 -> the nearest bfloat16 (ties to even), as binary64; normal range only."""
    u = np.ascontiguousarray(d).view(np.uint64)
    half = np.uint64(1 << 44)  # binary64 keeps 52 bits, bfloat16 7
    odd = (u >> np.uint64(45)) & np.uint64(1)
    return (((u + half - np.uint64(1) + odd) >> np.uint64(45)) << np.uint64(45)).view(np.float64)


def part(rng, N, m_times_half_n):
    """N bfloat16 values, multiples of 2^-7 but for the last 24, whose sum is exactly the given one."""
    c = rng.integers(-128, 129, N) / 128.0
    c[-24:] = 0.0
    rest = m_times_half_n - c.sum()
    for i in range(24):
        c[N - 24 + i] = 0.0 if rest == 0.0 else (np.array([rest]).view(np.uint64) >> np.uint64(45) << np.uint64(45)).view(np.float64)[0]
        rest -= c[N - 24 + i]
    assert rest == 0.0
    return c


@pytest.mark.parametrize("tiny", [2.0 ** -30, -(2.0 ** -30), 0.0])
@pytest.mark.parametrize("n", [6, 12, 15])
def test_one_rounding(n, tiny):
    import torch

    import paper_2005_04635_amd as pkg

    N, rng = 1 << n, np.random.default_rng(n)
    mean2 = 1.0 + 2.0 ** -8 + tiny  # of 2^-7-spaced values from it, those between 1 and 2 end halfway
    marks = [3, N // 2, N // 2 + 1]
    sign = np.ones(N)
    sign[marks] = -1.0
    flipped = [part(rng, N, mean2 * N / 2), part(rng, N, -mean2 * N / 2)]
    c = [sign * p for p in flipped]
    want = [round_bf16(m - p) for m, p in zip((mean2, -mean2), flipped)]
    state = np.stack(c, axis=1).astype(np.float32)  # exact
    g = pkg.Grover(n, "cbf16", marks=marks, form="fused")
    g.write_state((state[:, 0] + 1j * state[:, 1]).astype(np.complex64))
    g.iterate(1)
    got = np.asarray(g.read_state())
    g.close()
    assert np.array_equal(got.real.astype(np.float64), want[0]) and np.array_equal(got.imag.astype(np.float64), want[1])
    if tiny:
        through = [round_bf16((m - p).astype(np.float32).astype(np.float64)) for m, p in zip((mean2, -mean2), flipped)]
        assert any(np.count_nonzero(a != b) > N // 16 for a, b in zip(through, want))
