"""The blocked Walsh-Hadamard passes in three groups with tiles of 2^12 (segments of 32 and of 8 amplitudes), 2^13 and
2^14, on the states that are split so: complex64 n = 26, 30, 31 (16 GiB) and 34 (128 GiB), complex128 n = 33, all on the
device and in place, a chunk at a time.

A basis state has the transform 2^(-n/2) (-1)^popcount(i & j).  Its unnormalised butterflies add zeros and units, which is
exact, so only the scale of an odd n rounds: 2^-22 of the amplitude.  The second transform adds 2^n values of one
magnitude that cancel or add up, exact up to that rounding in each.  Two iterations from the uniform state keep two
values; they round once per pass, at most 4k + 1 of them, so the state is off by at most (4k + 1) 2^-24 of its norm, and
2 (2kn + 4k + 2) 2^-53 for the binary64 steps."""
from __future__ import annotations

import math

import pytest

pytestmark = pytest.mark.gpu

CHUNK = 1 << 24


def signs(torch, j, bits):
    """(-1)^popcount(i & j) for i < 2^bits."""
    s = torch.ones(1, dtype=torch.float32, device="cuda")
    for q in range(bits):
        s = torch.cat([s, -s if (j >> q) & 1 else s])
    return s


@pytest.mark.parametrize("n,dtype", [(26, "c64"), (30, "c64"), (31, "c64"), (33, "c128"), (34, "c64")])
def test_three_groups(n, dtype):
    import torch

    import paper_2005_04635_amd as pkg

    need = (16 if dtype == "c128" else 8) << n
    if torch.cuda.get_device_properties(0).total_memory < need + (8 << 30):
        pytest.skip(f"needs {need >> 30} GiB of device memory")
    print(f"three groups n={n} {dtype}", flush=True)
    N, j = 1 << n, 0x2B5A7C3D1 % (1 << n)
    torch.cuda.empty_cache()
    g = pkg.Grover(n, dtype, marks=[1, N - 1])
    g.state.zero_()
    g.state[j] = 1.0
    low, scale = signs(torch, j, 24), 2.0 ** (-n / 2)
    g.hadamard_all(blocked=True)
    for c in range(0, N, CHUNK):
        s = -1.0 if bin((c & j) >> 24).count("1") % 2 else 1.0
        x = g.state[c:c + CHUNK]
        assert float((x.real - low * (s * scale)).abs().max()) <= (scale * 2.0 ** -22 if n % 2 else 0.0)
        assert float(x.imag.abs().max()) == 0.0
    g.hadamard_all(blocked=True)
    g.state[j] -= 1.0
    worst = max(float(torch.view_as_real(g.state[c:c + CHUNK]).abs().max()) for c in range(0, N, CHUNK))
    assert worst <= (2.0 ** -22 if n % 2 else 0.0)
    k = 2
    g.reset().gate_iterate_blocked(k)
    angle = math.asin(math.sqrt(2.0 / N))
    a, u = math.sin((2 * k + 1) * angle) / math.sqrt(2.0), math.cos((2 * k + 1) * angle) / math.sqrt(N - 2.0)
    off = sum((complex(g.state[i]).real - a) ** 2 + complex(g.state[i]).imag ** 2 for i in (1, N - 1))
    g.state[1] = u
    g.state[N - 1] = u
    for c in range(0, N, CHUNK):
        x = g.state[c:c + CHUNK]
        off += float((x.real.double() - u).square().sum() + x.imag.double().square().sum())
    eps = 2.0 ** -24 if dtype == "c64" else 2.0 ** -53
    g.close()
    del g
    torch.cuda.empty_cache()
    assert math.sqrt(off) <= (4 * k + 1) * eps + 2 * (2 * k * n + 4 * k + 2) * 2.0 ** -53
