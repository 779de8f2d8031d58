"""The blocked Walsh-Hadamard passes on small states: every n up to 15, where the one-wave kernel, the number of layouts
and the number of groups change, against the n-fold product in numpy; and the memory around a state, which the one-wave
kernel reaches through a buffer of the state's size.

Bound: every stage is unitary up to a power of two and rounds each amplitude once, so it adds at most 2^-53 of the norm;
storing in complex64 adds 2^-24 of it per pass.  k iterations have 2kn stages and at most 4k + 1 passes, and the
reference makes the same binary64 errors."""
from __future__ import annotations

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


def transform(x, n):
    for q in range(n):
        v = x.reshape(-1, 2, 1 << q)
        x = np.concatenate([v[:, :1] + v[:, 1:], v[:, :1] - v[:, 1:]], axis=1).reshape(-1)
    return x


@pytest.mark.parametrize("dtype", ["f64", "c64", "c128"])
@pytest.mark.parametrize("n", range(1, 16))
def test_small_states(n, dtype):
    import torch

    import paper_2005_04635_amd as pkg

    N, k, guard = 1 << n, 3, 512
    marks = sorted({0, N // 2, N - 1})
    psi = workloads.random_state(n, seed=80 + n, real=dtype == "f64")
    tdt = {"f64": torch.float64, "c64": torch.complex64, "c128": torch.complex128}[dtype]
    x = torch.from_numpy(psi.real.copy() if dtype == "f64" else psi).to("cuda").to(tdt)
    start = x.cpu().numpy().astype(np.complex128)
    whole = torch.full((N + 2 * guard,), 3.0, dtype=tdt, device="cuda")
    state = whole[guard:guard + N]
    g = pkg.Grover(n, dtype, marks=marks, state=state)
    eps = 2.0 ** -24 if dtype == "c64" else 2.0 ** -53
    state.copy_(x)
    g.hadamard_all(blocked=True)
    want = transform(start, n) * 2.0 ** (-n / 2)
    assert np.linalg.norm(state.cpu().numpy() - want) <= 3 * eps + 2 * (n + 4) * 2.0 ** -53
    state.copy_(x)
    g.gate_iterate_blocked(k)
    want = start.copy()
    for _ in range(k):
        want[marks] *= -1
        want = transform(want, n)
        want[1:] *= -1
        want = transform(want, n) / N
    assert np.linalg.norm(state.cpu().numpy() - want) <= (4 * k + 1) * eps + 2 * (2 * k * n + 4 * k + 2) * 2.0 ** -53
    g.close()
    assert bool((whole[:guard] == 3.0).all()) and bool((whole[guard + N:] == 3.0).all())
