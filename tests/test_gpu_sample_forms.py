"""The sampler's two forms at their edges: one launch up to 16384 amplitudes, prefix sums of groups of 8, 16 or 64 beyond,
every storage type, states whose probability sits in few places (first and last amplitude of a group, of a block and
of the state, long runs of zeros) and states spread evenly.  Indices are integers defined by the state's bits alone, so
they must equal the oracle's on the same state."""
from __future__ import annotations

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2005_04635_amd as pkg

    pkg.load()
    return pkg


def sparse(n):
    N = 1 << n
    psi = np.zeros(N, dtype=np.complex128)
    for i in (0, 15, 16, 31, 4095, 4096, 8191, 8192, 12287, N // 2 - 1, N - 1):
        psi[i % N] += 0.25 + 0.125 * (i % 3)
    return psi / np.sqrt(np.sum(np.abs(psi) ** 2))


@pytest.mark.parametrize("dtype", ["f64", "c64", "c128", "cbf16"])
@pytest.mark.parametrize("n", [2, 4, 7, 10, 13, 14, 15, 16, 19, 25])
@pytest.mark.parametrize("kind", ["sparse", "random"])
def test_sampler_forms(G, orc, n, dtype, kind):
    print(f"sampler n={n} {dtype} {kind}", flush=True)
    psi = sparse(n) if kind == "sparse" else workloads.random_state(n, seed=60 + n)
    if dtype == "f64":
        psi = np.abs(psi)
    g = G.Grover(n, dtype, marks=[], form="fused").write_state(psi)
    state = g.read_state().astype(np.complex128)
    for shots in (1, 3000):
        u = workloads.uniforms_u53(5 + shots, shots)
        u[0] = (1 << 53) - 1
        assert np.array_equal(g.sample(shots, u53=u), orc.sample(state, u)), shots
    seeded = g.sample(500, seed=77)
    assert np.array_equal(seeded, orc.sample(state, workloads.uniforms_u53(77, 500)))
    g.close()
