"""The sampler's probabilities as integers over their whole range: q = floor(p 2^62) for p in [1, 2) and [2, 4) (states of
total below 4 need not be normalised), for p around 2^-62, where q is 0, 1 or 2, and for subnormal p.  The group sums and
the search within a group convert the bits on their own and must agree, and both with the oracle, exactly.  Totals of 4 and more do not
fit the integers: the indices are then unspecified, but lie in the state."""
from __future__ import annotations

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

DTYPES = ["f64", "c64", "c128", "cbf16"]
SIZES = [10, 14, 15, 17, 25]


@pytest.fixture(scope="module")
def G():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2005_04635_amd as pkg

    pkg.load()
    return pkg


def state_of(n, dtype, values):
    """Zeros but for `values` at scattered places, two of them neighbours in a group."""
    N = 1 << n
    psi = np.zeros(N, dtype=np.complex128)
    at = sorted({i % N for i in (3, 4, 77, 1023, N // 2 - 1, N // 2, N - 5, N - 1)})
    for i, v in zip(at, (values * len(at))[: len(at)]):
        psi[i] = v
    return psi.real.copy() if dtype == "f64" else psi


def shots_of(shots, total_ends=True):
    u = workloads.uniforms_u53(9, shots)
    if total_ends:
        u[0], u[1] = 0, (1 << 53) - 1
    return u


LARGE = {"one to two": [1.25, 0.25], "two to four": [1.5625, 0.125], "just below two": [np.sqrt(3.9375 / 2), 0.0]}


@pytest.mark.parametrize("kind", list(LARGE))
@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("n", SIZES)
def test_large_probabilities(G, orc, n, dtype, kind):
    print(f"sampler n={n} {dtype} {kind}", flush=True)
    a, b = LARGE[kind]
    psi = state_of(n, dtype, [0.0])
    psi[(1 << n) // 2 + 1] = a if dtype == "f64" else a * (1.0 if kind != "just below two" else (0.8 + 0.6j))
    psi[3] = b
    g = G.Grover(n, dtype, marks=[], form="fused").write_state(psi)
    state = g.read_state().astype(np.complex128)
    assert float(np.sum(np.abs(state) ** 2)) < 4.0
    u = shots_of(3000)
    assert np.array_equal(g.sample(3000, u53=u), orc.sample(state, u))
    g.close()


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("n", SIZES)
def test_tiny_probabilities(G, orc, n, dtype):
    print(f"sampler n={n} {dtype} tiny", flush=True)
    # p = 2^-62 (q = 1), just below it (0), 2^-61 (2), 2^-64 (0) and, where the storage has it, subnormal p
    values = [2.0 ** -31, 2.0 ** -31 * (1 - 2.0 ** -8), 2.0 ** -30.5, 2.0 ** -32] + ([1e-160] if dtype in ("f64", "c128") else [])
    psi = state_of(n, dtype, values)
    g = G.Grover(n, dtype, marks=[], form="fused").write_state(psi)
    state = g.read_state().astype(np.complex128)
    u = shots_of(2000)
    want = orc.sample(state, u)
    assert len(set(want.tolist())) > 1
    assert np.array_equal(g.sample(2000, u53=u), want)
    g.close()


@pytest.mark.parametrize("value", [2.0, 3.0, 1e30, float("inf"), float("nan")])
@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("n", [10, 15, 25])
def test_beyond_the_integers(G, n, dtype, value):
    print(f"sampler n={n} {dtype} value {value}", flush=True)
    psi = state_of(n, dtype, [0.25, 0.125])
    psi[(1 << n) // 2 + 2] = value
    g = G.Grover(n, dtype, marks=[], form="fused").write_state(psi)
    try:
        shots = g.sample(500, u53=shots_of(500))
        assert int(shots.max()) < 1 << n
    except G.GroverError as e:  # the total may come out as zero
        assert e.status == -1
    g.reset()
    assert int(g.sample(500, u53=shots_of(500)).max()) < 1 << n
    g.close()
