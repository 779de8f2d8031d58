"""The blocked Walsh-Hadamard passes at the edges of their splits of the qubits (one group; a low and a high one with
short and long segments; three groups; tiles of 2^11 .. 2^14, more tiles than workgroups), against binary64 butterflies
in plain PyTorch.

Bound: every stage is unitary up to a power of two and rounds each amplitude once, so it adds at most 2^-53 of the norm;
storing in complex64 adds 2^-24 of it per pass.  k iterations have 2kn stages and at most 4k + 1 passes, and the
reference makes the same binary64 errors.
"""
from __future__ import annotations

import pytest

pytestmark = pytest.mark.gpu

CASES = [(n, "c64") for n in (1, 4, 10, 11, 12, 13, 14, 18, 19, 21, 23, 25, 26)]
CASES += [(n, "c128") for n in (2, 11, 13, 14, 19, 22, 24, 26, 27)] + [(n, "f64") for n in (3, 12, 13, 15, 20, 23, 25, 26)]


def transform(torch, x, n):
    """Unnormalised butterflies of all qubits, in place."""
    for q in range(n):
        v = x.view(-1, 2, 1 << q)
        d = v[:, 0] - v[:, 1]
        v[:, 0] += v[:, 1]
        v[:, 1] = d


@pytest.mark.parametrize("marked", ["none", "few", "many"])
@pytest.mark.parametrize("n,dtype", CASES)
def test_gate_iterations_and_transform(n, dtype, marked):
    import torch

    import paper_2005_04635_amd as pkg

    N, k = 1 << n, 2
    many = min(N // 2, 9000)  # above the length that a workgroup reads through for each tile of 2^14
    marks = {"none": [], "few": sorted({0, N // 2, N - 1}), "many": list(range(N // 2, N // 2 + many))}[marked]
    gen = torch.Generator(device="cuda").manual_seed(n)
    real = torch.float64 if dtype != "c64" else torch.float32
    x = torch.randn(N, generator=gen, device="cuda", dtype=real)
    if dtype != "f64":
        x = torch.complex(x, torch.randn(N, generator=gen, device="cuda", dtype=real))
    x /= torch.linalg.vector_norm(x)
    start = x.to(torch.float64 if dtype == "f64" else torch.complex128)
    eps = 2.0 ** -24 if dtype == "c64" else 2.0 ** -53

    def distance(got, want):
        return float(torch.linalg.vector_norm(torch.view_as_real(got.to(want.dtype) - want).flatten()
                                              if dtype != "f64" else got - want))

    g = pkg.Grover(n, dtype, marks=marks)
    want = start.clone()
    for _ in range(k):
        want[torch.tensor(marks, dtype=torch.int64, device="cuda")] *= -1
        transform(torch, want, n)
        want[1:] *= -1
        transform(torch, want, n)
        want /= N
    g.state.copy_(x)
    g.gate_iterate_blocked(k)
    norm = float(torch.linalg.vector_norm(x.to(start.dtype)))
    assert distance(g.state, want) <= norm * ((4 * k + 1) * eps + 2 * (2 * k * n + 4 * k + 2) * 2.0 ** -53)
    want = start.clone()
    transform(torch, want, n)
    want *= 2.0 ** (-n / 2)
    g.state.copy_(x)
    g.hadamard_all(blocked=True)
    assert distance(g.state, want) <= norm * (3 * eps + 2 * (n + 4) * 2.0 ** -53)
    g.close()
