"""Marked sets of every length on the on-chip kernels: up to 16 marks of a member are gone through in the lanes of its
waves, more are scattered through LDS, and beyond 64 the member's part of the list is searched for first.

Tolerances: complex64 stores each part rounded to 2^-24 relative and sums in binary64, so k iterations of a normalised
state stay within (k + 1) 2^-23 of the exact ones per part; binary64 storage within (k + 1) 2^-50.  An iteration's bound
scales with the largest amplitude, of at most 1 here."""
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


def marked(n, m, how):
    N = 1 << n
    if how == "spread":
        return sorted(np.random.default_rng(1000 * n + m).choice(N, size=m, replace=False).tolist())
    if how == "low":  # all in the first member, the others' parts of the list are empty
        return list(range(m))
    return list(range(N - m, N))  # all in the last one


CASES = [(n, d, "resident", m) for n, d in ((7, "c64"), (8, "f64"), (9, "c128"), (10, "c64"), (12, "f64"), (14, "c128"), (14, "c64"))
         for m in (15, 16, 17, 63, 64, 65, 127)]
CASES += [(n, d, "fused", m) for n, d in ((13, "c64"), (16, "c128"), (21, "f64")) for m in (16, 17, 64, 65, 4097)]
CASES += [(n, "c64", "held", m) for n in (15, 17, 20, 23) for m in (16, 17, 64, 65, 1000)]


@pytest.mark.parametrize("how", ["spread", "low", "high"])
@pytest.mark.parametrize("n,dtype,form,m", CASES)
def test_list_lengths(G, orc, n, dtype, form, m, how):
    print(f"marks n={n} {dtype} {form} m={m} {how}", flush=True)
    marks, k = marked(n, m, how), 2
    psi = workloads.random_state(n, seed=70 + n, real=dtype == "f64")
    psi = psi.real.copy() if dtype == "f64" else psi.astype(np.complex64 if dtype == "c64" else np.complex128)
    want = psi.astype(np.complex128)
    orc.iterate(want, marks, k)
    g = G.Grover(n, dtype, marks=marks, form=form).write_state(psi)
    got = g.iterate(k).read_state().astype(np.complex128)
    g.sync()
    g.close()
    assert float(np.max(np.abs(got - want))) <= (k + 1) * (2.0 ** -23 if dtype == "c64" else 2.0 ** -50)


@pytest.mark.parametrize("n,m", [(12, 40), (16, 200), (20, 1000)])
def test_batch_and_phase_lists(G, orc, n, m):
    """The batched and the phase kernels find their marks in the same way (m above 16 in a member)."""
    import torch

    marks = marked(n, m, "low")
    b = G.GroverBatch([n, n], [m, 1], [marks, [5]], iterations=[3, 2]).run()
    b.sync()
    want = orc.search(n, marks, 3)
    assert float(np.max(np.abs(b.read_state(0).astype(np.complex128) - want))) <= 4 * 2.0 ** -23
    b.close()
    e = G.GroverPhase(n, marks, 3)
    full = torch.full((1, 3), np.pi, dtype=torch.float64, device="cuda")
    loss = float(e.forward(full, full)[0])  # phases of pi are the plain iteration
    e.sync()
    e.close()
    assert abs(loss - (1.0 - float(np.sum(np.abs(want[marks]) ** 2)))) <= m * 4 * 2.0 ** -22


@pytest.mark.parametrize("n,dtype,m", [(10, "f64", 64), (14, "c64", 300), (14, "c128", 1000)])
def test_long_list_costs_little(G, n, dtype, m):
    """One iteration per call: the marks are found anew in each, which must not take longer than the iteration."""
    import torch

    def us(marks):
        g = G.Grover(n, dtype, marks=marks, form="resident")
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        best = 1e9
        for _ in range(8):
            a.record()
            for _ in range(100):
                g.iterate(1)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b) * 10.0)
        g.close()
        return best

    one, many = us([3]), us(marked(n, m, "spread"))
    print(f"n={n} {dtype}: {one:.2f} us with one mark, {many:.2f} with {m}", flush=True)
    assert many <= 2.0 * one
