"""The on-chip kernels (one workgroup; a team, in the held and the fused form) at the sizes where it can go wrong: every number of vectors
per thread it is compiled for (1 to 64, registers and LDS), members smaller than a workgroup, the smallest and the
largest team, and marked sets that sit in one row, in several rows of a wave, or too densely to be listed.

Tolerances: complex64 stores each part rounded to 2^-24 relative and sums in binary64, so k iterations of a
normalised state stay within (k + 1) 2^-23 of the exact ones per part; binary64 storage within (k + 1) 2^-50."""
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


def start(n, dtype):
    psi = workloads.random_state(n, seed=900 + n, real=dtype == "f64")
    return psi.real.copy() if dtype == "f64" else psi.astype(np.complex64 if dtype == "c64" else np.complex128)


def marked(n, how):
    N = 1 << n
    if how == "one":
        return [N // 3]
    if how == "rows":  # several rows of one wave, both amplitudes of a vector, the first and the last amplitude
        return sorted({i % N for i in (0, 1, 1024, 1026, 3 * 1024 + 7, N // 2, N // 2 + 1024, N - 1)})
    if how == "row":  # a whole row of vectors above the first
        return list(range(N // 2, N // 2 + 1024))
    return list(range(0, N, 2)) + [1]  # too many for a member to list


CASES = ([(n, "c64", "held", "rows", "f64") for n in (1, 2, 8, 9, 10, 11, 13, 15, 17, 19, 20, 21, 22, 23)]
         + [(n, "c64", "held", how, up) for n in (10, 12, 14, 18) for how in ("one", "dense") for up in ("f64", "f32")]
         + [(n, d, "resident", how, "f64") for n in (1, 3, 6, 7, 8, 9, 10, 11, 12, 13, 14) for d in ("f64", "c64", "c128")
            for how in ("rows", "dense")]
         + [(n, "c64", "resident", "rows", "f32") for n in (5, 8, 10, 12, 14)]
         + [(n, "c64", form, "row", "f64") for n, form in ((11, "resident"), (14, "resident"), (16, "held"), (22, "held"))]
         + [(n, d, "fused", "rows", "f64") for d in ("f64", "c128") for n in (14, 15, 18, 20, 22)]
         + [(24, "f64", "fused", "rows", "f64"), (23, "c128", "fused", "rows", "f64"), (23, "f64", "fused", "one", "f64"),
            (24, "c64", "auto", "rows", "f64"), (24, "c64", "fused", "one", "f32"), (16, "c64", "fused", "dense", "f64"),
            (13, "c128", "fused", "dense", "f64"), (21, "c64", "fused", "rows", "f32")])


@pytest.mark.parametrize("n,dtype,form,how,update", CASES)
def test_on_chip_iteration(G, orc, n, dtype, form, how, update):
    print(f"on chip n={n} {dtype} {form} marks={how} update={update}", flush=True)
    psi0, marks, k = start(n, dtype), marked(n, how), 3
    want = psi0.astype(np.complex128)
    orc.iterate(want, marks, k)
    g = G.Grover(n, dtype, marks=marks, form=form, update=update).write_state(psi0)
    got = g.iterate(1).iterate(k - 1).read_state()
    again = g.write_state(psi0).iterate(k).read_state()
    g.sync()
    g.close()
    assert np.array_equal(got.view(np.uint8), again.view(np.uint8))  # calls compose bit for bit
    scale = max(1.0, float(np.max(np.abs(want))))
    tol = (k + 1) * (2.0**-23 if dtype == "c64" else 2.0**-50) * scale
    assert float(np.max(np.abs(got.astype(np.complex128) - want))) <= tol
