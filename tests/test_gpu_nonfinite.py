"""Infinite and very large marked amplitudes in the single-state forms: an iteration is c' = 2S/N - s c with S = sum of s c,
in binary64 whatever the values, so an infinite marked amplitude gives S = -inf and unmarked amplitudes of -inf (a sum
that adds c and takes 2c off would be NaN), and marked amplitudes above half the largest binary64 value, whose sum with
the others is small, give finite ones.

Finite parts are compared with binary64 numpy at 2^-50 of the largest (complex64: 2^-22)."""
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


def iterated(part, sign):
    """One iteration of the real or the imaginary parts."""
    with np.errstate(all="ignore"):
        total = float(np.sum((sign * part).astype(np.longdouble)))
        return 2.0 * total / part.size - sign * part


FORMS = [(n, d, "resident") for n, d in ((3, "f64"), (7, "c64"), (10, "f64"), (11, "c128"), (13, "c64"), (14, "c128"))]
FORMS += [(13, "f64", "fused"), (16, "c64", "fused"), (18, "c128", "fused"), (23, "f64", "fused"), (24, "c64", "fused"), (17, "c64", "held")]


CASES = [(*f, v) for f in FORMS for v in ("inf", "-inf", "large") if (f[1], v) != ("c64", "large")]  # no such binary32


@pytest.mark.parametrize("rows", ["one", "several"])
@pytest.mark.parametrize("n,dtype,form,value", CASES)
def test_one_iteration(G, n, dtype, form, value, rows):
    print(f"{n} {dtype} {form} {value} {rows}", flush=True)
    N = 1 << n
    marks = [N // 2 + 1] if rows == "one" else sorted({i % N for i in (1, 1024, 1026, 3 * 1024 + 7, N // 2 + 1, N // 2 + 1024, N - 1)})
    sign = np.ones(N)
    sign[marks] = -1.0
    psi = workloads.random_state(n, seed=40 + n, real=dtype == "f64")
    re, im = psi.real.copy(), psi.imag.copy()
    if value == "large":
        re *= 1e300
        re[N // 2 + 1] = 1.2e308  # marked: -1.2e308 in the sum
        re[N // 2 + 2] = 1.2e308  # unmarked, of the next vector or the same one
    else:
        re[N // 2 + 1] = float(value)
    if dtype == "c64":
        with np.errstate(all="ignore"):
            re, im = re.astype(np.float32).astype(np.float64), im.astype(np.float32).astype(np.float64)
    state = np.empty(N, dtype={"f64": np.float64, "c64": np.complex64, "c128": np.complex128}[dtype])
    if dtype == "f64":
        state[:] = re
    else:
        state.real, state.imag = re, im
    g = G.Grover(n, dtype, marks=marks, form=form).write_state(state)
    got = g.iterate(1).read_state()
    g.sync()
    g.close()
    eps = 2.0 ** -22 if dtype == "c64" else 2.0 ** -50
    for have, part in ((got.real, re), (got.imag, im)):
        want = iterated(part, sign)
        have = have.astype(np.float64)
        finite = np.isfinite(want)
        assert np.array_equal(have[~finite], want[~finite], equal_nan=True)
        assert np.all(np.isfinite(have[finite]))
        scale = float(np.max(np.abs(part[np.isfinite(part)]))) if finite.any() else 0.0
        with np.errstate(all="ignore"):
            assert np.all(np.abs(have[finite] - want[finite]) <= eps * scale)
        if dtype == "f64":
            break
