"""A team that cannot be co-resident: the fused form and AUTO stream the state instead, the held form is refused.  The
check itself passes here; GROVER_TEAM_CHECK=fail makes it report the opposite.  And the streaming kernel with binary64
sums on states that are otherwise held on chip: calls compose bit for bit.

Tolerances: complex64 stores each part rounded to 2^-24 relative and sums in binary64, so k iterations of a normalised
state stay within (k + 1) 2^-23 of the exact ones per part; binary64 storage within (k + 1) 2^-50."""
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
    psi = workloads.random_state(n, seed=30 + n, real=dtype == "f64")
    return psi.real.copy() if dtype == "f64" else psi.astype(np.complex64 if dtype == "c64" else np.complex128)


def tolerance(dtype, k):
    return (k + 1) * (2.0 ** -23 if dtype == "c64" else 2.0 ** -50)


@pytest.mark.parametrize("n,dtype,form,update", [(15, "c64", "auto", "f64"), (20, "c64", "auto", "f32"), (23, "c64", "auto", "f64"),
                                                 (13, "c64", "fused", "f64"), (18, "f64", "fused", "f64"), (22, "c128", "fused", "f64"),
                                                 (24, "c64", "auto", "f64")])
def test_streams_instead(G, orc, monkeypatch, n, dtype, form, update):
    print(f"fallback n={n} {dtype} {form}", flush=True)
    monkeypatch.setenv("GROVER_TEAM_CHECK", "fail")
    psi, marks, k = start(n, dtype), [1, (1 << n) // 3], 3
    g = G.Grover(n, dtype, marks=marks, form=form, update=update)
    assert g.query(G.grover.Q_FORM) == G.grover.FORMS["fused"]
    g.write_state(psi).iterate(k)
    g.sync()
    got = g.read_state()
    want = psi.astype(np.complex128)
    orc.iterate(want, marks, k)
    assert float(np.max(np.abs(got.astype(np.complex128) - want))) <= tolerance(dtype, k)
    assert abs(g.reset().norm() - 1.0) < 1e-5
    g.close()
    monkeypatch.delenv("GROVER_TEAM_CHECK")
    if form == "auto" and n < 24:
        g = G.Grover(n, dtype, marks=marks, update=update)
        assert g.query(G.grover.Q_FORM) == G.grover.FORMS["held"]
        g.close()


def test_held_form_is_refused(G, monkeypatch):
    monkeypatch.setenv("GROVER_TEAM_CHECK", "fail")
    with pytest.raises(G.GroverError) as e:
        G.Grover(17, "c64", marks=[1], form="held")
    assert e.value.status == -4


@pytest.mark.parametrize("n,dtype", [(13, "c64"), (19, "f64"), (18, "c128"), (24, "c64")])
def test_streamed_calls_compose(G, orc, monkeypatch, n, dtype):
    monkeypatch.setenv("GROVER_FUSED_TEMPORAL", "1")
    psi, marks, k = start(n, dtype), workloads.distinct_marks(n, 9, seed=n), 5
    g = G.Grover(n, dtype, marks=marks, form="fused").write_state(psi)
    got = g.iterate(2).iterate(k - 2).read_state()
    again = g.write_state(psi).iterate(k).read_state()
    g.sync()
    g.close()
    assert np.array_equal(got.view(np.uint8), again.view(np.uint8))
    want = psi.astype(np.complex128)
    orc.iterate(want, marks, k)
    assert float(np.max(np.abs(got.astype(np.complex128) - want))) <= tolerance(dtype, k)
