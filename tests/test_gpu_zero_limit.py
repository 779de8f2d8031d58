"""A wait limit of zero (GROVER_BARRIER_TIMEOUT_MS=0): kernels whose teams wait on each other give up, whether or not a
member would have had to wait (that of a team of one never, those of a few members not always); every workgroup exits, the
time-out is reported, and a context with a limit works."""
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


@pytest.mark.parametrize("n,form", [(6, "held"), (10, "held"), (13, "held"), (16, "held"), (20, "held"), (22, "held"), (13, "fused"), (23, "fused")])
def test_single_state(G, orc, monkeypatch, n, form):
    print(f"zero limit n={n} {form}", flush=True)
    monkeypatch.setenv("GROVER_BARRIER_TIMEOUT_MS", "0")
    g = G.Grover(n, "c64", marks=[5], form=form)
    for _ in range(5):
        g.iterate(3)
        with pytest.raises(G.GroverError) as e:
            g.sync()
        assert e.value.status == -7
    g.close()
    monkeypatch.delenv("GROVER_BARRIER_TIMEOUT_MS")
    g = G.Grover(n, "c64", marks=[5], form=form).iterate(3)
    g.sync()
    assert float(np.max(np.abs(g.read_state() - orc.search(n, [5], 3)))) <= 4 * 2.0 ** -23
    g.close()


@pytest.mark.parametrize("n", [8, 15, 17, 20])
def test_phase_on_chip(G, monkeypatch, n):
    import torch

    print(f"zero limit phase n={n}", flush=True)
    monkeypatch.setenv("GROVER_BARRIER_TIMEOUT_MS", "0")
    phi, theta = (torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in workloads.phase_schedule(6, seed=2, batch=1))
    e = G.GroverPhase(n, [5], 6, batch=1)
    e.set_form("held")
    for _ in range(5):
        e.forward(phi, theta)
        with pytest.raises(G.GroverError) as err:
            e.sync()
        assert err.value.status == G.grover.GROVER_E_TIMEOUT
    e.close()


def test_batch_teams(G, monkeypatch):
    monkeypatch.setenv("GROVER_BARRIER_TIMEOUT_MS", "0")
    b = G.GroverBatch([16, 16, 17], [1, 2, 1], [[5], [6, 7], [8]], iterations=[3, 3, 3])
    for _ in range(5):
        b.run()
        with pytest.raises(G.GroverError) as e:
            b.sync()
        assert e.value.status == -7
    b.close()
