"""The on-chip phase kernels at every number of vectors per thread they are compiled for (1 to 32 forward, 1 to 16
adjoint), with marked sets in one row and in several rows of a wave (which take another compiled form), and with
anchors (checkpoints re-read in the reverse sweep) at every step, at some and at the first step only.  Bounds: those
of the general phase tests, which hold for any order of additions."""
from __future__ import annotations

import numpy as np
import pytest

import workloads
from test_gpu_phase import G, cuda, forward_bound, grad_bound, loss_bound  # noqa: F401

pytestmark = pytest.mark.gpu

CASES = [(n, how, every) for n in (9, 10, 11, 12, 13, 14, 15, 16) for how in ("one", "rows") for every in (1, 3, 20)]
CASES += [(n, "row", 3) for n in (11, 12, 14, 15)]  # a whole row of vectors above the first, more marks than are listed


@pytest.mark.parametrize("n,how,every", CASES)
def test_on_chip_phase(G, orc, n, how, every):  # noqa: F811
    N, K = 1 << n, 7
    marks = [N // 3] if how == "one" else list(range(N // 2, N // 2 + 1024)) if how == "row" else sorted({i % N for i in (0, 1, 1024, 1026, 5 * 1024 + 4, N // 2, N - 1)})
    print(f"phase on chip n={n} marks={how} every={every}", flush=True)
    phi, theta = workloads.phase_schedule(K, seed=700 + n, spread=0.3, batch=2)
    eng = G.GroverPhase(n, marks, K, batch=2, checkpoint_every=every).set_form("held")
    g = np.array([1.0, -0.5])
    loss = eng.forward(cuda(phi), cuda(theta))
    eng.sync()
    states = [eng.read_state(b).astype(np.complex128) for b in range(2)]
    dphi, dtheta = (x.cpu().numpy() for x in eng.backward(cuda(g)))
    eng.sync()
    for b in range(2):
        want = orc.phase_search(n, marks, phi[b], theta[b])
        assert np.max(np.abs(states[b] - want)) <= forward_bound(K)
        assert abs(float(loss[b]) - orc.phase_loss(want, marks)) <= loss_bound(K)
        wphi, wtheta = orc.phase_grad_adjoint(n, marks, phi[b], theta[b])
        tol = grad_bound(K, every, g[b])
        assert np.max(np.abs(dphi[b] - g[b] * wphi)) <= tol
        assert np.max(np.abs(dtheta[b] - g[b] * wtheta)) <= tol
    eng.close()
