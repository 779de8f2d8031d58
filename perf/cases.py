"""The work that programs have this library do, as cases that a timing tool can run.

A case is a dict of plain values; `prepare` makes what a program holds before the call (the context, its marked
set, input tensors), `run` makes one pass through the public entry points and returns what it computed, `exact`
says what that is in 64-bit arithmetic without this library, and `work` what the pass cannot do without.

Kinds of work:
  search   one search from the uniform state: reset, `iterations` Grover iterations, optionally measurement shots
  measure  the norm and `shots` measurement shots of a state that a search has reached
  batch    many searches of uneven size in one launch
  phase    one training step of the generalized iteration: losses of all schedules and both gradients
  gate     iterations of the conventional gate-level simulator in its blocked form
"""
import math
import random

import numpy as np
import torch

import paper_2005_04635_amd as grover

ELEM_BYTES = {"f64": 8, "c64": 8, "c128": 16, "cbf16": 4}
TORCH_TYPES = {"f64": torch.float64, "c64": torch.complex64, "c128": torch.complex128}
# registers and LDS of 256 CUs: a state no larger can stay on chip for all iterations of a call
ON_CHIP_BYTES = 256 * (512 + 160) * 1024
# amplitude updates of the largest listed search, and so the most that a drawn one may ask for (in 8-byte units)
MOST_UPDATES = (1 << 28) * 200


def optimal(n, m):
    return int(math.pi / 4 * math.sqrt(2.0**n / m))


def listed():
    return [
        # the plain search: real binary64, one solution, its optimal iterations and 10^4 shots; latency only
        dict(name="search_n10_f64_shots", kind="search", n=10, m=1, dtype="f64", update="f64", accum="f64",
             iterations=25, shots=10_000),
        # a small complex search with a few solutions: one workgroup
        dict(name="search_n13_c64", kind="search", n=13, m=3, dtype="c64", update="f64", accum="f64",
             iterations=optimal(13, 3), shots=0),
        # a single-solution search of the size range that papers tabulate, with the faster binary32 update
        dict(name="search_n16_c64_u32", kind="search", n=16, m=1, dtype="c64", update="f32", accum="f64",
             iterations=optimal(16, 1), shots=0),
        # the same at n = 20 with the default update
        dict(name="search_n20_c64", kind="search", n=20, m=1, dtype="c64", update="f64", accum="f64",
             iterations=optimal(20, 1), shots=0),
        # full precision storage at a middle size
        dict(name="search_n21_c128", kind="search", n=21, m=2, dtype="c128", update="f64", accum="f64",
             iterations=optimal(21, 2), shots=0),
        # a 128 MiB state, advanced by part of its search
        dict(name="search_n24_c64", kind="search", n=24, m=1, dtype="c64", update="f64", accum="f64", iterations=801,
             shots=0),
        # reduced storage at the size of the precision study
        dict(name="search_n26_cbf16", kind="search", n=26, m=4, dtype="cbf16", update="f64", accum="f64",
             iterations=300, shots=0),
        # the large instance: a 2 GiB state that streams from memory, advanced by part of its search
        dict(name="search_n28_c64", kind="search", n=28, m=8, dtype="c64", update="f64", accum="f64", iterations=200,
             shots=0),
        # measurement of the large instance: its norm and 10^6 shots from resident uniforms
        dict(name="measure_n28_c64", kind="measure", n=28, m=8, dtype="c64", progress=1.0, shots=1_000_000),
        # a thousand searches of mixed size, as a service or a study of many instances runs them
        dict(name="batch_1024", kind="batch", count=1024, n_min=8, n_max=20, m_max=8, update="f64"),
        # a training step over 64 phase schedules
        dict(name="phase_n20_b64", kind="phase", n=20, m=3, K=64, batch=64),
        # the conventional simulator for comparison, at an odd qubit count
        dict(name="gate_n25_c64", kind="gate", n=25, m=2, dtype="c64", iterations=4),
    ]


def draw(rng):
    kind = rng.choices(["search", "measure", "batch", "phase", "gate"], [10, 3, 3, 3, 3])[0]
    if kind == "search":
        dtype = rng.choices(["c64", "f64", "c128", "cbf16"], [5, 2, 2, 1])[0]
        n = rng.randint(8, 25 if dtype == "c128" else 26)
        m = min(2 ** (n - 3), int(2 ** rng.uniform(0, 6)))
        update, accum = "f64", "f64"
        if dtype == "c64":
            update, accum = rng.choices([("f64", "f64"), ("f32", "f64"), ("f64", "f32"), ("f64", "f32_kahan")],
                                        [6, 3, 1, 1])[0]
        k = max(1, int(optimal(n, m) * rng.uniform(0.4, 1.0)))
        k = min(k, MOST_UPDATES * 8 // (4 * (1 << n) * max(8, ELEM_BYTES[dtype])))
        shots = int(10 ** rng.uniform(2, 5)) if dtype in ("f64", "c128") and rng.random() < 0.5 else 0
        return dict(kind=kind, n=n, m=m, dtype=dtype, update=update, accum=accum, iterations=k, shots=shots)
    if kind == "measure":
        n = rng.randint(12, 28)
        return dict(kind=kind, n=n, m=int(2 ** rng.uniform(0, 6)), dtype=rng.choice(["c64", "c64", "f64", "c128"]),
                    progress=rng.choice([0.0, 0.5, 1.0]), shots=int(10 ** rng.uniform(3, 6.3)))
    if kind == "batch":
        n_max = rng.randint(12, 20)
        return dict(kind=kind, count=int(2 ** rng.uniform(5, 10)), n_min=rng.randint(8, n_max - 2), n_max=n_max,
                    m_max=rng.choice([1, 4, 8]), update=rng.choice(["f64", "f64", "f32"]))
    if kind == "phase":
        n = rng.randint(10, 22)
        return dict(kind=kind, n=n, m=int(2 ** rng.uniform(0, 4)), K=rng.randint(12, 96),
                    batch=int(2 ** rng.uniform(0, min(7, 26 - n))))
    dtype = rng.choice(["c64", "c64", "f64", "c128"])
    return dict(kind=kind, n=rng.randint(10, 26), m=int(2 ** rng.uniform(0, 4)), dtype=dtype,
                iterations=rng.randint(1, 8))


def _marks(n, m, seed):
    """m distinct indices: one among the first 512, so that the head of a large state shows it, the others anywhere."""
    r = random.Random(1_000_003 * seed + 1009 * n + m)
    first = r.randrange(min(1 << n, 512))
    others = [i for i in r.sample(range(1 << n), m) if i != first]
    return sorted([first] + others[: m - 1])


def _batch_instances(case, seed):
    r = random.Random(case["count"])  # the sizes are the case's, the marked sets the seed's
    n = [r.randint(case["n_min"], case["n_max"]) for _ in range(case["count"])]
    m = [r.randint(1, case["m_max"]) for _ in n]
    r = random.Random(7919 * seed + case["count"])
    return n, m, [sorted(r.sample(range(1 << a), b)) for a, b in zip(n, m)]


def _phase_inputs(case, seed):
    g = torch.Generator().manual_seed(seed)
    z = torch.randn(2, case["batch"], case["K"], generator=g, dtype=torch.float64)
    phi, theta = math.pi + 0.1 * z
    return phi, theta


def _reached(case, seed, dtype, device):
    """The state a search has reached after the given part of its optimal iterations: its marked and its other
    amplitudes have one value each."""
    n, m = case["n"], case["m"]
    angle = math.asin(math.sqrt(m / 2.0**n))
    k = int(case["progress"] * optimal(n, m))
    out = torch.full((1 << n,), math.cos((2 * k + 1) * angle) / math.sqrt(2.0**n - m), dtype=dtype, device=device)
    out[torch.tensor(_marks(n, m, seed), device=device)] = math.sin((2 * k + 1) * angle) / math.sqrt(m)
    return out


class _DeviceArray:
    """Complex64 device memory of another owner, which it keeps alive, for torch to view."""

    def __init__(self, owner, ptr, count):
        self.owner = owner
        self.__cuda_array_interface__ = dict(shape=(count,), typestr="<c8", data=(ptr, False), version=2)


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("search", "gate"):
        g = grover.Grover(case["n"], case["dtype"], _marks(case["n"], case["m"], seed),
                          accum=case.get("accum", "f64"), update=case.get("update", "f64"))
        return dict(kind=kind, g=g, iterations=case["iterations"], shots=case.get("shots", 0), seed=seed)
    if kind == "measure":
        g = grover.Grover(case["n"], case["dtype"], _marks(case["n"], case["m"], seed))
        g.state.copy_(_reached(case, seed, TORCH_TYPES[case["dtype"]], "cuda"))
        gen = torch.Generator(device="cuda").manual_seed(seed)
        u = torch.randint(0, 1 << 53, (case["shots"],), generator=gen, device="cuda", dtype=torch.int64)
        return dict(kind=kind, g=g, u53=u, shots=case["shots"])
    if kind == "batch":
        n, m, marks = _batch_instances(case, seed)
        b = grover.GroverBatch(n, m, marks, update=case["update"])
        first, _ = grover.grover_batch_state(b.b, 0)
        last, size = grover.grover_batch_state(b.b, len(n) - 1)
        states = torch.as_tensor(_DeviceArray(b, first, (last + size - first) // 8), device="cuda")
        states.owner = b  # the memory is the batch's: whoever holds the view holds the batch
        return dict(kind=kind, b=b, states=states)
    phi, theta = _phase_inputs(case, seed)
    engine = grover.GroverPhase(case["n"], _marks(case["n"], case["m"], seed), case["K"], batch=case["batch"])
    return dict(kind=kind, engine=engine, phi=phi.cuda().requires_grad_(), theta=theta.cuda().requires_grad_())


def run(state):
    kind = state["kind"]
    if kind == "search":
        g = state["g"].reset().iterate(state["iterations"])
        if state["shots"]:
            return dict(state=g.state, shots=g.sample(state["shots"], seed=state["seed"], device_out=True))
        return dict(state=g.state)
    if kind == "gate":
        return dict(state=state["g"].reset().gate_iterate_blocked(state["iterations"]).state)
    if kind == "measure":
        g = state["g"]
        return dict(norm=g.norm(), shots=g.sample(state["shots"], u53=state["u53"], device_out=True))
    if kind == "batch":
        state["b"].run()
        return dict(states=state["states"])
    loss = state["engine"].loss(state["phi"], state["theta"])
    dphi, dtheta = torch.autograd.grad(loss.sum(), (state["phi"], state["theta"]))
    return dict(loss=loss.detach(), dphi=dphi, dtheta=dtheta)


def work(case):
    kind = case["kind"]
    if kind in ("search", "gate"):
        N, eb, k = 1 << case["n"], ELEM_BYTES[case["dtype"]], case["iterations"]
        parts = 1 if case["dtype"] == "f64" else 2
        if kind == "gate":  # H^n twice: n additions per part each; the state has to be read and written once
            return dict(bytes=2.0 * N * eb, flops=2.0 * parts * N * case["n"] * k)
        # from the uniform state: written once when it can stay on chip, else read and written every iteration,
        # for the next sum needs every amplitude of this one; a subtraction and an addition per part
        moved = N * eb if N * eb <= ON_CHIP_BYTES else 2.0 * N * eb * k
        return dict(bytes=moved + 8.0 * case["shots"], flops=2.0 * parts * N * k)
    if kind == "measure":
        N, eb = 1 << case["n"], ELEM_BYTES[case["dtype"]]
        return dict(bytes=N * eb + 16.0 * case["shots"], flops=4.0 * N)
    if kind == "batch":
        n, m, _ = _batch_instances(case, 0)
        return dict(bytes=sum(8.0 * 2**a for a in n), flops=sum(4.0 * 2**a * optimal(a, b) for a, b in zip(n, m)))
    # states are left in memory by the forward run; state and adjoint state take a step back together
    N, B, K = 1 << case["n"], case["batch"], case["K"]
    return dict(bytes=8.0 * N * B + 32.0 * B * K, flops=3 * 4.0 * N * B * K)


def _two_values(n, m, k):
    """The unmarked and the marked amplitude after k iterations from the uniform state, by the iteration itself."""
    N = 2.0**n
    u = a = 1.0 / math.sqrt(N)
    for _ in range(k):
        twice_mean = 2.0 * ((N - m) * u - m * a) / N
        u, a = twice_mean - u, twice_mean + a
    return u, a


def _two_valued(n, marks, k, device="cpu"):
    u, a = _two_values(n, len(marks), k)
    out = torch.full((1 << n,), u, dtype=torch.float64, device=device)
    out[torch.tensor(marks, device=device)] = a
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind in ("search", "gate"):
        device = "cuda" if torch.cuda.is_available() else "cpu"
        out = _two_valued(case["n"], _marks(case["n"], case["m"], seed), case["iterations"], device)
        if case["dtype"] == "cbf16":  # re, im, re, im, ...
            out = torch.stack((out, torch.zeros_like(out)), 1).reshape(-1)
        elif case["dtype"] != "f64":
            out = torch.complex(out, torch.zeros_like(out))
        return dict(state=out, shots=None) if case.get("shots") else dict(state=out)
    if kind == "measure":
        state = _reached(case, seed, TORCH_TYPES[case["dtype"]], "cpu")
        parts = torch.view_as_real(state) if state.is_complex() else state
        return dict(norm=float(np.sum(np.square(parts.numpy().astype(np.float64)))), shots=None)
    if kind == "batch":
        n, m, marks = _batch_instances(case, seed)
        out = torch.cat([_two_valued(a, x, optimal(a, b)) for a, b, x in zip(n, m, marks)])
        return dict(states=torch.complex(out, torch.zeros_like(out)))
    N, m = 2.0 ** case["n"], case["m"]
    phi, theta = (x.requires_grad_() for x in _phase_inputs(case, seed))
    u = torch.full((case["batch"],), 1.0 / math.sqrt(N), dtype=torch.complex128)
    a = u.clone()
    for j in range(case["K"]):
        a = torch.exp(1j * phi[:, j]) * a
        mean = (1.0 - torch.exp(1j * theta[:, j])) * ((N - m) * u + m * a) / N
        u, a = mean - u, mean - a
    loss = 1.0 - m * (a.real**2 + a.imag**2)
    dphi, dtheta = torch.autograd.grad(loss.sum(), (phi, theta))
    return dict(loss=loss.detach(), dphi=dphi, dtheta=dtheta)
