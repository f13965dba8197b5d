"""Single-flip Metropolis chains, two steps per launch, against the CPU oracle's
chain step for step where the launch shapes meet: odd and even step counts (a
last step alone, windows cut by the call's end), the three ways of holding rows
(n <= 15, n <= 30, above), tiles with one term and one past a whole tile, chain
counts that leave a pass of two with one chain, that split over workgroups and
that pass 64 per wave, one flip bit per step for every chain or each its own."""
import numpy as np
import pytest

import oracle as O
from paper_1808_00128_amd import workloads as W
from test_gpu_parity import B, gpu_ctx, normwise, say  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,chi,chains,calls,shared", [
    (1, 1, 1, (1,), True), (2, 3, 2, (2, 3), False), (15, 256, 3, (5, 4), False), (15, 257, 9, (6, 1), True),
    (16, 255, 8, (7,), False), (30, 513, 33, (3, 8), True), (30, 700, 5, (9,), False), (31, 257, 17, (4, 5), False),
    (50, 3000, 64, (11,), True), (62, 300, 7, (2, 1, 10), False), (12, 70, 300, (6,), False),
    (40, 1, 2100, (5,), False)])
def test_pairs_of_steps(B, n, chi, chains, calls, shared):  # noqa: F811
    rng = np.random.default_rng(7300 + n + chi)
    circ = W.random_circuit(n, 3 * n + 20, rng.uniform(0, 2 * np.pi, size=12), rng)
    say(f"metropolis pairs n={n} chi={chi} chains={chains} calls={calls} shared={shared}")
    ctx = gpu_ctx(B, dict(circuit=circ, chi=chi, mode="sparsify", seed=73))
    T = O.Terms(circ, chi, O.SPARSIFY, seed=73)
    x0 = np.empty(0, np.uint64)
    while x0.size < chains:
        alpha = rng.integers(0, chi, size=chains)
        x = np.array([T.term(int(a)).sample(int(f)) for a, f in zip(alpha, W.random_bitstrings(n, chains, rng))],
                     np.uint64)
        x0 = np.concatenate([x0, x[np.abs(T.amplitudes(x)) > 1e-9]])[:chains]
    steps = sum(calls)
    j, u = W.metropolis_streams(n, chains, steps, rng, shared_j=shared)
    otr, oacc, oamp = T.metropolis(x0, j, u)
    for graph in (False, True):
        ctx.metropolis_init(x0)
        at = 0
        for k in calls:
            tr, acc, amp = ctx.metropolis_step(np.ascontiguousarray(j[:, at:at + k]),
                                               np.ascontiguousarray(u[:, at:at + k]), graph=graph)
            assert np.array_equal(tr, otr[:, at:at + k]), (graph, at)
            assert np.array_equal(acc, oacc[:, at:at + k]), (graph, at)
            at += k
        assert normwise(amp, oamp) < 1e-10
