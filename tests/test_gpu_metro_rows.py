"""Single-flip Metropolis chains of up to 15 qubits against the CPU oracle on both
sides of the rule for the rows' form: rows that just fit the L2s and one term
more, one chain fewer than packing needs past them and that many, and as many
qubits as there are slots."""
import numpy as np
import pytest

import oracle as O
from paper_1808_00128_amd import workloads as W
from test_gpu_parity import B, gpu_ctx, normwise, say  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,chi,chains,shared", [
    (6, 300000, 1, False), (7, 246723, 1, False), (7, 246724, 1, True), (8, 216000, 1, False), (8, 216000, 2, False),
    (12, 143922, 3, False), (12, 143923, 3, False), (12, 143923, 4, True), (15, 115139, 6, False),
    (15, 115139, 6, True), (15, 115139, 7, False)])
def test_rows_form(B, n, chi, chains, shared):  # noqa: F811
    rng = np.random.default_rng(7400 + n + chi + chains)
    circ = W.random_circuit(n, 3 * n + 20, rng.uniform(0, 2 * np.pi, size=12), rng)
    say(f"metropolis rows n={n} chi={chi} chains={chains} shared={shared}")
    ctx = gpu_ctx(B, dict(circuit=circ, chi=chi, mode="sparsify", seed=74))
    T = O.Terms(circ, chi, O.SPARSIFY, seed=74)
    x0 = np.array([T.term(int(a)).sample(int(f)) for a, f in zip(rng.integers(0, chi, size=64),
                                                                 W.random_bitstrings(n, 64, rng))], np.uint64)
    x0 = np.resize(x0[np.abs(T.amplitudes(x0)) > 1e-9], chains)
    j, u = W.metropolis_streams(n, chains, 7, rng, shared_j=shared)
    otr, oacc, oamp = T.metropolis(x0, j, u)
    for graph in (False, True):
        ctx.metropolis_init(x0)
        at = 0
        for k in (5, 2):
            tr, acc, amp = ctx.metropolis_step(np.ascontiguousarray(j[:, at:at + k]),
                                               np.ascontiguousarray(u[:, at:at + k]), graph=graph)
            assert np.array_equal(tr, otr[:, at:at + k]), (graph, at)
            assert np.array_equal(acc, oacc[:, at:at + k]), (graph, at)
            at += k
        assert normwise(amp, oamp) < 1e-10
