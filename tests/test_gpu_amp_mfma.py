"""Matrix-core amplitudes (n <= 60) against the CPU oracle where the kernel's
cases meet: the register classes by number of 64-feature steps (n = 10/11,
22/23, 31/32, 41/42, 50/51), the largest n it takes and the first the table
kernel keeps (60/61), partial tiles of 32 terms, string counts around one wave's
and one workgroup's share and the switch from split to shared tiles, and
condition counts n - |v| of none, a part, a whole and several groups of three.

Tolerances as everywhere for amplitudes: m is whole-number arithmetic, so the
values are exact and only their sum rounds: FP64 within 1e-12, FP32C within
1e-6 of the oracle, normwise."""
import numpy as np
import pytest

import oracle as O
from paper_1808_00128_amd import workloads as W
from test_gpu_parity import TOL32, TOL64, B, _support_circuit, normwise, say  # noqa: F401

pytestmark = pytest.mark.gpu


# (n, qubits in the support, further (slot, H) pairs, chi, n_x)
EDGES = [
    (1, 1, 0, 1, 1), (3, 2, 1, 33, 4), (10, 10, 0, 31, 1), (11, 8, 2, 33, 129), (22, 19, 1, 32, 128),
    (23, 20, 3, 65, 257), (31, 28, 0, 64, 64), (32, 26, 0, 97, 65), (41, 35, 2, 64, 300), (42, 12, 3, 33, 129),
    (50, 50, 0, 40, 260), (50, 46, 2, 70, 300), (51, 38, 2, 70, 130), (59, 56, 2, 65, 64), (60, 20, 2, 33, 33),
    (60, 60, 0, 96, 513), (61, 58, 2, 33, 65),
]


@pytest.mark.parametrize("n,k,pairs,chi,n_x", EDGES)
def test_amplitudes_at_the_kernel_edges(B, n, k, pairs, chi, n_x):  # noqa: F811
    rng = np.random.default_rng(7000 + 100 * n + k)
    circ = _support_circuit(n, k, pairs, rng)
    say(f"amplitudes edges n={n} k={k} pairs={pairs} chi={chi} n_x={n_x}")
    if circ.n_slot == 0:  # every draw of a slotless circuit is the same term
        circ = W.from_list(n, [(W.OP_SLOT, 0, 0, 0.4)] + [g[:3] for g in circ.gates()])
    T = O.Terms(circ, chi, O.SPARSIFY, seed=n + k)
    ctx = B.Context([dict(circuit=circ, chi=chi, mode="sparsify", seed=n + k)])
    ctx.apply_circuit(circ)
    alpha = rng.integers(0, chi, size=n_x)
    flips = W.random_bitstrings(n, n_x, rng)
    xs = np.array([T.term(int(a)).sample(int(f)) for a, f in zip(alpha, flips)], np.uint64)
    xs[1::5] = W.random_bitstrings(n, n_x, rng)[1::5]
    ref = T.amplitudes(xs)
    assert np.max(np.abs(ref)) > 0
    assert normwise(ctx.amplitudes(xs), ref) < TOL64
    assert normwise(ctx.amplitudes(xs, fp32c=True), ref) < TOL32


def test_amplitudes_batch_of_split_and_shared_requests(B):  # noqa: F811
    """One call whose requests take the split and the shared kernel and, with
    n = 62, the table kernel, some on the same instance."""
    rng = np.random.default_rng(77)
    shapes = [(9, 40, 300), (33, 100, 20), (50, 70, 140), (62, 35, 90)]
    specs, terms, reqs, refs = [], [], [], []
    for i, (n, chi, n_x) in enumerate(shapes):
        circ = W.random_circuit(n, 12 * n, rng.uniform(0, 2 * np.pi, size=6), rng)
        specs.append(dict(circuit=circ, chi=chi, mode="sparsify", seed=i))
        terms.append(O.Terms(circ, chi, O.SPARSIFY, seed=i))
        for cnt in (n_x, 1):
            xs = np.array([terms[i].term(int(a)).sample(int(f)) for a, f in
                           zip(rng.integers(0, chi, size=cnt), W.random_bitstrings(n, cnt, rng))], np.uint64)
            reqs.append((i, xs))
            refs.append(terms[i].amplitudes(xs))
    say("amplitudes batch of split, shared and table requests")
    ctx = B.Context(specs)
    for i, sp in enumerate(specs):
        ctx.apply_circuit(sp["circuit"], inst=i)
    for _ in range(2):
        for a, ref in zip(ctx.amplitudes_batch(reqs), refs):
            assert normwise(a, ref) < TOL64
        for a, ref in zip(ctx.amplitudes_batch(reqs, fp32c=True), refs):
            assert normwise(a, ref) < TOL32
