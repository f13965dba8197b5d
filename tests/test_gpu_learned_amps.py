"""Learned chains whose proposals' amplitudes come from the matrix cores (calls of
eight steps or more, or amplitude records already there; n <= 60) against the same
chains through the caches (short calls), step for step, and the plain chain after
either, so that the caches are up to date however the steps were taken: chain counts
on both sides of a wave's and a workgroup's strings, terms on both sides of a tile
of 32 and of 256, widths at and past n = 60."""
import numpy as np
import pytest

import oracle as O
from paper_1808_00128_amd import workloads as W
from test_gpu_learned import B, say, start_states, varied_params  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,chi,chains", [(1, 1, 1), (10, 31, 3), (10, 33, 64), (50, 257, 65), (60, 300, 130),
                                          (61, 300, 40), (20, 700, 260), (50, 257, 15), (24, 300, 15), (25, 300, 15)])
def test_routes_agree(B, n, chi, chains):  # noqa: F811
    rng = np.random.default_rng(9100 + n + chains)
    circ = W.random_circuit(n, 8 * n + 10, rng.uniform(0, 2 * np.pi, size=5), rng)
    say(f"learned routes n={n} chi={chi} chains={chains}")
    spec = dict(circuit=circ, chi=chi, mode="sparsify", seed=91)
    T = O.Terms(circ, chi, O.SPARSIFY, seed=91)
    x0 = start_states(T, n, min(chains, 24), rng, chi)
    x0 = np.resize(x0, chains)
    calls = {"caches": (3, 4, 2, 5, 1), "records": (3, 12), "at once": (15,)}
    steps = 15
    u_mix, j, u_bits, u = W.learned_streams(n, chains, steps, rng)
    pj, pu = W.metropolis_streams(n, chains, 6, rng)
    out = {}
    for name, cuts in calls.items():
        ctx = B.Context([spec])
        ctx.apply_circuit(circ)
        net = B.MLP(ctx, n, 32, chains, varied_params(n, 32, seed=7))
        ctx.metropolis_init(x0)
        at, parts = 0, []
        for k in cuts:
            s = slice(at, at + k)
            parts.append(ctx.metropolis_step_learned(net, *(np.ascontiguousarray(a[:, s]) for a in (u_mix, j, u_bits, u)),
                                                     0.2, 0.01, 0.5))
            at += k
        ptr, pacc, pamp = ctx.metropolis_step(pj, pu)
        out[name] = [np.concatenate([p[i] for p in parts], axis=1) for i in range(3)] + [ptr, pacc, pamp]
        x = ptr[:, -1]
        ref = T.amplitudes(x)
        assert np.max(np.abs(pamp - ref)) <= 1e-11 * np.max(np.abs(ref)), name
        net.close()
        ctx.close()
    for name in ("records", "at once"):
        for a, e in zip(out[name][:5], out["caches"][:5]):
            assert np.array_equal(a, e), name
