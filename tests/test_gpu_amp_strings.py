"""The table amplitude kernel with one and two strings per lane (n > 60, and the
no-allocation call at any n), and what the autotuner of that choice times."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_1808_00128_amd import workloads as W
from test_gpu_parity import TOL32, TOL64, B, gpu_ctx, normwise, say  # noqa: F401

pytestmark = pytest.mark.gpu


def _device(x):
    return torch.from_numpy(x.view(np.int64)).cuda(), torch.zeros((x.size, 2), dtype=torch.float64, device="cuda:0")


@pytest.mark.parametrize("n,n_x", [(61, 255), (62, 257), (64, 513), (30, 256), (50, 700)])
@pytest.mark.parametrize("strings", [256, 512])
def test_strings_per_lane(B, n, n_x, strings):  # noqa: F811
    rng = np.random.default_rng(n)
    circ = W.random_circuit(n, 10 * n, rng.uniform(0, 2 * np.pi, size=6), rng)
    chi = 333
    say(f"table amplitudes n={n} n_x={n_x} strings={strings}")
    T = O.Terms(circ, chi, O.SPARSIFY, seed=9)
    xs = np.array([T.term(int(a)).sample(int(f)) for a, f in
                   zip(rng.integers(0, chi, size=n_x), W.random_bitstrings(n, n_x, rng))], np.uint64)
    ref = T.amplitudes(xs)
    ctx = gpu_ctx(B, dict(circuit=circ, chi=chi, mode="sparsify", seed=9))
    ctx.set_amp_strings(strings)
    x, out = _device(xs)
    for fp32c, tol in ((False, TOL64), (True, TOL32)):
        if n > 60:
            assert normwise(ctx.amplitudes(xs, fp32c=fp32c), ref) < tol
        ctx.amplitudes_noalloc(x, out, fp32c=fp32c)
        got = out.cpu().numpy()
        assert normwise(got[:, 0] + 1j * got[:, 1], ref) < tol


def test_autotuner_times_the_kernel_it_chooses_for(B):  # noqa: F811
    """At n = 50 the matrix cores take the call, but the choice is the table
    kernel's: what the tuner reports is that kernel's time, not less than 0.6 of a
    no-allocation call (which has the prologue, a tenth, on top), and the value is
    that of the smaller one."""
    n, chi, n_x = 50, 40000, 4096
    rng = np.random.default_rng(3)
    circ = W.random_circuit(n, 1000, rng.uniform(0, 2 * np.pi, size=10), rng)
    say("strings-per-item autotuner at n=50")
    ctx = gpu_ctx(B, dict(circuit=circ, chi=chi, mode="sparsify", seed=9))
    x, out = _device(W.random_bitstrings(n, n_x, rng))
    ref = ctx.amplitudes(x, fp32c=True).clone()
    ctx.set_amp_strings(-1)
    assert torch.equal(ctx.amplitudes(x, fp32c=True), ref)
    used, ms = ctx.amp_strings()
    assert used == (256 if ms[0] < ms[1] else 512)
    times = []
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        ctx.amplitudes_noalloc(x, out, fp32c=True)
        b.record()
        b.synchronize()
        times.append(a.elapsed_time(b))
    assert min(ms) > 0.6 * min(times)
