"""The evolution autotuner against the default: what it keeps is no slower, and the
times it reports are those of repeated runs."""
import numpy as np
import pytest
import torch

from paper_1808_00128_amd import workloads as W
from test_gpu_parity import B, say  # noqa: F401

pytestmark = pytest.mark.gpu


def _ms(ctx, g, reps=12):
    times = []
    for _ in range(reps):
        ctx.reset(3)
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        ctx.apply_gates(g)
        b.record()
        b.synchronize()
        times.append(a.elapsed_time(b))
    return min(times)


@pytest.mark.parametrize("n,gates,slots,chi", [(50, 2000, 40, 65536), (24, 500, 30, 20000)])
def test_tuned_is_no_slower_than_the_default(B, n, gates, slots, chi):  # noqa: F811
    rng = np.random.default_rng(n)
    circ = W.random_circuit(n, gates, rng.uniform(0, 2 * np.pi, size=slots), rng)
    g = B.gate_array(circ)
    say(f"evolution autotuner n={n} chi={chi}")
    ctx = B.Context([dict(circuit=circ, chi=chi, mode="sparsify", seed=3)])
    plain = _ms(ctx, g)
    ctx.set_evolve_lanes(-1)
    ctx.reset(3)
    ctx.apply_gates(g)
    tuned = _ms(ctx, g)
    assert tuned < 1.05 * plain
    # Events around the call here, around the evolution's launches there.
    lanes, ms = ctx.evolve_lanes()
    for v, t in zip(B.TUNE_SHAPES, ms):
        if t > 0 and v in (4 | 0x100, 8 | 0x100, 16 | 0x100):
            ctx.set_evolve_lanes(v)
            run = _ms(ctx, g)
            assert 0.7 * run < t < 1.15 * run, (hex(v), t, run)
