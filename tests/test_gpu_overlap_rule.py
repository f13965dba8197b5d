"""Inner products of CH forms where the kets of one call go to different kernels: sets
that hold terms of two sizes, with bra counts around those from which a size is taken
by the bit-sliced kernels (the rule's own values, read from its formula), against the
CPU oracle's sums for the two halves."""
import numpy as np
import pytest

import oracle as O
from paper_1808_00128_amd import workloads as W
from test_gpu_parity import B, normwise, say  # noqa: F401
from test_gpu_quad_pairs import TOL64, _spread

pytestmark = pytest.mark.gpu


def _takes(n, bras, nc, w):
    small = max(40.0, 9.5 * n - 40.0) * (1.55 if n >= 55 else 1.0)
    us = (small, max(100.0, 20.0 * n - 300.0), max(800.0, 35.4 * n - 70.0) * (1.5 if n >= 56 else 1.25))
    k = 0 if nc <= 27 else 1 if nc <= 47 else 2
    usual = (22, 40, 54)[k]
    per = max(1, bras // ((bras + 127) // 128))
    cost = 0 if n <= 23 and bras >= 8 else int(us[k] * 10 / 32)
    return nc <= 59 and cost * (32 + w) * 20 <= per * (110 + 9 * usual) * (29 if usual >= 32 + 2 * w else 20)


# (n, |v| of the two halves, |v| of the bras, bras)
CASES = [(50, 18, 40, 44, 19), (50, 18, 40, 44, 40), (50, 20, 42, 44, 25), (50, 10, 49, 50, 33), (50, 10, 49, 50, 31),
         (36, 27, 28, 36, 12), (36, 27, 28, 36, 20), (60, 27, 28, 60, 24), (60, 40, 59, 60, 129), (28, 5, 28, 8, 12),
         (20, 3, 20, 0, 9), (20, 3, 20, 0, 7), (54, 50, 51, 49, 33), (54, 50, 51, 49, 25), (62, 40, 61, 60, 70), (60, 12, 40, 60, 28), (50, 18, 40, 44, 15), (40, 10, 20, 5, 128)]


def test_cases_are_on_both_sides():
    """Of the halves, both, only the smaller, only the larger forms are taken."""
    kinds = {(_takes(n, bras, a + n - kb, n - kb), _takes(n, bras, b + n - kb, n - kb)) for n, a, b, kb, bras in CASES}
    assert {(True, False), (True, True), (False, True)} <= kinds


@pytest.mark.parametrize("n,ka,kk,kb,bras", CASES)
def test_mixed_sizes(B, n, ka, kk, kb, bras):  # noqa: F811
    rng = np.random.default_rng(8300 + n + bras)
    half = 33
    ca, ck, cb = _spread(n, ka, rng, 4, True), _spread(n, kk, rng, 4, True), _spread(n, kb, rng, 4, True)
    say(f"CH x CH mixed sizes n={n} |v|={ka},{kk} bras={bras} |v_b|={kb}")
    spec = [dict(circuit=c, chi=m, mode="sparsify", seed=s) for c, m, s in ((ca, 2 * half, 5), (ck, half, 6), (cb, bras, 7))]
    ctx = B.Context(spec)
    for i, c in enumerate((ca, ck, cb)):
        ctx.apply_circuit(c, inst=i)
    t = ctx.get_terms(0, half, inst=1)
    ctx.set_terms(half, t["F"], t["G"], t["M"], t["gamma"], t["v"], t["s"], t["omega"], t["b"], inst=0)
    Tb = O.Terms(cb, bras, O.SPARSIFY, seed=7)
    first = np.arange(half, dtype=np.uint64)
    ref = (O.Terms(ca, 2 * half, O.SPARSIFY, seed=5, alphas=first).inner_ch(Tb)[0] +
           O.Terms(ck, half, O.SPARSIFY, seed=6).inner_ch(Tb)[0])
    assert np.any(ref != 0)
    for _ in range(2):
        assert normwise(ctx.inner_products_ch(2, inst=0)[0], ref) < TOL64
