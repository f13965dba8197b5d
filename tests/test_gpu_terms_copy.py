"""Copying a term store in one launch: byte arrays whose lengths leave every kind
of tail (1 to 16 bytes, whole and partial chunks, small and large stores), with and without slots,
terms and branches equal afterwards and independent of the source."""
import numpy as np
import pytest

from paper_1808_00128_amd import workloads as W
from test_gpu_parity import B, say  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,chi,slots", [(1, 1, 0), (1, 1, 1), (3, 17, 2), (7, 1023, 3), (16, 1024, 4), (16, 1025, 1),
                                         (64, 4099, 5), (21, 16384, 2),
                                         (64, 21001, 1)])
def test_copy(B, n, chi, slots):  # noqa: F811
    rng = np.random.default_rng(300 + n + chi)
    circ = W.random_circuit(n, 6 * n + 4, rng.uniform(0, 2 * np.pi, size=slots), rng)
    say(f"terms copy n={n} chi={chi} slots={slots}")
    specs = [dict(circuit=circ, chi=chi, mode="sparsify", seed=s) for s in (1, 2)]
    ctx = B.Context(specs)
    ctx.apply_circuit(circ, inst=0)
    want = ctx.get_terms(0, chi, inst=0)
    for _ in range(2):
        ctx.copy_terms(0, 1)
        got = ctx.get_terms(0, chi, inst=1)
        assert set(got) == set(want)
        for k in want:
            assert np.array_equal(got[k], want[k]), k
        ctx.apply_circuit(circ, inst=1)  # the copy moves on (same branches), the source stays
        again = ctx.get_terms(0, chi, inst=0)
        assert all(np.array_equal(again[k], want[k]) for k in want)
    ctx.apply_circuit(circ, inst=0)
    a, b = ctx.get_terms(0, chi, inst=0), ctx.get_terms(0, chi, inst=1)
    assert all(np.array_equal(a[k], b[k]) for k in a)
    ctx.close()
