"""Inner products by bit-sliced elimination against the CPU oracle at the edges of
the kernels' ranges: the number of variables at which the next kernel takes over
(27 | 28, 47 | 48, 59 | 60, with none and one at the bottom), rows outside the
echelon form past 32, odd and even counts of them, states that fill a word of 32,
a batch of 128 and one more, and for two CH forms the same numbers reached with
constraints of the bra (more of them than there are slots for among them), and
the count of bras from which these kernels are taken."""
import numpy as np
import pytest

import oracle as O
from paper_1808_00128_amd import workloads as W
from test_gpu_parity import B, gpu_ctx, normwise, say  # noqa: F401

pytestmark = pytest.mark.gpu

TOL64 = 1e-12


def _spread(n, k, rng, slots, mix):
    """|v| = k for every term: Hadamards on k qubits of |0..0>, then gates and
    phase slots that leave v alone (mix: CX among them, so that columns of G have
    bits outside the k qubits' rows)."""
    ops = (W.OP_S, W.OP_CX, W.OP_CZ) if mix else (W.OP_S, W.OP_CZ)
    gates = [(W.OP_H, q, 0) for q in rng.choice(n, size=k, replace=False).tolist()]
    body = W.random_clifford_gates(n, 6 * n, rng, ops=ops) if n > 1 else [(W.OP_S, 0, 0)]
    pos = set(rng.choice(len(body), size=min(slots, len(body)), replace=False).tolist())
    for i, g in enumerate(body):
        gates.append(g)
        if i in pos:
            gates.append((W.OP_SLOT, int(rng.integers(n)), 0, float(rng.uniform(0, 2 * np.pi))))
    return W.from_list(n, gates)


@pytest.mark.parametrize("n,k,chi,L", [
    (1, 0, 1, 1), (1, 1, 2, 33), (28, 0, 9, 31), (28, 27, 40, 32), (28, 28, 70, 129), (45, 44, 33, 128),
    (45, 45, 17, 5), (48, 47, 19, 33), (50, 48, 18, 100), (59, 59, 12, 64), (60, 60, 12, 130), (61, 3, 50, 40), (62, 27, 31, 95), (63, 44, 20, 20),
    (64, 59, 9, 65), (64, 60, 9, 65), (64, 33, 16, 257)])
def test_equatorial_edges(B, n, k, chi, L):  # noqa: F811
    rng = np.random.default_rng(8100 + 64 * n + k)
    circ = _spread(n, k, rng, 5, True)
    say(f"bit-sliced inner products n={n} |v|={k} chi={chi} L={L}")
    ctx = gpu_ctx(B, dict(circuit=circ, chi=chi, mode="sparsify", seed=n + k))
    T = O.Terms(circ, chi, O.SPARSIFY, seed=n + k)
    Aoff, Adiag = W.random_equatorial(n, L, rng)
    for _ in range(2):  # the second call finds every buffer used
        ov, eta, _ = ctx.inner_products(Aoff, Adiag)
        ref, eta_ref = T.inner(Aoff, Adiag)
        assert normwise(ov, ref) < TOL64
        np.testing.assert_allclose(eta, eta_ref, rtol=1e-9, atol=1e-12 * eta_ref.max())


@pytest.mark.parametrize("n,kk,kb,chi,bras", [
    (1, 1, 0, 3, 16), (20, 12, 5, 40, 16), (20, 12, 4, 40, 7), (20, 12, 4, 40, 8), (33, 20, 25, 40, 33), (33, 20, 24, 40, 128),
    (50, 40, 46, 30, 129), (50, 40, 45, 30, 40), (50, 10, 18, 20, 40), (50, 10, 17, 20, 40), (61, 45, 47, 12, 20),
    (61, 45, 46, 12, 20), (50, 40, 43, 30, 40), (50, 40, 42, 30, 40), (64, 64, 64, 1, 1), (64, 62, 63, 8, 17)])
def test_ch_edges(B, n, kk, kb, chi, bras):  # noqa: F811
    rng = np.random.default_rng(8200 + 64 * n + kk + kb)
    ck, cb = _spread(n, kk, rng, 4, True), _spread(n, kb, rng, 4, True)
    say(f"bit-sliced CH x CH n={n} |v_k|={kk} |v_b|={kb} chi={chi} bras={bras}")
    sk, sb = (dict(circuit=c, chi=m, mode="sparsify", seed=s) for c, m, s in ((ck, chi, 5), (cb, bras, 6)))
    ctx = B.Context([sk, sb])
    ctx.apply_circuit(ck, inst=0)
    ctx.apply_circuit(cb, inst=1)
    if n == kk == kb:  # no free index for the lift
        with pytest.raises(B.ChsimError, match="EUNSUPPORTED"):
            ctx.inner_products_ch(1, inst=0)
        return
    Tk, Tb = O.Terms(ck, chi, O.SPARSIFY, seed=5), O.Terms(cb, bras, O.SPARSIFY, seed=6)
    ref, rtot = Tk.inner_ch(Tb)
    assert np.any(ref != 0)
    for _ in range(2):
        ov, tot = ctx.inner_products_ch(1, inst=0)
        assert normwise(ov, ref) < TOL64
        assert abs(tot - rtot) <= TOL64 * max(1.0, np.sqrt(np.sum(np.abs(ref) ** 2)))
