"""Evolution with tableau columns in registers, bit-exact against the CPU oracle
where its shapes meet: ceil(n / lanes) columns per lane at and past each
boundary, one- and two-word columns (n = 32, 33), partly filled last lanes,
waves and workgroups (4, 8 and 16 lanes per term hold 16, 8 and 4 terms per
wave), gates on both halves of a column, slots with conditional gates of every
kind (a Hadamard among them), and diagonal slots moved past the gates they
commute with, in one call and cut into segments."""
import ctypes as C

import numpy as np
import pytest

import oracle as O
from paper_1808_00128_amd import workloads as W
from test_gpu_parity import B, compare_terms, say  # noqa: F401

pytestmark = pytest.mark.gpu

LDS = 0x100


@pytest.mark.parametrize("lanes", [4 | LDS, 8 | LDS, 16 | LDS])
@pytest.mark.parametrize("n,chi", [(1, 5), (4, 64), (5, 65), (16, 17), (17, 63), (31, 33), (32, 16), (33, 257),
                                   (40, 31), (41, 66), (52, 15), (53, 70), (63, 129), (64, 40)])
def test_columns_at_the_shape_edges(B, n, chi, lanes):  # noqa: F811
    rng = np.random.default_rng(900 + n)
    circ = W.random_circuit(n, 14 * n + 20, rng.uniform(0, 2 * np.pi, size=7), rng)
    say(f"evolution columns n={n} chi={chi} lanes={lanes:#x}")
    T = O.Terms(circ, chi, O.SPARSIFY, seed=n)
    for cuts in ((), (n + 3,)):  # one call, and the state stored and loaded again
        ctx = B.Context([dict(circuit=circ, chi=chi, mode="sparsify", seed=n)])
        ctx.set_evolve_lanes(lanes)
        g = B.gate_array(circ)
        edges = [0, *cuts, g.size]
        for lo, hi in zip(edges, edges[1:]):
            ctx.apply_gates(g[lo:hi])
        compare_terms(ctx, T, np.arange(chi, dtype=np.uint64))


class _Branches:
    """A decomposition of equal weights over the given gate lists."""

    def __init__(self, B, lists):  # noqa: F811
        flat = [g for gs in lists for g in gs]
        self.coeff = (C.c_double * (2 * len(lists)))(*([0.5, 0.0] * len(lists)))
        self.off = (C.c_uint32 * (len(lists) + 1))(*np.cumsum([0] + [len(gs) for gs in lists]).tolist())
        self.gates = (B.Gate * max(1, len(flat)))(*[B.Gate(op, q, r, 0, 0) for op, q, r in flat])
        self.decomp = B.Decomp(len(lists), self.coeff, self.off, self.gates)


@pytest.mark.parametrize("lanes", [0, 4 | LDS, 8 | LDS, 16 | LDS, 64])
@pytest.mark.parametrize("n", [6, 37])
def test_general_slot_branches(B, monkeypatch, n, lanes):  # noqa: F811
    """Branches of Hadamards, CX, CZ and S: the gates are conditional per term."""
    rng = np.random.default_rng(n)
    circ = W.random_circuit(n, 160, [0.1] * 6, rng)
    lists = [[W.random_clifford_gates(n, int(rng.integers(0, 6)), rng) for _ in range(3)] for _ in range(6)]
    lists[2] = [[(W.OP_S, 1, 0)], [(W.OP_CZ, 1, n - 1)], []]  # diagonal: net gates, moved as late as they commute
    decs = [_Branches(B, gs) for gs in lists]
    monkeypatch.setattr(B, "slot_decompositions", lambda c: decs)
    chi = 70
    say(f"general branches n={n} lanes={lanes:#x}")
    ctx = B.Context([dict(circuit=circ, chi=chi, mode="sparsify", seed=4)])
    ctx.set_evolve_lanes(lanes)
    ctx.apply_circuit(circ)
    got = ctx.get_terms(0, chi)
    for a in range(chi):
        ch, k = O.CHForm(n), 0
        for op, q, r, _ in circ.gates():
            if op == W.OP_SLOT:
                for g in lists[k][int(got["branch"][a, k])]:
                    ch.apply(*g)
                k += 1
            else:
                ch.apply(op, q, r)
        want = ch.export()
        for f in ("F", "G", "M", "gamma"):
            assert np.array_equal(got[f][a], want[f]), (f, a)
        for f in ("v", "s", "omega"):
            assert int(got[f][a]) == want[f], (f, a)


@pytest.mark.parametrize("share", [0, 2])
def test_deferred_diagonal_slots(B, share):  # noqa: F811
    """Slots before, between and right at the gates that stop them (a Hadamard
    on, a CX into one of their qubits), several on one qubit, CCZ among them."""
    n = 7
    H, S, CX, CZ, SL, CCZ = W.OP_H, W.OP_S, W.OP_CX, W.OP_CZ, W.OP_SLOT, W.OP_CCZ
    gates = [(H, q, 0) for q in range(n)]
    gates += [(SL, 0, 0, 0.3), (CX, 0, 1), (CZ, 0, 2), (S, 0, 0), (SL, 0, 0, 2.1), (SL, 1, 0, 1.0), (CX, 2, 0),
              (CCZ, 3, 4, 5), (CX, 3, 1), (H, 6, 0), (CX, 1, 4), (CCZ, 0, 3, 6), (SL, 5, 0, 4.0), (H, 5, 0), (SL, 2, 0, 0.7),
              (CX, 2, 6), (H, 3, 0), (S, 2, 0), (CZ, 2, 5), (H, 0, 0), (SL, 6, 0, 5.0)]
    circ = W.from_list(n, gates)
    chi = 300
    say(f"deferred slots share={share}")
    ctx = B.Context([dict(circuit=circ, chi=chi, mode="sparsify", seed=8)])
    ctx.set_prefix_share(share)
    ctx.apply_circuit(circ)
    compare_terms(ctx, O.Terms(circ, chi, O.SPARSIFY, seed=8), np.arange(chi, dtype=np.uint64))
