"""More work than one grid holds (a launch of 2^32 threads or more is cut short
without an error): amplitudes of more than 2^27 strings, against a call with each
string once, and inner products over more than 2^26 terms, against the sums over all
amplitudes."""
import numpy as np
import pytest
import torch

from paper_1808_00128_amd import workloads as W
from test_gpu_parity import B, gpu_ctx, say  # noqa: F401

pytestmark = pytest.mark.gpu


def test_more_strings_than_a_grid(B):  # noqa: F811
    n, chi, n_x = 3, 5, (1 << 27) + 5
    circ = W.random_circuit(n, 30, [0.3, 1.1, 2.0], np.random.default_rng(5))
    say(f"amplitudes n_x={n_x}")
    ctx = gpu_ctx(B, dict(circuit=circ, chi=chi, mode="sparsify", seed=1))
    one = torch.from_numpy(ctx.amplitudes(np.arange(8, dtype=np.uint64)).view(np.float64).reshape(8, 2)).cuda()
    x = torch.arange(n_x, dtype=torch.int64, device="cuda:0") & 7
    out = torch.full((n_x, 2), 7.0, dtype=torch.float64, device="cuda:0")
    ctx.amplitudes(x, out=out)
    torch.cuda.synchronize()
    assert bool(torch.all((out[: n_x // 8 * 8].view(-1, 8, 2) - one).abs() <= 1e-14))
    assert bool(torch.all((out[n_x // 8 * 8:] - one[: n_x % 8]).abs() <= 1e-14))


def test_more_terms_than_a_grid_of_waves(B):  # noqa: F811
    n, chi = 4, (1 << 26) + 9
    rng = np.random.default_rng(6)
    # Hadamards on two qubits only, so that |v| = 2 and the bras have constraints.
    circ = W.from_list(n, [(W.OP_H, 0, 0), (W.OP_H, 2, 0), (W.OP_SLOT, 0, 0, 0.7), (W.OP_CX, 0, 1), (W.OP_SLOT, 1, 0, 1.9),
                           (W.OP_CZ, 1, 2), (W.OP_SLOT, 2, 0, 2.3), (W.OP_CX, 2, 3), (W.OP_S, 3, 0)])
    say(f"inner products chi={chi}")
    ctx = B.Context([dict(circuit=circ, chi=chi, mode="sparsify", seed=1), dict(circuit=circ, chi=9, mode="sparsify", seed=2)])
    ctx.apply_circuit(circ, inst=0)
    ctx.apply_circuit(circ, inst=1)
    x = np.arange(16, dtype=np.uint64)
    psi = ctx.amplitudes(x)
    Aoff, Adiag = W.random_equatorial(n, 5, rng)
    bits = (x[:, None] >> np.arange(n, dtype=np.uint64)) & np.uint64(1)
    ref = []
    for off, diag in zip(Aoff, Adiag):
        A = ((off[:, None] >> np.arange(n, dtype=np.uint64)) & np.uint64(1)).astype(np.int64)
        np.fill_diagonal(A, diag)
        q = np.einsum("xa,ab,xb->x", bits.astype(np.int64), A, bits.astype(np.int64))
        ref.append(np.sum((1j ** (-q % 4)) * psi) / 4)
    # Sums of 2^26 terms in two orders: each rounds by at most 2^26 units of 2^-53.
    tol = 2.0 ** -26 * np.max(np.abs(psi))
    assert np.allclose(ctx.inner_products(Aoff, Adiag)[0], ref, rtol=0, atol=tol)
    bras = []
    bra = B.Context([dict(circuit=circ, chi=1, mode="sparsify", seed=2)])
    t = ctx.get_terms(0, 9, inst=1)
    for l in range(9):
        bra.set_terms(0, *[np.ascontiguousarray(t[k][l:l + 1]) for k in ("F", "G", "M", "gamma", "v", "s", "omega")],
                      np.ones(1, np.complex128))
        bras.append(bra.amplitudes(x))
    ov = ctx.inner_products_ch(1, inst=0)[0]
    assert np.allclose(ov, np.conj(bras) @ psi, rtol=0, atol=4 * tol)
