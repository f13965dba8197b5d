"""What this framework is timed on: the calls that a program makes through
`paper_1808_00128_amd.binding`, over the range of sizes they are made at.

listed() and draw() give the cases, prepare() what a program has in hand before
the call, run() one pass, work() the bytes and operations a pass cannot do
without, and exact() the same outputs in 64 bits from plain torch (CH forms
evolved gate by gate, amplitudes summed term by term, dense state vectors
where n is small), with none of the library's code.

Kinds:
  step      redraw the terms, evolve them through the circuit, evaluate
            amplitudes: one pass of the hot path, as bench.py times it;
  amps      amplitudes of a few or of many strings on terms that are evolved;
  batch     amplitudes of several uneven instances in one call;
  norm      norm estimation with random equatorial states;
  marginal  chain-rule sampling of output bits (projections and norms);
  overlaps  inner products with stabilizer states given as CH forms;
  chains    Metropolis steps with single flips;
  learned   Metropolis steps with the learned flip-mask proposal;
  train     loss and gradients of the proposal network.
"""
import math

import numpy as np
import torch

from paper_1808_00128_amd import binding as B
from paper_1808_00128_amd import workloads as W

DEV = "cuda:0"


# ---------------------------------------------------------------------------
# Cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # The smallest call: the n = 12 exact sum over 8 T gates, every string.
        dict(name="tiny-exact", kind="step", circuit="random", n=12, gates=200, slots=8, chi=256, mode="exact",
             n_x=4096, fp32c=False),
        # The benchmark's step: n = 50, 2000 gates, 40 phase slots, FP32C sums.
        dict(name="step-n50", kind="step", circuit="random", n=50, gates=2000, slots=40, chi=65536, mode="sparsify",
             n_x=4096, fp32c=True),
        # Hidden shift with CCZ: terms near basis states, strings drawn from them.
        dict(name="step-ccz-n40", kind="step", circuit="ccz", n=40, gates=0, slots=16, chi=110610, mode="sparsify",
             n_x=4096, fp32c=False),
        # A few amplitudes of a large, ragged term set (a serving call).
        dict(name="amps-few-n57", kind="amps", circuit="random", n=57, gates=1140, slots=35, chi=200003,
             mode="sparsify", n_x=33, fp32c=True),
        # Several circuits of different n and chi in one call, odd counts.
        dict(name="batch-uneven", kind="batch", inst=9, n_lo=20, n_hi=60, chi_lo=1024, chi_hi=65536, n_x=1000,
             fp32c=False),
        # Norm estimation at the paper's scale: chi = 2^18, 1024 equatorial states.
        dict(name="norm-n40", kind="norm", n=40, gates=200, slots=30, chi=262144, L=1024),
        # Chain-rule sampling of four bits on a small odd instance.
        dict(name="marginal-n20", kind="marginal", n=20, gates=300, slots=14, chi=3001, L=100, w=4),
        # Overlaps of a term set with 256 stabilizer states.
        dict(name="overlaps-n40", kind="overlaps", n=40, gates=200, slots=30, chi=65536, bras=256),
        # Chains at the QAOA workload's size, one flip bit per step for all chains.
        dict(name="chains-n50", kind="chains", n=50, triples=60, chi=1048576, chains=64, steps=100, shared=True,
             host=False),
        # Chains started and run from host arrays on a small instance, own flip bits.
        dict(name="chains-n12", kind="chains", n=12, triples=16, chi=65536, chains=64, steps=200, shared=False,
             host=True),
        # Learned proposal on the QAOA instance.
        dict(name="learned-n50", kind="learned", n=50, triples=60, chi=262144, chains=64, steps=24, hidden=256),
        # One training step of the proposal network (forward and backward).
        dict(name="train-n50", kind="train", n=50, hidden=256, rows=1024),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "ccz", "amps", "amps", "batch", "norm", "norm", "marginal", "overlaps",
                       "overlaps", "chains", "chains", "learned", "train"])
    if kind == "step":
        n = rng.randint(9, 60)
        return dict(kind="step", circuit="random", n=n, gates=rng.randint(8 * n, 40 * n), slots=rng.randint(8, 45),
                    chi=_log_int(rng, 300, 70000), mode="sparsify", n_x=_log_int(rng, 100, 5000),
                    fp32c=rng.random() < 0.5)
    if kind == "ccz":
        n = 2 * rng.randint(6, 24)
        return dict(kind="step", circuit="ccz", n=n, gates=0, slots=2 * rng.randint(3, 8),
                    chi=_log_int(rng, 1000, 110610), mode="sparsify", n_x=_log_int(rng, 100, 4096),
                    fp32c=rng.random() < 0.5)
    if kind == "amps":
        n = rng.randint(9, 64)
        return dict(kind="amps", circuit="random", n=n, gates=rng.randint(8 * n, 30 * n), slots=rng.randint(8, 45),
                    chi=_log_int(rng, 1000, 200003), mode="sparsify", n_x=_log_int(rng, 1, 2000),
                    fp32c=rng.random() < 0.5)
    if kind == "batch":
        return dict(kind="batch", inst=rng.randint(3, 12), n_lo=20, n_hi=60, chi_lo=1000,
                    chi_hi=_log_int(rng, 2000, 65536), n_x=_log_int(rng, 50, 1500), fp32c=rng.random() < 0.5)
    if kind == "norm":
        n = rng.randint(12, 50)
        return dict(kind="norm", n=n, gates=rng.randint(4 * n, 20 * n), slots=rng.randint(8, 35),
                    chi=_log_int(rng, 500, 60000), L=_log_int(rng, 30, 1000))
    if kind == "marginal":
        n = rng.randint(10, 24)
        return dict(kind="marginal", n=n, gates=rng.randint(5 * n, 15 * n), slots=rng.randint(8, 20),
                    chi=_log_int(rng, 500, 6000), L=_log_int(rng, 50, 300), w=rng.randint(2, 6))
    if kind == "overlaps":
        n = rng.randint(12, 50)
        return dict(kind="overlaps", n=n, gates=rng.randint(4 * n, 20 * n), slots=rng.randint(8, 35),
                    chi=_log_int(rng, 500, 65536), bras=_log_int(rng, 7, 256))
    if kind == "chains":
        return dict(kind="chains", n=rng.randint(12, 50), triples=rng.randint(14, 60), chi=_log_int(rng, 4000, 600000),
                    chains=rng.choice([8, 33, 64, 100]), steps=rng.randint(11, 120), shared=rng.random() < 0.5,
                    host=rng.random() < 0.5)
    if kind == "learned":
        return dict(kind="learned", n=rng.randint(12, 50), triples=rng.randint(14, 60),
                    chi=_log_int(rng, 4000, 262144), chains=rng.choice([8, 33, 64]), steps=rng.randint(5, 30),
                    hidden=rng.choice([128, 256]))
    return dict(kind="train", n=rng.randint(12, 60), hidden=rng.choice([128, 256, 512]), rows=_log_int(rng, 200, 4000))


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
def _rng(seed, tag):
    return np.random.default_rng([int(seed), tag])


def _circuit(case, rng):
    """(circuit, the string a hidden-shift circuit prepares or None)."""
    n = case["n"]
    if case.get("circuit") == "ccz":
        circ, s = W.hidden_shift_circuit(n, case["slots"], rng)
        return circ, s
    if case.get("mode") == "exact":
        thetas = [np.pi / 4] * case["slots"]
    else:
        thetas = rng.uniform(0.0, 2 * np.pi, size=case["slots"])
    return W.random_circuit(n, case["gates"], thetas, rng), None


def _spec(circ, chi, seed, mode="sparsify"):
    return dict(circuit=circ, chi=chi, mode=mode, seed=int(seed) * 7919 + 13)


def _to_gpu(x):
    return torch.from_numpy(np.ascontiguousarray(x).view(np.int64)).to(DEV)


def _batch_specs(case, seed):
    rng = _rng(seed, 5)
    specs, xs = [], []
    for k in range(case["inst"]):
        n = int(rng.integers(case["n_lo"], case["n_hi"] + 1))
        chi = int(round(np.exp(rng.uniform(np.log(case["chi_lo"]), np.log(case["chi_hi"])))))
        circ = W.random_circuit(n, 10 * n, rng.uniform(0, 2 * np.pi, size=int(rng.integers(10, 41))), rng)
        specs.append(_spec(circ, chi, seed * 100 + k))
        xs.append(W.random_bitstrings(n, case["n_x"], rng))
    return specs, xs


def _qaoa(case, seed):
    """The QAOA circuit on the line beta = pi/4, gamma = 0.35, as bench.py runs it."""
    rng = _rng(seed, 6)
    triples = min(case["triples"], math.comb(case["n"], 3))
    return W.qaoa_circuit(case["n"], triples, rng, gamma=0.35, beta=np.pi / 4)[0]


def _starts(ctx, n, chi, count, rng):
    """Chain starts: strings sampled from single terms, of non-zero amplitude."""
    xs = []
    while len(xs) < count:
        cand = ctx.sample_terms(rng.integers(0, chi, size=2 * count), W.random_bitstrings(n, 2 * count, rng))
        amp = ctx.amplitudes(cand)
        xs += [int(x) for x, a in zip(cand, amp) if abs(a) > 0]
    return np.array(xs[:count], np.uint64)


def _equatorial(n, L, rng):
    """L uniform matrices A of M_n, as W.random_equatorial lays them out."""
    up = np.triu(rng.integers(0, 2, size=(L, n, n), dtype=np.uint8), 1)
    bits = (up | up.transpose(0, 2, 1)).astype(np.uint64)
    off = (bits << np.arange(n, dtype=np.uint64)[None, None, :]).sum(axis=2, dtype=np.uint64)
    return off, rng.integers(0, 4, size=(L, n), dtype=np.uint8)


def _chain_streams(case, seed):
    return W.metropolis_streams(case["n"], case["chains"], case["steps"], _rng(seed, 8), shared_j=case["shared"])


def _train_data(case, seed):
    rng = _rng(seed, 9)
    n = case["n"]
    params = W.mlp_init(n, case["hidden"], seed=int(seed) % 100003)
    x = W.random_bitstrings(n, case["rows"], rng)
    flips = (rng.random((case["rows"], n)) < 0.15).astype(np.uint64)  # a chain's move over a correlation time
    return params, x, (flips << np.arange(n, dtype=np.uint64)[None, :]).sum(axis=1, dtype=np.uint64)


def prepare(case, seed):
    kind = case["kind"]
    st = dict(case=case, kind=kind)
    if kind in ("step", "amps"):
        rng = _rng(seed, 1)
        circ, s = _circuit(case, rng)
        spec = _spec(circ, case["chi"], seed, case["mode"])
        ctx = B.Context([spec])
        st.update(ctx=ctx, gates=B.gate_array(circ), seed=spec["seed"])
        if s is not None:
            # The hidden string and strings of the terms' own distributions
            # (uniform ones would have amplitude zero for nearly every term).
            ctx.apply_gates(st["gates"])
            alpha, flips = _ccz_picks(case, rng)
            x = np.concatenate([np.array([s], np.uint64), ctx.sample_terms(alpha, flips)])
        elif case["mode"] == "exact":
            x = rng.permutation(2 ** case["n"])[:case["n_x"]].astype(np.uint64)
        else:
            x = W.random_bitstrings(case["n"], case["n_x"], rng)
        if kind == "amps":
            ctx.apply_gates(st["gates"])
        st.update(x=_to_gpu(x), out=torch.empty((x.size, 2), dtype=torch.float64, device=DEV))
    elif kind == "batch":
        specs, xs = _batch_specs(case, seed)
        ctx = B.Context(specs)
        for k, sp in enumerate(specs):
            ctx.apply_circuit(sp["circuit"], inst=k)
        st.update(ctx=ctx, reqs=[(k, _to_gpu(x)) for k, x in enumerate(xs)])
    elif kind in ("norm", "marginal"):
        circ = _circuit(case, _rng(seed, 2))[0]
        spec = _spec(circ, case["chi"], seed)
        ctx = B.Context([spec] if kind == "norm" else [spec, spec])
        ctx.apply_circuit(circ)
        rng = _rng(seed, 3)
        off, diag = _equatorial(case["n"], case["L"], rng)
        st.update(ctx=ctx, off=off, diag=diag)
        if kind == "marginal":
            st.update(qubits=rng.permutation(case["n"])[:case["w"]].astype(np.uint32), u=rng.random(case["w"]))
    elif kind == "overlaps":
        ck, cb = _overlap_circuits(case, seed)
        ctx = B.Context([_spec(ck, case["chi"], seed), _spec(cb, case["bras"], seed + 1)])
        ctx.apply_circuit(ck, inst=0)
        ctx.apply_circuit(cb, inst=1)
        st.update(ctx=ctx)
    elif kind in ("chains", "learned"):
        circ = _qaoa(case, seed)
        ctx = B.Context([_spec(circ, case["chi"], seed)])
        ctx.apply_circuit(circ)
        x0 = _starts(ctx, case["n"], case["chi"], case["chains"], _rng(seed, 7))
        st.update(ctx=ctx, x0=x0)
        shape = (case["chains"], case["steps"])
        if kind == "chains":
            st["j"], st["u"] = _chain_streams(case, seed)
        else:
            um, j, ub, u = W.learned_streams(case["n"], *shape, _rng(seed, 8))
            st["net"] = B.MLP(ctx, case["n"], case["hidden"], max(64, case["chains"]),
                              W.mlp_init(case["n"], case["hidden"], seed=int(seed) % 100003))
            st["streams"] = (torch.from_numpy(um).to(DEV), torch.from_numpy(j.astype(np.int32)).to(DEV),
                             torch.from_numpy(ub).to(DEV), torch.from_numpy(u).to(DEV))
        if kind == "learned" or not case["host"]:
            ctx.metropolis_init(x0)
            if kind == "chains":
                st["j"] = torch.from_numpy(st["j"].astype(np.int32)).to(DEV)
                st["u"] = torch.from_numpy(st["u"]).to(DEV)
            st.update(trace=torch.empty(shape, dtype=torch.int64, device=DEV),
                      acc=torch.empty(shape, dtype=torch.uint8, device=DEV),
                      flips=torch.empty(shape, dtype=torch.int32, device=DEV),
                      amp=torch.empty((case["chains"], 2), dtype=torch.float64, device=DEV))
    else:
        params, x, t = _train_data(case, seed)
        # The network lives on a context's GPU; a program has one with its circuit.
        circ = W.random_circuit(case["n"], 10, [0.1], _rng(seed, 4))
        ctx = B.Context([_spec(circ, 16, seed)])
        st.update(ctx=ctx, net=B.MLP(ctx, case["n"], case["hidden"], case["rows"], params), x=x, t=t)
    return st


def _ccz_picks(case, rng):
    alpha = rng.integers(0, case["chi"], size=case["n_x"] - 1).astype(np.uint64)
    return alpha, W.random_bitstrings(case["n"], case["n_x"] - 1, rng)


def _overlap_circuits(case, seed):
    n = case["n"]
    rng = _rng(seed, 11)
    ck = W.random_circuit(n, case["gates"], rng.uniform(0, 2 * np.pi, size=case["slots"]), rng)
    cb = W.random_circuit(n, 10 * n, rng.uniform(0, 2 * np.pi, size=30), rng)
    return ck, cb


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------
def run(st):
    kind, case = st["kind"], st["case"]
    ctx = st["ctx"]
    if kind == "step":
        ctx.reset(st["seed"])
        ctx.apply_gates(st["gates"])
        return ctx.amplitudes(st["x"], fp32c=case["fp32c"], out=st["out"])
    if kind == "amps":
        return ctx.amplitudes(st["x"], fp32c=case["fp32c"], out=st["out"])
    if kind == "batch":
        return ctx.amplitudes_batch(st["reqs"], fp32c=case["fp32c"])
    if kind == "norm":
        ov, eta, mean = ctx.inner_products(st["off"], st["diag"])
        return {"overlap": ov, "eta": eta, "mean": mean}
    if kind == "marginal":
        bits, prob, est = ctx.sample_marginal(st["qubits"], st["off"], st["diag"], st["u"])
        return {"bits": bits, "prob": prob, "est": est}
    if kind == "overlaps":
        ov, tot = ctx.inner_products_ch(1, inst=0)
        return {"overlap": ov, "total": np.array([tot])}
    if kind == "chains":
        if case["host"]:
            ctx.metropolis_init(st["x0"])
            tr, acc, amp = ctx.metropolis_step(st["j"], st["u"])
            return {"trace": tr.view(np.int64), "accepted": acc, "amp": amp}
        ctx.metropolis_step_device(st["j"], st["u"], st["trace"], st["acc"], st["amp"])
        return {"trace": st["trace"], "accepted": st["acc"], "amp": st["amp"]}
    if kind == "learned":
        ctx.metropolis_step_learned_device(st["net"], *st["streams"], 0.1, 0.002, 0.5, st["trace"], st["acc"],
                                           st["flips"])
        return {"trace": st["trace"], "accepted": st["acc"], "flips": st["flips"]}
    loss, grads = st["net"].loss_grad(st["x"], st["t"])
    return {"loss": loss, "grads": grads}


# ---------------------------------------------------------------------------
# Work of one pass: bytes read and written once, and operations (32-bit
# integer operations on bit-packed rows, or multiply-adds counted twice for
# the network) of the method's formulas.
# ---------------------------------------------------------------------------
def _term_bytes(n, chi):
    return float(chi) * (25 * n + 33)  # rows of F, G, M and gamma; v, s, omega, b


def _evolve_work(n, chi, gates, slots):
    h = gates / 4.0
    return float(chi) * (h * 35 * n + (gates - h + slots) * 10)


def _amp_work(n, chi, n_x):
    return float(chi) * n_x * (3 * n + 20)  # 6 per set bit of a uniform string, 20 for the test and the phase


def work(case):
    k, n = case["kind"], case["n"] if "n" in case else 40
    if k == "step":
        gates = case["gates"] if case["circuit"] == "random" else 8 * n
        return dict(bytes=_term_bytes(n, case["chi"]) + case["chi"] * case["slots"] + 24.0 * case["n_x"],
                    flops=_evolve_work(n, case["chi"], gates, case["slots"]) + _amp_work(n, case["chi"], case["n_x"]))
    if k == "amps":
        return dict(bytes=_term_bytes(n, case["chi"]) + 24.0 * case["n_x"], flops=_amp_work(n, case["chi"], case["n_x"]))
    if k == "batch":
        chi = (case["chi_hi"] - case["chi_lo"]) / math.log(case["chi_hi"] / case["chi_lo"])  # mean of the law
        return dict(bytes=case["inst"] * (_term_bytes(n, chi) + 24.0 * case["n_x"]),
                    flops=case["inst"] * _amp_work(n, chi, case["n_x"]))
    if k in ("norm", "marginal"):
        times = 1 if k == "norm" else 2 * case["w"]
        pairs = float(case["chi"]) * case["L"]
        return dict(bytes=times * (_term_bytes(n, case["chi"]) + case["L"] * (9.0 * n + 24)),
                    flops=times * pairs * (6 * n * n + 2 * (0.62 * n + 1) ** 2))
    if k == "overlaps":
        pairs = float(case["chi"]) * case["bras"]
        return dict(bytes=_term_bytes(n, case["chi"] + case["bras"]) + 16.0 * case["bras"],
                    flops=pairs * 2 * (2 * n * n + 3 * (0.62 * n + 1) ** 2))
    if k == "chains":
        # Per chain and step: the cached word read and written, row j once per step.
        per = 16.0 * case["chains"] + 17 * (1 if case["shared"] else min(n, case["chains"])) + 33
        return dict(bytes=case["steps"] * case["chi"] * per, flops=40.0 * case["steps"] * case["chi"] * case["chains"])
    if k == "learned":
        per = 17.0 * n + 16 * case["chains"] + 33
        h = case["hidden"]
        return dict(bytes=case["steps"] * case["chi"] * per,
                    flops=case["steps"] * (100.0 * case["chi"] * case["chains"] +
                                           4.0 * case["chains"] * (2 * n * h + h * h)))
    h, r = case["hidden"], case["rows"]
    p = 2 * n * h + h * h
    return dict(bytes=8.0 * p + 16.0 * r, flops=6.0 * r * p)


# ---------------------------------------------------------------------------
# The same outputs in 64 bits, in plain torch: the circuit's Clifford branches
# drawn as the interface documents, CH forms (F, G, M, gamma, v, s, omega)
# updated rule by rule for all terms at once (rows [n, chi] of int64 words),
# amplitudes by right multiplication of the Paulis of x's set bits.
# ---------------------------------------------------------------------------
_M32 = 0xFFFFFFFF


def _par(x):
    for sh in (32, 16, 8, 4, 2, 1):
        x = x ^ (x >> sh)
    return x & 1


def _pop(x):
    x = x - ((x >> 1) & 0x5555555555555555)
    x = (x & 0x3333333333333333) + ((x >> 2) & 0x3333333333333333)
    x = (x + (x >> 4)) & 0x0F0F0F0F0F0F0F0F
    x = x + (x >> 8)
    x = x + (x >> 16)
    return (x + (x >> 32)) & 0x7F


def _lowest(x):
    return x & -x


def _philox_uniform(seed, alpha, slot):
    """53-bit uniforms of Philox4x32-10, counter (alpha, slot, tag), key seed."""
    c = [alpha & _M32, (alpha >> 32) & _M32, torch.full_like(alpha, slot), torch.full_like(alpha, 0x53504152)]
    k0, k1 = seed & _M32, (seed >> 32) & _M32
    for r in range(10):
        if r:
            k0, k1 = (k0 + 0x9E3779B9) & _M32, (k1 + 0xBB67AE85) & _M32
        p0, p1 = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57
        c = [((p1 >> 32) & _M32) ^ c[1] ^ k0, p1 & _M32, ((p0 >> 32) & _M32) ^ c[3] ^ k1, p0 & _M32]
    return ((c[0] << 21) | (c[1] >> 11)).to(torch.float64) / 9007199254740992.0


def _slots(circ):
    """Per slot: the branches' coefficients and gate lists [(S, q, power) | (CZ, a, b)]."""
    out, third = [], circ.third()
    for o, q, r, t in zip(circ.op.tolist(), circ.q.tolist(), circ.r.tolist(), third.tolist()):
        if o == W.OP_SLOT:
            theta = float(circ.theta[len(out)])
            k = math.floor(theta / (math.pi / 2))
            h = (theta - k * math.pi / 2) / 2
            e = complex(math.cos(h), math.sin(h))
            out.append(([e * (math.cos(h) - math.sin(h)), e * (1 - 1j) * math.sin(h)],
                        [[("S", q, k % 4)], [("S", q, (k + 1) % 4)]]))
        elif o == W.OP_CCZ:
            ab, ac, bc = ("CZ", q, r), ("CZ", q, t), ("CZ", r, t)
            za, zb, zc = ("S", q, 2), ("S", r, 2), ("S", t, 2)
            out.append(([1 / 6] * 7 + [-1 / 6],
                        [[], [ab], [ac], [bc], [ab, ac, za], [ab, bc, zb], [ac, bc, zc], [ab, ac, bc, za, zb, zc]]))
    return out


class _Terms:
    def __init__(self, spec):
        circ, chi = spec["circuit"], spec["chi"]
        n = self.n = circ.n
        slots = _slots(circ)
        alpha = torch.arange(chi, device=DEV)
        b = torch.full((chi,), 1.0, dtype=torch.complex128, device=DEV)
        branch = []
        radix = 1
        for p, (c, _) in enumerate(slots):
            w = [abs(z) for z in c]
            if spec["mode"] == "exact":
                j = (alpha // radix) % len(c)
                radix *= len(c)
                b = b * torch.tensor(c, dtype=torch.complex128, device=DEV)[j]
            else:
                cum = torch.tensor(np.cumsum(w), dtype=torch.float64, device=DEV)
                j = (_philox_uniform(spec["seed"], alpha, p) * cum[-1])[:, None].ge(cum[None, :-1]).sum(1)
                unit = [z / x if x > 0 else 0.0 for z, x in zip(c, w)]
                b = b * sum(w) * torch.tensor(unit, dtype=torch.complex128, device=DEV)[j]
            branch.append(j)
        self.b = b if spec["mode"] == "exact" else b / chi
        eye = torch.ones(n, dtype=torch.int64, device=DEV) << torch.arange(n, device=DEV)
        self.F, self.G = eye[:, None].repeat(1, chi), eye[:, None].repeat(1, chi)
        self.M = torch.zeros((n, chi), dtype=torch.int64, device=DEV)
        self.g = torch.zeros((n, chi), dtype=torch.int64, device=DEV)
        self.v, self.s, self.w = (torch.zeros(chi, dtype=torch.int64, device=DEV) for _ in range(3))
        k = 0
        for o, q, r in zip(circ.op.tolist(), circ.q.tolist(), circ.r.tolist()):
            if o == W.OP_H:
                self._hadamard(q)
            elif o == W.OP_S:
                self._left(("S", q, 1), None)
            elif o == W.OP_CZ:
                self._left(("CZ", q, r), None)
            elif o == W.OP_CX:
                self.g[q] = (self.g[q] + self.g[r] + 2 * _par(self.M[q] & self.F[r])) & 3
                self.G[r] ^= self.G[q]
                self.F[q] ^= self.F[r]
                self.M[q] ^= self.M[r]
            else:
                for j, gates in enumerate(slots[k][1]):
                    on = -(branch[k] == j).to(torch.int64)
                    for g in gates:
                        self._left(g, on)
                k += 1

    def _left(self, gate, on):
        op, q, r = gate
        if op == "CZ":
            gq, gr = self.G[q].clone(), self.G[r].clone()
            self.M[q] ^= gr if on is None else gr & on
            self.M[r] ^= gq if on is None else gq & on
        elif r & 3:
            if r & 1:
                self.M[q] ^= self.G[q] if on is None else self.G[q] & on
            self.g[q] = (self.g[q] - (r if on is None else r * -on)) & 3

    def _hadamard(self, p):
        F, G, M, v, s = self.F, self.G, self.M, self.v, self.s
        Fp, Gp, Mp = F[p].clone(), G[p].clone(), M[p].clone()
        t = s ^ (Gp & v)
        u = s ^ (Fp & ~v) ^ (Mp & v)
        alpha = _par(Gp & ~v & s)
        beta = _par((Mp & ~v & s) ^ (Fp & v & (Mp ^ s)))
        delta = (self.g[p] + 2 * (alpha + beta)) & 3
        d = t ^ u
        same = d == 0
        V0, V1 = d & ~v, d & v
        use0 = V0 != 0
        X = torch.where(use0, V0, V1)
        eq = torch.where(same, 0, _lowest(X))
        Wm = X & ~eq
        tq, vq = (t & eq) != 0, (v & eq) != 0
        # H^{v_q}(|y_q> + i^delta |1 - y_q>) as 2^{1/2} e^{i pi dw/4} S^a H^b |c>.
        dp = torch.where(tq, (4 - delta) & 3, delta)
        ph = torch.where(tq, 2 * delta, 0)
        a = dp & 1
        b = torch.where(vq, dp & 1, 1)
        c = torch.where(vq, ((dp == 1) | (dp == 2)).to(torch.int64), dp >> 1)
        dw = ph + torch.where(vq, torch.where(dp == 1, 1, torch.where(dp == 3, 7, 0)), 0)
        a = torch.where(same, 0, a)
        dw = torch.where(same, torch.where(delta == 1, 1, 7), dw)
        # V_C on the rows: R[CX] of the batch, then R[CZ] and R[S_q].
        W1, W0 = torch.where(use0, 0, Wm), torch.where(use0, Wm, 0)
        e1, e0 = torch.where(use0, 0, eq), torch.where(use0, eq, 0)
        V10 = torch.where(use0, V1, 0)
        fq, gq, mq = -((F & eq) != 0).to(torch.int64), -((G & eq) != 0).to(torch.int64), -((M & eq) != 0).to(torch.int64)
        pf = -_par(F & torch.where(use0, V1, Wm))
        pg, pm = -_par(G & W0), -_par(M & W0)
        nG = G ^ (W1 & gq) ^ (e0 & pg)
        nM = M ^ (W1 & mq) ^ (e0 & (pf ^ pm)) ^ (V10 & fq)
        nF = F ^ (e1 & pf) ^ (W0 & fq)
        g = self.g + 2 * (fq & pf & -(use0.to(torch.int64)) & 1)
        fq2 = ((nF & eq) != 0).to(torch.int64) * a
        self.F, self.G, self.M = nF, nG, nM ^ (eq & -fq2)
        self.g = (g - fq2) & 3
        y = torch.where(tq, u ^ eq, t)
        self.s = torch.where(same, t, (y & ~eq) | torch.where(c != 0, eq, 0))
        self.v = torch.where(same, v, (v & ~eq) | torch.where(b != 0, eq, 0))
        self.w = (self.w + 4 * alpha + dw) & 7

    def amplitudes(self, x):
        """<x|psi> for an int64 tensor x of strings."""
        chi, n = self.v.numel(), self.n
        out = torch.empty(x.numel(), dtype=torch.complex128, device=DEV)
        scale = self.b * torch.pow(2.0, -0.5 * _pop(self.v).to(torch.float64))
        root = torch.exp(1j * math.pi / 4 * torch.arange(8, dtype=torch.float64, device=DEV))
        step = max(1, (1 << 26) // chi)
        for i in range(0, x.numel(), step):
            xs = x[i:i + step, None]
            u = torch.zeros((xs.shape[0], chi), dtype=torch.int64, device=DEV)
            acc, mu = torch.zeros_like(u), torch.zeros_like(u)
            for p in range(n):
                on = -((xs >> p) & 1)
                u ^= self.F[p] & on
                acc ^= u & self.M[p] & on
                mu += self.g[p] & on
            k = (self.w + 2 * mu + 4 * (_par(acc) + _par(u & (self.v & self.s)))) & 7
            val = root[k] * scale
            val[((u ^ self.s) & ~self.v) != 0] = 0
            out[i:i + step] = val.sum(1)
        return out

    def sample(self, alpha, flips):
        """One string per (term, word of uniform bits): w = s, flipped on v by the word, x = w G^T."""
        a = torch.from_numpy(alpha.astype(np.int64)).to(DEV)
        w = self.s[a] ^ (self.v[a] & torch.from_numpy(flips.view(np.int64)).to(DEV))
        return sum((_par(self.G[p][a] & w) << p) for p in range(self.n))


def _pairs(z):
    return torch.view_as_real(z.resolve_conj().contiguous()).cpu()


def _equatorial_rows(n, off, diag, x):
    """conj(phi_A(x)) = 2^{-n/2} i^{-x A x^T} for one A and all strings x."""
    q = torch.zeros_like(x)
    for p in range(n):
        bit = (x >> p) & 1
        upper = int(off[p]) >> (p + 1) << (p + 1)
        q += bit * (int(diag[p]) + 2 * _par(x & upper))
    return torch.tensor([1, -1j, -1, 1j], dtype=torch.complex128, device=DEV)[q & 3] * 2.0 ** (-n / 2)


def _dense_etas(n, psi, off, diag):
    x = torch.arange(2 ** n, device=DEV)
    return torch.stack([torch.dot(_equatorial_rows(n, off[l], diag[l], x), psi) for l in range(off.shape[0])])


def _exact_chains(case, seed):
    circ = _qaoa(case, seed)
    T = _Terms(_spec(circ, case["chi"], seed))
    n, C, steps = case["n"], case["chains"], case["steps"]
    # The starts are drawn from the terms and kept where their amplitude is not zero.
    rng = _rng(seed, 7)
    xs = []
    while len(xs) < C:
        alpha = rng.integers(0, case["chi"], size=2 * C)
        cand = T.sample(alpha.astype(np.uint64), W.random_bitstrings(n, 2 * C, rng))
        amp = T.amplitudes(cand)
        xs += [int(v) for v, z in zip(cand.tolist(), amp.tolist()) if abs(z) > 1e-14]
    x = torch.tensor(xs[:C], device=DEV)
    j, u = _chain_streams(case, seed)
    j, u = torch.from_numpy(j.astype(np.int64)).to(DEV), torch.from_numpy(u).to(DEV)
    amp = T.amplitudes(x)
    for t in range(steps):
        y = x ^ (torch.ones_like(x) << j[:, t])
        ay = T.amplitudes(y)
        ok = u[:, t] < ay.abs().square() / amp.abs().square()
        x, amp = torch.where(ok, y, x), torch.where(ok, ay, amp)
    return amp


def _exact_train(case, seed):
    params, x, t = _train_data(case, seed)
    n = case["n"]
    P = {k: torch.from_numpy(v).to(DEV, torch.float64).requires_grad_() for k, v in params.items()}
    sh = torch.arange(n, device=DEV)
    bits = ((_to_gpu(x)[:, None] >> sh) & 1).to(torch.float64)
    tgt = ((_to_gpu(t)[:, None] >> sh) & 1).to(torch.float64)
    h = torch.relu((1 - 2 * bits) @ P["W1"].T + P["b1"])
    h = torch.relu(h @ P["W2"].T + P["b2"])
    loss = torch.nn.functional.binary_cross_entropy_with_logits(h @ P["W3"].T + P["b3"], tgt)
    loss.backward()
    return {"loss": float(loss), "grads": {k: v.grad for k, v in P.items()}}


def exact(case, seed):
    kind = case["kind"]
    if kind in ("step", "amps"):
        rng = _rng(seed, 1)
        circ, s = _circuit(case, rng)
        T = _Terms(_spec(circ, case["chi"], seed, case["mode"]))
        if s is not None:
            alpha, flips = _ccz_picks(case, rng)
            x = torch.cat([torch.tensor([s], device=DEV), T.sample(alpha, flips)])
        elif case["mode"] == "exact":
            x = torch.from_numpy(rng.permutation(2 ** case["n"])[:case["n_x"]].astype(np.int64)).to(DEV)
        else:
            x = _to_gpu(W.random_bitstrings(case["n"], case["n_x"], rng))
        return _pairs(T.amplitudes(x))
    if kind == "batch":
        specs, xs = _batch_specs(case, seed)
        return [_pairs(_Terms(sp).amplitudes(_to_gpu(x))) for sp, x in zip(specs, xs)]
    if kind in ("norm", "marginal") and case["n"] <= 20 and case["chi"] * 2 ** case["n"] <= 1 << 33:
        n = case["n"]
        circ = _circuit(case, _rng(seed, 2))[0]
        psi = _Terms(_spec(circ, case["chi"], seed)).amplitudes(torch.arange(2 ** n, device=DEV))
        rng = _rng(seed, 3)
        off, diag = _equatorial(n, case["L"], rng)
        if kind == "norm":
            ov = _dense_etas(n, psi, off, diag)
            eta = 2.0 ** n * ov.abs().square()
            return {"overlap": ov.cpu().numpy(), "eta": eta.cpu(), "mean": float(eta.mean())}
        qubits, u = rng.permutation(n)[:case["w"]], rng.random(case["w"])
        x = torch.arange(2 ** n, device=DEV)
        est, prob = np.zeros((case["w"], 2)), np.zeros(case["w"])
        for j, q in enumerate(qubits.tolist()):
            half = [torch.where(((x >> q) & 1) == b, psi, 0) for b in (0, 1)]
            est[j] = [float((2.0 ** n * _dense_etas(n, h, off, diag).abs().square()).mean()) for h in half]
            p0 = est[j, 0] / est[j].sum() if est[j].sum() > 0 else 0.5
            bit = 0 if u[j] < p0 else 1
            prob[j] = p0 if bit == 0 else 1.0 - p0
            psi = half[bit]
        return {"bits": None, "prob": prob, "est": est}
    if kind == "overlaps" and case["n"] <= 20 and (case["chi"] + case["bras"]) * 2 ** case["n"] <= 1 << 33:
        ck, cb = _overlap_circuits(case, seed)
        x = torch.arange(2 ** case["n"], device=DEV)
        psi = _Terms(_spec(ck, case["chi"], seed)).amplitudes(x)
        T = _Terms(_spec(cb, case["bras"], seed + 1))
        ov = []
        for l in range(case["bras"]):
            one = object.__new__(_Terms)
            one.n = T.n
            for f in ("F", "G", "M", "g"):
                setattr(one, f, getattr(T, f)[:, l:l + 1])
            for f in ("v", "s", "w"):
                setattr(one, f, getattr(T, f)[l:l + 1])
            one.b = torch.ones_like(T.b[l:l + 1])
            ov.append(torch.vdot(one.amplitudes(x), psi))
        ov = torch.stack(ov)
        return {"overlap": ov.cpu().numpy(), "total": torch.vdot(T.b, ov).reshape(1).cpu().numpy()}
    if kind == "chains" and case["chi"] * case["chains"] * case["steps"] * case["n"] <= 3 << 34:
        amp = _exact_chains(case, seed)
        return {"trace": None, "accepted": None, "amp": amp.cpu().numpy() if case["host"] else _pairs(amp)}
    if kind == "train":
        return _exact_train(case, seed)
    return None
