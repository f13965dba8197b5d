#!/usr/bin/env python3
"""Benchmark of the sum-over-Cliffords hot path on one MI355X.

A step is one pass of the hot path over the n = 50 amplitude workload
(2000 Clifford gates + 40 phase slots, chi = 2^16 sparsified terms, 4096
uniform bitstrings): re-draw the chi terms (branch choices and b_alpha),
evolve them through the circuit, and evaluate all chi x 4096 term amplitudes
with the FP32 compensated sum.  Inputs are resident in HBM before the timed
region.  value = chi * |x| / (seconds per step).

Prints one JSON line.  Extra keys: per-phase times measured with HIP events
on the library's stream, the roofline of the dominant kernel (against the
chip's published peak and against the int32 issue, HBM copy and LDS read
rates measured in the same run), the FP64 path, and the CPU oracle timed on
a bounded sample of the same workload (all host threads, and one thread).
Further sections (`--sections`): norm estimation with equatorial states,
inner products with stabilizer states given as CH forms, Metropolis chains
(plain and learned proposals on the n = 50 QAOA instance, and the matched
total-variation comparison on its n = 12 twin), a batch of 64 uneven
instances, and the hidden-shift circuit with CCZ gates (sparsification bound
and chain-rule sampling of output bits).  Progress lines go to stderr.
"""
import argparse
import hashlib
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

# MI355X 32-bit VALU lane rate: the FP32 vector peak (157.3 TFLOP/s, an FMA
# being 2 flops) is 78.6 T lane-operations/s = 256 CUs x 128 lanes/clk x
# 2.4 GHz.  32-bit integer ops issue at that lane rate: the in-run
# microbenchmark (chsim_measure_peaks) measures about 63 T int32 ops/s, above
# the 64 lanes/clk/CU (39.3 T) figure, which therefore is not a bound.
INT32_PEAK_OPS = 256 * 128 * 2.4e9
HBM_PEAK_BPS = 8.0e12


def algorithmic_ops_evolve(stats, n):
    """Int32 operations of one evolution on bit-packed rows, from the gate
    applications it executed (per term, or per shared prefix state), counted
    per rule of this implementation: S-type 3, CZ 4, CX 12, H 28 n + 40, a
    general-branch gate 12."""
    return float(stats["H"] * (28 * n + 40) + stats["CX"] * 12 + stats["CZ"] * 4 + stats["S"] * 3
                 + stats["cond"] * 12)


def table_ops_evolve(stats, n):
    """The same executed gate applications at the hot-path table's per-unit
    figure: 35 int32 operations per tableau row (n rows) per Hadamard and 10
    per other gate."""
    return float(stats["H"] * 35 * n + (stats["CX"] + stats["CZ"] + stats["S"] + stats["cond"]) * 10)


# MI355X LDS: 256 CUs x 128 B/clk x 2.4 GHz.
LDS_PEAK_BPS = 256 * 128 * 2.4e9
# FP4 matrix cores: 1024 SIMDs, a 32x32x64 product (2^17 operations) per 32 clocks at 2.4 GHz.
FP4_PEAK_OPS = 1024 * 2.0**17 / 32 * 2.4e9

# Peaks measured in this run by chsim_measure_peaks (int32 VALU in TOP/s, HBM
# copy in GB/s, LDS reads in TB/s); filled in main() before any section.
MEASURED = {}


def roof(bound, achieved, peak, unit, measured=None, **extra):
    """A roofline record: achieved against the chip's published (or unit-count
    derived) peak, and against the peak measured in this run."""
    d = {"bound": bound, "achieved": round(achieved, 4), "peak": round(peak, 3), "unit": unit,
         "frac": round(achieved / peak, 4)}
    if measured:
        d["peak_measured"] = round(measured, 3)
        d["frac_of_measured"] = round(achieved / measured, 4)
    d.update(extra)
    return d


def amp_lds_bytes_per_pair(n, v_words):
    """LDS bytes the table kernel (n > 60) reads per (term, x): 8-byte table
    lookups, ceil(n / 4) for a term whose zero test is packed into its
    quadratic-form rows (n - |v| <= 64 - n), twice that otherwise, plus one
    lookup of the term's value; returned with the packed fraction of the
    sampled terms."""
    vc = np.array([bin(int(w)).count("1") for w in np.asarray(v_words).ravel()])
    packed = (n - vc) <= (64 - n)
    nch = (n + 3) // 4
    per = np.where(packed, nch, 2 * nch) + 1
    return 8.0 * float(np.mean(per)), float(np.mean(packed))


def amp_fp4_ops_per_pair(n):
    """FP4 operations (multiply and add counted apart) of the matrix-core
    amplitude kernel per (term, x): 64 features per step, n (n + 1) / 2 + 1
    features."""
    return 128.0 * ((n * (n + 1) // 2 + 1 + 63) // 64)


def algorithmic_ops_amp(xs):
    """Int32 operations per (term, x): 6 per set bit (XOR, AND, POPCOUNT on
    64-bit words) + 20 for the zero test and the phase."""
    pc = np.array([bin(int(v)).count("1") for v in xs])
    return float(np.mean(6 * pc + 20))


def progress(msg):
    """One flushed line on stderr per bench section, so that a run that stops
    early shows how far it got (the JSON result stays the only stdout line)."""
    print(f"[bench] {time.strftime('%H:%M:%S')} {msg}", file=sys.stderr, flush=True)


def cpu_baseline(cfg, sample_terms, threads, single_terms=2048):
    """The oracle on the host cores: `sample_terms` terms on `threads` threads
    (std::thread over terms and strings), and `single_terms` terms on one
    thread; both evolve their terms and evaluate them on all strings."""
    import oracle as O

    circ = cfg["circuit"]

    def leg(count, th):
        t0 = time.perf_counter()
        T = O.Terms(circ, cfg["chi"], O.SPARSIFY, seed=cfg["seed"],
                    alphas=np.arange(count, dtype=np.uint64), threads=th)
        t1 = time.perf_counter()
        T.amplitudes(cfg["x"])
        t2 = time.perf_counter()
        return count * cfg["x"].size / (t2 - t0), t1 - t0, t2 - t1

    v, te, ta = leg(sample_terms, threads)
    v1, te1, ta1 = leg(single_terms, 1)
    return dict(value=v, unit="evals/s", cores=threads, kind="oracle", nproc=os.cpu_count(),
                sample=f"first {sample_terms} of {cfg['chi']} terms evolved + their amplitudes on all "
                       f"{cfg['x'].size} strings ({te:.2f} s evolve, {ta:.2f} s amplitudes)",
                single_thread={"value": v1, "unit": "evals/s", "cores": 1,
                               "sample": f"first {single_terms} terms, all {cfg['x'].size} strings "
                                         f"({te1:.2f} s evolve, {ta1:.2f} s amplitudes)"})


# Sources each counter-measured kernel is built from (its launch planning in
# api.hip included): the recorded bytes stay valid while these files are unchanged.
KERNEL_SOURCES = {
    "k_evolve": ["evolve_kernel.hpp", "evolve.hip", "evolve_l4.hip", "evolve_l8.hip",
                 "evolve_wide.hip", "evolve_w64.hip", "prefix.hip", "device_common.hpp", "internal.hpp",
                 "api.hip"],
    "k_evolve_cols": ["evolve_cols.hpp", "bitops.hpp", "evolve_w64.hip", "evolve.hip", "prefix.hip",
                     "device_common.hpp", "internal.hpp", "api.hip"],
    "k_amp_mfma<float>": ["amplitude_mfma.hip", "device_common.hpp", "internal.hpp", "api.hip"],
    "k_amp<float>": ["amplitude.hip", "device_common.hpp", "internal.hpp", "api.hip"],
    "k_quad_pairs": ["quad_pairs.hip", "inner.hip", "bitops.hpp", "device_common.hpp", "internal.hpp", "api.hip"],
    "k_quad_pairs(ch)": ["quad_pairs.hip", "inner_ch.hip", "bitops.hpp", "device_common.hpp", "internal.hpp", "api.hip"],
}


def kernel_sources_sha256(kernel):
    """Hash of the sources `kernel` is built from (counter-derived traffic is
    only reported while it still describes the code being run)."""
    csrc = os.path.join(ROOT, "paper_1808_00128_amd", "csrc")
    h = hashlib.sha256()
    for f in KERNEL_SOURCES[kernel]:
        with open(os.path.join(csrc, f), "rb") as fh:
            h.update(f.encode())
            h.update(fh.read())
    return h.hexdigest()


def counter_traffic(kernel):
    """HBM bytes per launch of `kernel` from the committed rocprofv3 byte
    counters (profiles/traffic_counters.json), or None if its sources changed
    since they were taken."""
    path = os.path.join(ROOT, "profiles", "traffic_counters.json")
    try:
        with open(path) as fh:
            k = json.load(fh).get("kernels", {}).get(kernel)
    except (OSError, ValueError):
        return None
    if k is None or k.get("sources_sha256") != kernel_sources_sha256(kernel):
        return None
    return float(k["bytes_per_launch"])


def shape_name(value):
    """Evolution mapping of a lanes value: lanes per term and what they hold."""
    lanes = value & 0xff
    what = "columns" if value & 0x100 else "rows"
    return f"{lanes} lanes/term, {what} in registers"


def tuned_name(B, lanes, tune_ms):
    """What the autotuner kept.  The default, which mixes mappings span by span, reads
    as 4 lanes with columns; it was kept unless that value was the fastest."""
    name = shape_name(lanes)
    if lanes != (4 | B.CHSIM_EVOLVE_LDS):
        return name
    times = [t for t in tune_ms if t > 0]
    fastest = times and min(times) == tune_ms[B.TUNE_SHAPES.index(lanes)]
    return f"default, or {name}" if fastest else "default (mixed by span)"


def mean_popcount(words):
    return float(np.mean([bin(int(w)).count("1") for w in np.asarray(words).ravel()]))


def bench_norm(torch, B, W, L=1024):
    """Norm-estimation workload: n = 40, 200 Clifford gates + 30 phase slots,
    chi = 2^18, L equatorial states; all chi * L inner products per call."""
    cfg = W.config_norm(L=L)
    circ = cfg["circuit"]
    ctx = B.Context([cfg])
    ctx.set_evolve_lanes(-1)
    ctx.apply_circuit(circ)
    ctx.inner_products(cfg["Aoff"][:8], cfg["Adiag"][:8])  # warm-up
    terms = ctx.get_terms(0, 256)
    mean_v = mean_popcount(terms["v"])
    n, chi = circ.n, cfg["chi"]
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    ov, eta, eta_mean = ctx.inner_products(cfg["Aoff"], cfg["Adiag"])
    t1 = time.perf_counter()
    ctx.close()
    pairs = chi * L
    # The hot-path table's count per (term, A): 4 n^2 (off-diagonal K_A) + 2 n^2
    # (its mod-4 diagonal) + 2 N^2 (elimination, N = |v| + 1).
    ops_pair = 6 * n * n + 2 * (mean_v + 1) ** 2
    achieved = ops_pair * pairs / (t1 - t0) / 1e12
    return {"workload": cfg["name"] + ": n=40, 200 Clifford + 30 phase slots, chi=2^18, L=1024",
            "seconds": t1 - t0, "inner_products_per_s": pairs / (t1 - t0),
            "eta_mean": eta_mean, "eta_sem": float(np.std(eta, ddof=1) / np.sqrt(L)),
            "mean_v_weight": mean_v,
            "roofline": roof("alu", achieved, INT32_PEAK_OPS / 1e12, "TOP/s (int32)", MEASURED.get("valu"),
                             kernel="k_quad_prep + k_quad_pairs (bit-sliced, 128 states per wave)",
                             traffic=counter_traffic("k_quad_pairs"), ops_per_pair=ops_pair,
                             count="6 n^2 + 2 (|v| + 1)^2 int32 ops per (term, A)")}


def bench_inner_ch(torch, B, W, L=256):
    """Norm-estimation workload (n = 40, chi = 2^18) against L random stabilizer
    states given as CH forms (the terms of a random Clifford circuit with 30
    phase slots): every <theta_l|phi_alpha>, chi * L pairs, and the mean of
    2^n |<theta_l|psi>|^2."""
    cfg = W.config_norm(L=8)
    circ = cfg["circuit"]
    n, chi = circ.n, cfg["chi"]
    rng = np.random.default_rng(1500)
    cb = W.random_circuit(n, 400, rng.uniform(0, 2 * np.pi, size=30), rng)
    ctx = B.Context([cfg, dict(circuit=cb, chi=L, mode="sparsify", seed=1501)])
    ctx.set_evolve_lanes(-1)
    ctx.apply_circuit(circ, inst=0)
    ctx.apply_circuit(cb, inst=1)
    ctx.inner_products_ch(1, inst=0)  # warm-up (records, kernels)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    ov, _ = ctx.inner_products_ch(1, inst=0)
    t1 = time.perf_counter()
    vb = ctx.get_terms(0, L, inst=1)["v"]
    vk = ctx.get_terms(0, 256, inst=0)["v"]
    ctx.close()
    pairs = chi * L
    # Per pair: the equations of the bra's support (n rows of G selected by a
    # column of F: n^2 bit-ANDs/XORs on 64-bit words), the bilinear form on the
    # free directions (n^2), their Gram rows (N^2) and the elimination (2 N^2),
    # N = |v| + 1, as 64-bit word operations (2 int32 ops each).
    N = mean_popcount(vk) + 1
    ops_pair = 2 * (2 * n * n + 3 * N * N)
    achieved = ops_pair * pairs / (t1 - t0) / 1e12
    eta = (2.0 ** n) * np.abs(ov) ** 2
    return {"workload": f"{cfg['name']} terms (n=40, chi=2^18) x {L} stabilizer states from a random "
                        "400-gate Clifford circuit with 30 phase slots",
            "seconds": t1 - t0, "inner_products_per_s": pairs / (t1 - t0),
            "eta_mean": float(eta.mean()), "eta_sem": float(eta.std(ddof=1) / np.sqrt(L)),
            "mean_v_weight_bra": mean_popcount(vb), "mean_v_weight_ket": mean_popcount(vk),
            "roofline": roof("alu", achieved, INT32_PEAK_OPS / 1e12, "TOP/s (int32)", MEASURED.get("valu"),
                             kernel="k_chrec + k_quad_prep + k_quad_pairs (bit-sliced, 128 states per wave)",
                             traffic=counter_traffic("k_quad_pairs(ch)"), ops_per_pair=ops_pair,
                             count="2 (2 n^2 + 3 (|v| + 1)^2) int32 ops per pair (64-bit word operations x 2)")}


def start_points(ctx, n, chi, count, rng):
    """Chain starts: a term drawn uniformly (all |b_alpha| are equal) and a
    string sampled from it, kept if <x|psi> != 0."""
    from paper_1808_00128_amd import workloads as W

    xs = []
    while len(xs) < count:
        alpha = rng.integers(0, chi, size=4 * count)
        flips = W.random_bitstrings(n, 4 * count, rng)
        cand = ctx.sample_terms(alpha, flips)
        amp = ctx.amplitudes(cand)
        xs += [int(x) for x, a in zip(cand, amp) if abs(a) > 0]
    return np.array(xs[:count], np.uint64)


def run_plain(torch, ctx, x0, jstream, ustream, graph=None):
    """The chains' steps launched kernel by kernel (timed); with a dict in
    `graph`, the same steps again from a recorded HIP graph: time of the
    replay and whether the trajectories agree."""
    dev = torch.device("cuda:0")
    stream = torch.cuda.current_stream()
    n_chain, steps = jstream.shape
    ctx.metropolis_init(x0)
    j = torch.from_numpy(jstream.astype(np.int32)).to(dev)
    u = torch.from_numpy(ustream).to(dev)
    trace = torch.empty((n_chain, steps), dtype=torch.int64, device=dev)
    acc = torch.empty((n_chain, steps), dtype=torch.uint8, device=dev)
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    e0.record(stream)
    ctx.metropolis_step_device(j, u, trace, acc)
    e1.record(stream)
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1)
    tr, ac = trace.cpu().numpy().view(np.uint64), acc.cpu().numpy()
    if graph is not None:
        trace2 = torch.empty_like(trace)
        acc2 = torch.empty_like(acc)
        same = True
        for rep in range(2):  # the first call records the graph, the second replays it
            ctx.metropolis_init(x0)
            torch.cuda.synchronize()
            e0.record(stream)
            ctx.metropolis_step_device(j, u, trace2, acc2, graph=True)
            e1.record(stream)
            torch.cuda.synchronize()
            same = same and bool(torch.equal(trace, trace2)) and bool(torch.equal(acc, acc2))
        graph.update(ms_per_step_graph=e0.elapsed_time(e1) / steps, ms_per_step_launches=ms / steps,
                     trajectories_equal=same)
    return tr, ac, ms


def run_learned(torch, ctx, net, x0, streams, eps, pi_min, pi_max):
    dev = torch.device("cuda:0")
    stream = torch.cuda.current_stream()
    u_mix, jj, u_bits, uu = streams
    n_chain, steps = jj.shape
    ctx.metropolis_init(x0)
    t_umix = torch.from_numpy(u_mix).to(dev)
    t_j = torch.from_numpy(jj.astype(np.int32)).to(dev)
    t_ub = torch.from_numpy(np.ascontiguousarray(u_bits)).to(dev)
    t_u = torch.from_numpy(uu).to(dev)
    trace = torch.empty((n_chain, steps), dtype=torch.int64, device=dev)
    acc = torch.empty((n_chain, steps), dtype=torch.uint8, device=dev)
    flips = torch.empty((n_chain, steps), dtype=torch.int32, device=dev)
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    e0.record(stream)
    ctx.metropolis_step_learned_device(net, t_umix, t_j, t_ub, t_u, eps, pi_min, pi_max, trace, acc,
                                       flips)
    e1.record(stream)
    torch.cuda.synchronize()
    return (trace.cpu().numpy().view(np.uint64), acc.cpu().numpy(), flips.cpu().numpy(),
            e0.elapsed_time(e1))


def train_proposal(B, W, ctx, n, trace, burn, delta, epochs=20, hidden=256, batch=1024, lr=1e-3):
    """Pairs (x_t, x_t ^ x_{t+delta}) from plain chains after burn-in."""
    xt = trace[:, burn:-delta].ravel()
    tgt = trace[:, burn:-delta].ravel() ^ trace[:, burn + delta:].ravel()
    net = B.MLP(ctx, n, hidden, max(batch, trace.shape[0]), W.mlp_init(n, hidden))
    t0 = time.perf_counter()
    losses = net.train(xt, tgt, batch=batch, epochs=epochs, lr=lr)
    t1 = time.perf_counter()
    return net, {"pairs": int(xt.size), "delta": int(delta), "epochs": epochs, "batch": batch,
                 "lr": lr, "seconds": t1 - t0, "loss_first": float(losses[0]),
                 "loss_last": float(losses[-1])}


def chain_step_bytes(chi, n, n_chain):
    """HBM bytes of one chain step when every row of a term is read (the
    flip-mask kernel stages all n rows: F_p, M_p 8 B each, gamma_p 1 B), each
    chain's cached word read and the proposal word written (16 B), and the
    term's constants (33 B)."""
    return float(chi * (17 * n + 16 * n_chain + 33))


# Steps per window of deferred chain-cache updates in the single-flip kernel.
METRO_WINDOW = 4


def own_chain_step_bytes(chi, n_chain, win=METRO_WINDOW):
    """HBM bytes of one single-flip step when every launch takes one step (one
    flip bit per step shared by the chains): each chain's cached word read (8 B)
    and written once per window (8 / win B), the rows F_j, M_j, gamma_j (17 B)
    of the proposal bit and of the window's pending steps ((win + 1) / 2 on
    average), and the term's constants (33 B)."""
    return float(chi * (8 * n_chain + 8 * n_chain / win + 17 * (1 + (win + 1) / 2) + 33))


def pair_chain_step_bytes(chi, n_chain, win=METRO_WINDOW):
    """The same as the kernel moves them, two steps per launch: the cached word
    read once per two steps (4 B), the pending rows ((win + 2) / 2 per launch)
    and the constants once per two steps."""
    return float(chi * (4 * n_chain + 8 * n_chain / win + 17 * (1 + (win + 2) / 4) + 33 / 2))


def record_step_bytes(n, chi):
    """Bytes of the amplitude records that an FP64 pass over the strings of a learned
    step reads: per 32 terms S KB of weights, S = ceil((n (n + 1) / 2 + 1) / 64), the
    head and 2 KB of doubles (not the KB of floats)."""
    return float(-(-chi // 32) * 1024 * ((n * (n + 1) // 2 + 1 + 63) // 64 + 3))


def table_chain_step_bytes(chi, n_chain):
    """The hot-path table's per-step bytes for single flips with one j per step
    shared by all chains: 16 B of state read + write per chain, 17 B for row j
    of F, M, gamma and 33 B of term constants per term."""
    return float(chi * (16 * n_chain + 17 + 33))


def chain_report(stats, trace, acc, ms, burn, obs, flips=None):
    tau, win, err = stats.tau_int(obs)
    ess = obs.size / (2 * tau)
    out = {"ms_per_step": ms / trace.shape[1], "acceptance": float(acc.mean()), "tau_int": tau,
           "tau_int_err": err, "ess": ess, "ess_per_s": ess / (ms / 1e3)}
    if flips is not None:
        out["mean_flips"] = float(flips[:, burn:].mean())
    return out


# QAOA instance of the Metropolis sections: the paper's beta = pi/4 (its
# Clifford mixer line) and gamma near the extremum of E(gamma) on that line
# (E(0.367) is the minimum of the n = 12..14 instances of the same shape,
# scanned densely; E(-gamma) = -E(gamma)).
QAOA_BETA = float(np.pi / 4)
QAOA_GAMMA = 0.35


def bench_learned(torch, B, W, stats, steps=1000, n_chain=64, chi=1 << 20, eps=0.1,
                  pi_min=0.002, pi_max=0.5):
    """QAOA n = 50, chi = 2^20 (beta = pi/4, gamma = 0.35, one flip bit per step
    shared by the chains): plain chains, a proposal trained on them, learned
    chains with the trained and with the untrained network."""
    cfg = W.config_qaoa(chi=chi, n_chain=n_chain, steps=steps, gamma=QAOA_GAMMA, beta=QAOA_BETA, shared_j=True)
    circ = cfg["circuit"]
    n = circ.n
    ctx = B.Context([cfg])
    ctx.set_evolve_lanes(-1)
    ctx.apply_circuit(circ)
    rng = np.random.default_rng(cfg["seed"] + 1)
    x0 = start_points(ctx, n, chi, n_chain, rng)
    burn = steps // 5
    graph = {}
    progress("metropolis: plain chains (launches, then graph record and replay)")
    tr, ac, ms = run_plain(torch, ctx, x0, cfg["jstream"], cfg["ustream"], graph=graph)
    cost = stats.qaoa_cost(tr[:, burn:], cfg["triples"], cfg["d"])
    plain = chain_report(stats, tr, ac, ms, burn, cost)
    plain["hip_graph"] = graph
    sbytes = table_chain_step_bytes(chi, n_chain)
    achieved = sbytes * steps / (ms / 1e3) / 1e9
    obytes = pair_chain_step_bytes(chi, n_chain)
    plain["roofline"] = roof("hbm", achieved, HBM_PEAK_BPS / 1e9, "GB/s", MEASURED.get("hbm"),
                             kernel="k_propose_pair (single flips, shared j, two steps per launch, "
                                    f"cache writes deferred over windows of {METRO_WINDOW} steps) + k_metro_accept",
                             traffic=None, bytes_per_step=sbytes,
                             count="chi (16 chains + 17 + 33) B per step (state r/w, row j, constants)",
                             bytes_per_step_own=obytes,
                             own_count=f"chi (4 chains + 8 chains / {METRO_WINDOW} + 17 (1 + "
                                       f"{(METRO_WINDOW + 2) / 4}) + 33 / 2) B per step (state read once per "
                                       "two steps, written once per window, proposal and pending rows, constants)",
                             frac_own_count=round(obytes * steps / (ms / 1e3) / HBM_PEAK_BPS, 4),
                             bytes_per_step_all_rows=chain_step_bytes(chi, n, n_chain))
    delta = max(1, int(round(plain["tau_int"])))
    progress("metropolis: training the proposal")
    net, train = train_proposal(B, W, ctx, n, tr, burn, delta)
    streams = W.learned_streams(n, n_chain, steps, np.random.default_rng(cfg["seed"] + 2))
    progress("metropolis: learned chains")
    ltr, lac, lfl, lms = run_learned(torch, ctx, net, x0, streams, eps, pi_min, pi_max)
    lcost = stats.qaoa_cost(ltr[:, burn:], cfg["triples"], cfg["d"])
    learned = chain_report(stats, ltr, lac, lms, burn, lcost, lfl)
    lbytes = chain_step_bytes(chi, n, n_chain)
    lach = lbytes * steps / (lms / 1e3) / 1e9
    lown = record_step_bytes(n, chi)
    learned["roofline"] = roof("hbm", lach, HBM_PEAK_BPS / 1e9, "GB/s", MEASURED.get("hbm"),
                               kernel="k_mlp_fused (masks and network) + k_amp_mfma<double> (proposals) + k_learned_accept",
                               traffic=None, bytes_per_step=lbytes,
                               count="chi (17 n + 16 chains + 33) B per step (every row staged for the masks)",
                               bytes_per_step_own=lown,
                               own_count="the amplitude records: (n (n + 1) / 2 + 1) / 64 + 3 KB per 32 terms and "
                                         "step (weights, head, doubles; the caches are brought up to date once "
                                         "per call; condition words past the third level not counted)",
                               frac_own_count=round(lown * steps / (lms / 1e3) / HBM_PEAK_BPS, 4))
    net.close()
    progress("metropolis: learned chains with the untrained network")
    unet = B.MLP(ctx, n, 256, max(1024, n_chain), W.mlp_init(n, 256))
    utr, uac, ufl, ums = run_learned(torch, ctx, unet, x0, streams, eps, pi_min, pi_max)
    unet.close()
    ucost = stats.qaoa_cost(utr[:, burn:], cfg["triples"], cfg["d"])
    untrained = chain_report(stats, utr, uac, ums, burn, ucost, ufl)
    ctx.close()
    return {"workload": f"{cfg['name']}: QAOA p=1, {len(cfg['triples'])} triples, gamma={QAOA_GAMMA}, "
                        f"beta=pi/4, {n_chain} chains x {steps} steps, one flip bit per step for all chains",
            "gamma": QAOA_GAMMA, "beta": QAOA_BETA,
            "plain": dict(plain, mean_cost=float(cost.mean())),
            "learned": dict(learned, mean_cost=float(lcost.mean()), eps=eps, pi_min=pi_min,
                            pi_max=pi_max, network="50-256-256-50 ReLU, BF16 MFMA", training=train),
            "learned_untrained": dict(untrained, mean_cost=float(ucost.mean())),
            "ess_per_s_learned_over_plain": learned["ess_per_s"] / plain["ess_per_s"],
            "ess_per_step_trained_over_untrained": (learned["ess"] / untrained["ess"])
            if untrained["ess"] > 0 else None}


def bench_matched_tv(torch, B, W, stats, n=12, triples=16, chi=1 << 16, n_chain=64, steps=12800,
                     eps=0.1, pi_min=0.002, pi_max=0.5, target=0.05):
    """n = 12 twin of the QAOA workload (beta = pi/4, gamma = 0.35): steps and
    seconds until the pooled samples of 64 chains are within `target` total
    variation of the exact law (all 4096 amplitudes), plain vs learned proposal
    (trained on the plain chains) vs the untrained network.  `iid_floor` is the
    TV of the same number of independent exact samples: no chain can go below it."""
    rng = np.random.default_rng(2012)
    circ = W.qaoa_circuit(n, triples, rng, gamma=QAOA_GAMMA, beta=QAOA_BETA)[0]
    spec = dict(circuit=circ, chi=chi, mode="sparsify", seed=2012)
    ctx = B.Context([spec])
    ctx.apply_circuit(circ)
    P = np.abs(ctx.amplitudes(np.arange(2**n, dtype=np.uint64))) ** 2
    P /= P.sum()
    x0 = np.array(rng.choice(2**n, size=n_chain, p=P), np.uint64)  # start in equilibrium
    j, u = W.metropolis_streams(n, n_chain, steps, rng, shared_j=True)
    graph = {}
    tr, ac, ms = run_plain(torch, ctx, x0, j, u, graph=graph)
    tau, _, _ = stats.tau_int(np.array([bin(int(v)).count("1") for v in tr.ravel()],
                                       np.float64).reshape(tr.shape))
    net, train = train_proposal(B, W, ctx, n, tr, 0, max(1, int(round(tau))), epochs=30, hidden=128)
    streams = W.learned_streams(n, n_chain, steps, rng)
    ltr, lac, lfl, lms = run_learned(torch, ctx, net, x0, streams, eps, pi_min, pi_max)
    net.close()
    unet = B.MLP(ctx, n, 128, 1024, W.mlp_init(n, 128))
    utr, uac, ufl, ums = run_learned(torch, ctx, unet, x0, streams, eps, pi_min, pi_max)
    unet.close()
    ctx.close()
    checkpoints = [25, 50, 100, 200, 400, 800, 1600, 3200, 6400, 12800]

    def curve(t):
        return {c: stats.total_variation(t[:, :c].ravel(), P) for c in checkpoints if c <= steps}

    cp, cl, cu = curve(tr), curve(ltr), curve(utr)
    iid = rng.choice(2**n, size=(n_chain, steps), p=P).astype(np.uint64)
    floor = curve(iid)

    def first(c):
        hit = [k for k, v in c.items() if v <= target]
        return min(hit) if hit else None

    def ess_per_step(t):
        obs = np.array([bin(int(v)).count("1") for v in t.ravel()], np.float64).reshape(t.shape)
        tt, _, _ = stats.tau_int(obs)
        return 1.0 / (2.0 * tt)

    sp, sl, su = first(cp), first(cl), first(cu)
    per_p, per_l, per_u = ms / steps, lms / steps, ums / steps
    return {"workload": f"qaoa-n{n}-{triples}triples-chi{chi}, gamma={QAOA_GAMMA}, beta=pi/4, "
                        f"{n_chain} chains started from P",
            "tv_target": target, "iid_floor": floor,
            "plain": {"tv_by_steps": cp, "steps_to_target": sp, "ms_per_step": per_p,
                      "seconds_to_target": (sp * per_p / 1e3) if sp else None,
                      "acceptance": float(ac.mean()), "ess_per_step_weight": ess_per_step(tr),
                      "hip_graph": graph},
            "learned": {"tv_by_steps": cl, "steps_to_target": sl, "ms_per_step": per_l,
                        "seconds_to_target": (sl * per_l / 1e3) if sl else None,
                        "acceptance": float(lac.mean()), "mean_flips": float(lfl.mean()),
                        "ess_per_step_weight": ess_per_step(ltr), "training": train},
            "learned_untrained": {"tv_by_steps": cu, "steps_to_target": su, "ms_per_step": per_u,
                                  "seconds_to_target": (su * per_u / 1e3) if su else None,
                                  "acceptance": float(uac.mean()), "mean_flips": float(ufl.mean()),
                                  "ess_per_step_weight": ess_per_step(utr)}}


def bench_uneven(torch, B, W, steps=2, warmup=1):
    """64 independent instances (n 20..60, chi 2^10..2^20, 1024 strings each):
    re-draw + evolve every instance, then all amplitudes in ONE batched launch
    (FP32C), against one amplitude call per instance."""
    cfg = W.config_uneven()
    insts = cfg["instances"]
    dev = torch.device("cuda:0")
    stream = torch.cuda.current_stream()
    ctx = B.Context(insts)
    gates = [B.gate_array(sp["circuit"]) for sp in insts]
    xs = [torch.from_numpy(sp["x"].view(np.int64)).to(dev) for sp in insts]
    for k in range(len(insts)):
        ctx.set_evolve_lanes(-1, inst=k)
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(4)]
    t_ev, t_batch, t_single = [], [], []
    outs = None
    for i in range(warmup + steps):
        ev[0].record(stream)
        for k, sp in enumerate(insts):
            ctx.reset(sp["seed"] + i, inst=k)
            ctx.apply_gates(gates[k], inst=k)
        ev[1].record(stream)
        outs = ctx.amplitudes_batch(list(enumerate(xs)), fp32c=True)
        ev[2].record(stream)
        for k in range(len(insts)):
            ctx.amplitudes(xs[k], inst=k, fp32c=True)
        ev[3].record(stream)
        torch.cuda.synchronize()
        if i >= warmup:
            t_ev.append(ev[0].elapsed_time(ev[1]))
            t_batch.append(ev[1].elapsed_time(ev[2]))
            t_single.append(ev[2].elapsed_time(ev[3]))
    evals = float(sum(sp["chi"] * sp["x"].size for sp in insts))
    fp4 = sum(amp_fp4_ops_per_pair(sp["circuit"].n) * sp["chi"] * sp["x"].size for sp in insts)
    ms_b = float(np.mean(t_batch))
    ms_s = float(np.mean(t_single))
    ms_e = float(np.mean(t_ev))
    ok = all(bool(torch.isfinite(o).all()) for o in outs)
    ctx.close()
    return {"workload": cfg["name"] + ": 64 circuits, n~U{20..60}, 40n Clifford gates + 10..60 phase "
                                      "slots, chi log-uniform 2^10..2^20 (sparsified), 1024 uniform x each",
            "total_terms": int(sum(sp["chi"] for sp in insts)), "evals": evals,
            "ms_evolve_all": ms_e, "ms_amplitudes_batched": ms_b, "ms_amplitudes_per_instance": ms_s,
            "evals_per_s_batched": evals / (ms_b / 1e3), "evals_per_s_per_instance": evals / (ms_s / 1e3),
            "evals_per_s_step": evals / ((ms_e + ms_b) / 1e3),
            "amplitude_roofline": roof("mfma", fp4 / (ms_b / 1e3) / 1e12, FP4_PEAK_OPS / 1e12, "TFLOP/s (FP4)"),
            "finite": ok}


def bench_hidden_shift(torch, B, W, steps=5, warmup=2):
    """Hidden-shift circuit with CCZ gates (n = 40, 16 CCZ, chi = floor(((4/3)^16 /
    0.3)^2) sparsified terms): each CCZ is a slot of eight diagonal Clifford
    branches (Eq. (CCZ decomposition)).  Strings: s and 4095 draws from the
    terms' own output distributions (uniform strings would give exactly zero
    amplitude for nearly every term).  Times evolution, FP32C and FP64 amplitudes."""
    cfg = W.config_hidden_shift()
    circ = cfg["circuit"]
    n, chi = circ.n, cfg["chi"]
    dev = torch.device("cuda:0")
    stream = torch.cuda.current_stream()
    ctx = B.Context([cfg, cfg])  # instance 1: scratch store for the marginal sampler
    ctx.set_evolve_lanes(-1)
    gates = B.gate_array(circ)
    ctx.apply_gates(gates)
    rng = np.random.default_rng(cfg["seed"] + 1)
    n_x = cfg["x"].size
    alpha = rng.integers(0, chi, size=n_x - 1).astype(np.uint64)
    xs = np.concatenate([[cfg["s"]], ctx.sample_terms(alpha, W.random_bitstrings(n, n_x - 1, rng))]).astype(np.uint64)
    x_dev = torch.from_numpy(xs.view(np.int64)).to(dev)
    out32 = torch.empty((n_x, 2), dtype=torch.float64, device=dev)
    out64 = torch.empty((n_x, 2), dtype=torch.float64, device=dev)
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(4)]
    t_ev, t_32, t_64 = [], [], []
    for i in range(warmup + steps):
        ev[0].record(stream)
        ctx.reset(cfg["seed"])
        ctx.apply_gates(gates)
        ev[1].record(stream)
        ctx.amplitudes(x_dev, fp32c=True, out=out32)
        ev[2].record(stream)
        ctx.amplitudes(x_dev, fp32c=False, out=out64)
        ev[3].record(stream)
        torch.cuda.synchronize()
        if i >= warmup:
            t_ev.append(ev[0].elapsed_time(ev[1]))
            t_32.append(ev[1].elapsed_time(ev[2]))
            t_64.append(ev[2].elapsed_time(ev[3]))
    st = ctx.evolution_stats()
    lanes, _ = ctx.evolve_lanes()
    pf_mode, pf_levels, pf_frac = ctx.prefix_share()
    # Sparsification tail bound: <Omega|Omega> by norm estimation over 1024
    # equatorial states, delta^2 = ||c||_1^2 / chi.
    Aoff, Adiag = W.random_equatorial(n, 1024, rng)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    est, sem, delta2, bound = ctx.sparsification_bound(Aoff, Adiag)
    t_bound = time.perf_counter() - t0
    # Chain-rule sampling of 8 output bits by norm estimation (256 equatorial
    # states per estimate, two estimates per bit); psi = |s>, so the bits are s's.
    mq = list(range(8))
    Am, Dm = W.random_equatorial(n, 256, rng)
    um = rng.uniform(size=len(mq))
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    mbits, mprob, _ = ctx.sample_marginal(mq, Am, Dm, um)
    t_marg = time.perf_counter() - t0
    a64 = out64.cpu().numpy()
    a32 = out32.cpu().numpy()
    c64 = a64[:, 0] + 1j * a64[:, 1]
    c32 = a32[:, 0] + 1j * a32[:, 1]
    rms = float(np.sqrt(np.mean(np.abs(c64) ** 2)))
    ctx.close()
    ms_ev, ms_32, ms_64 = float(np.mean(t_ev)), float(np.mean(t_32)), float(np.mean(t_64))
    # A CCZ slot is six conditional gates (its branches' net gates): CZ_ab, CZ_ac,
    # CZ_bc, each applied by four of the eight equally weighted branches, and
    # S^2 on a, b, c, each applied by two: 1.5 CZ (4 ops) + 0.75 S-type (3 ops)
    # = 8.25 int32 ops per CCZ per evolved state.
    ops_ev = float(st["H"] * (28 * n + 40) + st["CX"] * 12 + st["CZ"] * 4 + st["S"] * 3
                   + st["cond"] / 6 * 8.25)
    ops_sv = table_ops_evolve(st, n)
    evals = float(chi * n_x)
    achieved = ops_sv / (ms_ev / 1e3) / 1e12
    return {"workload": cfg["name"] + f": n={n}, {cfg['n_ccz']} CCZ (8 Clifford branches each), "
                                      f"{int((circ.op != W.OP_CCZ).sum())} Clifford gates, chi={chi} sparsified "
                                      "(delta=0.3), s + 4095 strings drawn from the terms",
            "chi": chi, "n_x": n_x, "ms_evolve": ms_ev, "ms_amplitudes_fp32c": ms_32,
            "ms_amplitudes_fp64": ms_64, "evals_per_s_fp32c": evals / (ms_32 / 1e3),
            "evals_per_s_step": evals / ((ms_ev + ms_32) / 1e3),
            "amplitude_at_s": [float(c64[0].real), float(c64[0].imag)],
            "sparsification_bound": {"omega_norm2_estimate": est, "omega_norm2_sem": sem, "delta2": delta2,
                                     "bound_psi_minus_omega_sq": bound,
                                     # psi = |s>: ||psi - Omega||^2 = <Omega|Omega> - 2 Re<s|Omega> + 1
                                     "psi_minus_omega_sq_from_estimate": est - 2 * float(c64[0].real) + 1,
                                     "equatorial_states": 1024, "seconds": t_bound},
            "marginal_sampling": {"qubits": mq, "bits": mbits.tolist(),
                                  "shift_bits": [int(cfg["s"] >> q & 1) for q in mq],
                                  "conditional_probabilities": [round(float(p), 4) for p in mprob],
                                  "equatorial_states_per_estimate": 256, "norm_estimates": 2 * len(mq),
                                  "seconds": t_marg},
            "fp32c_vs_fp64_normwise": float(np.max(np.abs(c32 - c64)) / rms) if rms > 0 else 0.0,
            "evolve_shape": shape_name(lanes),
            "evolve_prefix_share": {"mode": pf_mode, "checkpoint_levels": pf_levels,
                                    "estimated_work_fraction": round(pf_frac, 4), "distinct_prefixes": st["distinct"],
                                    "gate_applications": {k: st[k] for k in ("H", "CX", "CZ", "S", "cond")}},
            "evolve_roofline": roof("alu", achieved, INT32_PEAK_OPS / 1e12, "TOP/s (int32)", MEASURED.get("valu"),
                                    ops_per_launch=ops_sv,
                                    count="35 n per executed Hadamard, 10 per other gate application",
                                    ops_own_count=ops_ev,
                                    frac_own_count=round(ops_ev / (ms_ev / 1e3) / INT32_PEAK_OPS, 4))}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=10)
    ap.add_argument("--warmup", type=int, default=2)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--cpu-sample-terms", type=int, default=32768)
    ap.add_argument("--sections", default="amplitudes,norm,inner_ch,metropolis,uneven,hidden_shift",
                    help="comma list: amplitudes (the timed step), norm, inner_ch, metropolis, uneven, "
                         "hidden_shift")
    ap.add_argument("--copy-calibration", action="store_true",
                    help="run one plain 1 GiB device copy first (outside the timed region), so that "
                         "hardware byte counters can be scaled against a kernel of known traffic")
    ap.add_argument("--evolve-lanes", type=lambda v: int(v, 0), default=-1,
                    help="evolution mapping: -1 autotunes during warmup (default); otherwise a lanes "
                         "value (e.g. 0x108 = 8 lanes per term, columns in registers), so that counter runs "
                         "repeat the launches of a timed run")
    args = ap.parse_args()
    if args.gpus != 1:
        print(json.dumps({"error": "bench.py runs on one GPU; sharding the terms over several GPUs is designed but not built",
                          "n_gpus": args.gpus}), flush=True)
        sys.exit(2)

    import torch

    from paper_1808_00128_amd import binding as B
    from paper_1808_00128_amd import workloads as W

    assert torch.cuda.is_available(), "bench.py needs a GPU"
    torch.cuda.init()
    dev = torch.device("cuda:0")
    progress("measuring peaks (int32 VALU, HBM copy, LDS reads)")
    pk = B.measure_peaks(0)
    MEASURED.update(valu=pk["int32_valu_ops_per_s"] / 1e12, hbm=pk["hbm_copy_bytes_per_s"] / 1e9,
                    lds=pk["lds_read_bytes_per_s"] / 1e12)
    cfg = W.config_amplitudes()
    circ = cfg["circuit"]
    n, chi, xs = circ.n, cfg["chi"], cfg["x"]
    n_x = xs.size
    if args.copy_calibration:
        src = torch.empty(1 << 27, dtype=torch.float64, device=dev).fill_(1.0)
        dst = torch.empty_like(src)
        torch.cuda.synchronize()
        dst.copy_(src)
        torch.cuda.synchronize()
        del src, dst
    ctx = B.Context([cfg])
    ctx.set_evolve_lanes(args.evolve_lanes)  # -1: autotune the mapping during warmup
    gates = B.gate_array(circ)
    x_dev = torch.from_numpy(xs.view(np.int64)).to(dev)
    out32 = torch.empty((n_x, 2), dtype=torch.float64, device=dev)
    out64 = torch.empty((n_x, 2), dtype=torch.float64, device=dev)
    stream = torch.cuda.current_stream()

    ev = [torch.cuda.Event(enable_timing=True) for _ in range(4)]
    phase = {"reset": [], "evolve": [], "amplitudes": []}

    def step(i, record):
        if record:
            ev[0].record(stream)
        ctx.reset(cfg["seed"] + i)
        if record:
            ev[1].record(stream)
        ctx.apply_gates(gates)
        if record:
            ev[2].record(stream)
        ctx.amplitudes(x_dev, fp32c=True, out=out32)
        if record:
            ev[3].record(stream)
            torch.cuda.synchronize()
            phase["reset"].append(ev[0].elapsed_time(ev[1]))
            phase["evolve"].append(ev[1].elapsed_time(ev[2]))
            phase["amplitudes"].append(ev[2].elapsed_time(ev[3]))

    for i in range(max(1, args.warmup)):
        step(i, False)
    lanes, tune_ms = ctx.evolve_lanes()
    pf_mode, pf_levels, pf_frac = ctx.prefix_share()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for i in range(args.steps):
        step(args.warmup + i, True)
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    ms_step = (t1 - t0) * 1e3 / args.steps
    value = chi * n_x / (ms_step / 1e3)

    # FP64 path on the same terms (outside the timed region).
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    fp64_ms = []
    for _ in range(3):
        e0.record(stream)
        ctx.amplitudes(x_dev, fp32c=False, out=out64)
        e1.record(stream)
        torch.cuda.synchronize()
        fp64_ms.append(e0.elapsed_time(e1))
    a32 = out32.cpu().numpy()
    a64 = out64.cpu().numpy()
    c32 = a32[:, 0] + 1j * a32[:, 1]
    c64 = a64[:, 0] + 1j * a64[:, 1]
    rms = float(np.sqrt(np.mean(np.abs(c64) ** 2)))
    fp32c_vs_fp64 = float(np.max(np.abs(c32 - c64)) / rms) if rms > 0 else 0.0

    ev_stats = ctx.evolution_stats()
    ops_ev = algorithmic_ops_evolve(ev_stats, n)
    ops_sv = table_ops_evolve(ev_stats, n)
    ops_amp = algorithmic_ops_amp(xs) * chi * n_x
    ms_ev = float(np.mean(phase["evolve"]))
    ms_amp = float(np.mean(phase["amplitudes"]))
    ms_reset = float(np.mean(phase["reset"]))
    executed_apps = sum(ev_stats[k] for k in ("H", "CX", "CZ", "S", "cond"))
    if ms_ev >= ms_amp:
        dom = (f"{'k_evolve_cols' if lanes & B.CHSIM_EVOLVE_LDS else 'k_evolve'}<{lanes & 0xff},...> "
               f"(CH-form evolution, {shape_name(lanes)}; all evolution launches of one step)")
        traffic = counter_traffic("k_evolve_cols" if lanes & B.CHSIM_EVOLVE_LDS else "k_evolve")
        roofline = roof("alu", ops_sv / (ms_ev / 1e3) / 1e12, INT32_PEAK_OPS / 1e12, "TOP/s (int32)",
                        MEASURED.get("valu"), kernel=dom, traffic=traffic,
                        traffic_unit="bytes per launch (rocprofv3 FETCH_SIZE x 2 + WRITE_SIZE)",
                        ops_per_launch=ops_sv, ms_per_launch=round(ms_ev, 4),
                        count="35 n int32 ops per executed Hadamard application, 10 per other gate "
                              "application (executed: per term or per shared prefix state)",
                        ops_own_count=ops_ev,
                        own_count="per rule as implemented: H 28 n + 40, CX 12, CZ 4, S-type 3, general 12",
                        frac_own_count=round(ops_ev / (ms_ev / 1e3) / INT32_PEAK_OPS, 4))
    else:
        dom = "k_amp_mfma<float> + k_amp_mfma_reduce (amplitudes, FP32C)"
        roofline = roof("alu", ops_amp / (ms_amp / 1e3) / 1e12, INT32_PEAK_OPS / 1e12, "TOP/s (int32)",
                        MEASURED.get("valu"), kernel=dom, traffic=counter_traffic("k_amp_mfma<float>"),
                        ops_per_launch=ops_amp, ms_per_launch=round(ms_amp, 4),
                        count="8 |x| + 35 int32 ops per (term, x)")

    result = {
        "metric": "term-amplitude evals/s (chi*|x|/s)",
        "value": value,
        "unit": "evals/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms_step,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "u64 GF(2) core + fp32 two-sum, fp64 across blocks",
        "data": "synthetic",
        "config": {"workload": cfg["name"] + ": n=50, 2000 uniform {H,S,CX,CZ} + 40 phase slots "
                               "theta~U(0,2pi), sparsified chi=65536, 4096 uniform x, FP32C",
                   "n": n, "chi": chi, "n_x": n_x, "clifford_gates": int((circ.op != 4).sum()),
                   "phase_slots": circ.n_slot, "parallelism": "single GPU"},
        "phases_ms": {"reset": ms_reset, "evolve": ms_ev, "amplitudes_fp32c": ms_amp,
                      "amplitudes_fp64": float(np.mean(fp64_ms))},
        "evolve_prefix_share": {"mode": pf_mode, "checkpoint_levels": pf_levels,
                                "estimated_work_fraction": round(pf_frac, 4),
                                "distinct_prefixes": ev_stats["distinct"],
                                "gate_applications": {k: ev_stats[k] for k in ("H", "CX", "CZ", "S", "cond")},
                                "per_term_gate_applications": chi * circ.n_gates},
        "evolve_autotune": {"shape": tuned_name(B, lanes, tune_ms),
                            "ms_by_shape": {shape_name(v): round(t, 4)
                                            for v, t in zip(B.TUNE_SHAPES, tune_ms)}},
        "amplitude_kernel_evals_per_s": chi * n_x / (ms_amp / 1e3),
        "evolve_gates_per_s_per_term_count": chi * circ.n_gates / (ms_ev / 1e3),
        "evolve_gates_per_s_executed": executed_apps / (ms_ev / 1e3),
        "peaks_measured": dict(MEASURED),
        "fp32c_vs_fp64_normwise": fp32c_vs_fp64,
        "roofline": roofline,
        "amplitude_roofline": roof("mfma", amp_fp4_ops_per_pair(n) * chi * n_x / (ms_amp / 1e3) / 1e12,
                                   FP4_PEAK_OPS / 1e12, "TFLOP/s (FP4)",
                                   kernel="k_amp_mfma<float> (with k_amp_mfma_prep, k_amp_mfma_reduce)",
                                   fp4_ops_per_pair=amp_fp4_ops_per_pair(n),
                                   count="128 FP4 operations per step of 64 features, n (n + 1) / 2 + 1 features "
                                         "per (term, x); the support test's groups are not counted",
                                   paper_ops_per_s=round(ops_amp / (ms_amp / 1e3) / 1e12, 3),
                                   paper_count="8 |x| + 35 int32 ops per (term, x) (set-bit loop; this "
                                               "kernel does less work per pair)"),
    }
    ctx.close()
    del ctx
    progress(f"amplitudes step done: {ms_step:.3f} ms per step")
    sections = set(args.sections.split(","))
    if "norm" in sections:
        progress("section norm")
        result["norm_estimation"] = bench_norm(torch, B, W)
    if "uneven" in sections:
        progress("section uneven")
        result["uneven_batch"] = bench_uneven(torch, B, W)
    if "hidden_shift" in sections:
        progress("section hidden_shift")
        result["hidden_shift_ccz"] = bench_hidden_shift(torch, B, W)
    if "inner_ch" in sections:
        progress("section inner_ch (general stabilizer states)")
        result["inner_products_ch"] = bench_inner_ch(torch, B, W)
    if "metropolis" in sections:
        from paper_1808_00128_amd import stats

        progress("section metropolis (QAOA n=50, plain, training, learned)")
        result["metropolis"] = bench_learned(torch, B, W, stats)
        progress("section metropolis matched TV (n=12 twin)")
        result["metropolis"]["matched_tv"] = bench_matched_tv(torch, B, W, stats)
    if not args.no_cpu_baseline:
        threads = max(1, min(16, os.cpu_count() or 1))
        progress(f"cpu baseline ({threads} threads)")
        result["cpu_baseline"] = cpu_baseline(cfg, args.cpu_sample_terms, threads)
    progress("done")
    print(json.dumps(result), flush=True)


if __name__ == "__main__":
    main()
