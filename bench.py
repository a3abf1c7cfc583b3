#!/usr/bin/env python
"""Benchmark of the batched checkerboard Metropolis sweep on one MI355X.

Workload (the batched configuration of the paper's throughput experiments,
Results, Table 3 / Fig. 3, scaled to one MI355X): 1024 Ising replicas of
256x256 with beta on a 64-point grid over [0.30, 0.60] (16 replicas each),
plus 512 q-state Potts lattices with L drawn from {64, 128, 256, 512, 1024}
and q from {3, 4, 6, 8} at beta ~ U[0.9, 1.1] ln(1 + sqrt q), random initial
states, 10^4 sweeps per step.  Inputs are synthetic (seeded), resident in HBM
before timing starts.

Prints ONE JSON line.  ``value`` is spin-update attempts per ns over the
timed steps (all replicas, both colours; the library's production path of
cached hipGraph replays).  Right after the timed steps the same workload runs
``--prof-sweeps`` more sweeps with every kernel launch bracketed by HIP
events on the stream it is launched on; ``kernels`` lists those per-kernel
times and ``roofline`` reports the kernel with the largest share:

* a streamed Ising colour pass is HBM bound: 3 algorithmic bytes per attempt
  (read the colour's plane and the other plane, write the colour's plane);
* the streamed Potts pass and the LDS-resident kernel are bound by vector
  ALU issue: peak 256 CUs x 4 SIMDs x 16 lanes x 2.4 GHz = 39.3 T
  lane-instructions/s, achieved from the VALU instruction count per attempt
  that rocprofv3 (SQ_INSTS_VALU) measured on the same kernel source.

``traffic`` is the HBM bytes per launch from rocprofv3 FETCH_SIZE and
WRITE_SIZE, each scaled by what the counter reads for a plain device copy of
known size (``--copy-calibration-mib``), taken from the committed counter
summary when its kernel-source hash matches (else null).  ``--summarize-
counters DIR...`` writes that summary from rocprofv3 counter runs of this
script.  ``cpu_baseline`` times the oracle (plain C, OpenMP over replicas) on
the host cores for all replicas of the workload over a few sweeps, and on one
thread for a strided subset of the replicas.
"""
import argparse
import csv
import hashlib
import json
import os
import statistics
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0
VALU_PEAK = 256 * 4 * 16 * 2.4e9   # lane-instructions / s
BYTES_PER_ATTEMPT = 3              # streamed pass: read own + other plane, write own plane
COUNTERS = os.path.join(ROOT, "profiles", "counters_batched_ising_potts.json")
KERNEL_NAMES = {"stream_ising": "k_stream_pass_ising", "stream_potts": "k_stream_pass_potts",
                "resident": "k_resident", "persist_ising": "k_persist_ising",
                "persist_potts": "k_persist_potts"}
# kernels whose work is streamed colour passes (3 algorithmic HBM bytes per
# attempt); the HBM-bound ones among them
STREAMED = ("stream_ising", "stream_potts", "persist_ising", "persist_potts")
HBM_BOUND = ("stream_ising", "persist_ising")


def kernel_source_hash():
    h = hashlib.sha256()
    for f in ("lattice_kernels.hip", "item8.hpp", "spinmc_internal.hpp"):
        with open(os.path.join(ROOT, "paper_2304_01772_amd", "csrc", f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


def counter_entry(mode, kernel):
    """Per-attempt counters of one kernel under one schedule mode from the
    committed summary, or None if absent or taken on other kernel source."""
    if not os.path.exists(COUNTERS):
        return None
    with open(COUNTERS) as f:
        d = json.load(f)
    if d.get("kernel_source_hash") != kernel_source_hash():
        return None
    return d.get("modes", {}).get(mode, {}).get(kernel)


def roofline(kind, k, mode_name):
    """Roofline entry of one kernel kind from its live timing k (ms,
    launches, attempts per launch)."""
    avg_s = k["ms"] / k["launches"] * 1e-3
    att = k["attempts_per_launch"]
    kernel = KERNEL_NAMES[kind]
    ce = counter_entry(mode_name, kernel)
    traffic = None
    if ce and ce.get("fetch_bytes_per_attempt") is not None \
            and ce.get("write_bytes_per_attempt") is not None:
        traffic = int(round((ce["fetch_bytes_per_attempt"] + ce["write_bytes_per_attempt"]) * att))
    out = {"kernel": kernel, "launches": k["launches"], "avg_launch_us": round(avg_s * 1e6, 2),
           "attempts_per_launch": att, "attempts_per_ns": round(att / avg_s / 1e9, 1)}
    if kind in HBM_BOUND:
        b = BYTES_PER_ATTEMPT * att
        ach = b / avg_s / 1e9
        out.update(bound="hbm", achieved=round(ach, 1), peak=HBM_PEAK_GBS, unit="GB/s",
                   frac=round(ach / HBM_PEAK_GBS, 4), traffic=traffic, bytes_per_launch=b)
    else:
        out.update(bound="alu", achieved=None, peak=round(VALU_PEAK / 1e12, 2),
                   unit="T lane-instr/s", frac=None, traffic=traffic)
        if ce and ce.get("valu_lane_instr_per_attempt"):
            per = ce["valu_lane_instr_per_attempt"]
            ach = per * att / avg_s
            out.update(achieved=round(ach / 1e12, 2), frac=round(ach / VALU_PEAK, 4),
                       valu_lane_instr_per_attempt=per)
        if ce and ce.get("valu_busy_pct") is not None:
            # hardware VALU-busy share of the kernel's time (rocprofv3 VALUBusy)
            out["valu_busy_pct_counter"] = ce["valu_busy_pct"]
    if kind in STREAMED:
        # every streamed kernel priced against HBM as well (3 algorithmic bytes
        # per attempt), next to the fraction of its own bound
        gbs = BYTES_PER_ATTEMPT * att / avg_s / 1e9
        out["hbm_GBs_algorithmic"] = round(gbs, 1)
        out["frac_hbm"] = round(gbs / HBM_PEAK_GBS, 4)
        if traffic is not None:
            out["hbm_GBs_measured"] = round(traffic / avg_s / 1e9, 1)
            out["frac_hbm_measured"] = round(traffic / avg_s / 1e9 / HBM_PEAK_GBS, 4)
    return out


def profiled_kernels(smp, torch, sweeps):
    """Run `sweeps` sweeps with per-launch HIP-event timing; returns
    {kind: {ms, launches, avg_us, attempts_per_launch}}."""
    st, re_ = smp.schedule_sites(by_model=True)
    smp.profile(True)
    smp.sweep(sweeps)
    torch.cuda.synchronize()
    total = {"stream_ising": st["ising"] // 2 * 2 * sweeps,
             "stream_potts": st["potts"] // 2 * 2 * sweeps,
             "persist_ising": st["ising"] * sweeps, "persist_potts": st["potts"] * sweeps,
             "resident": (re_["ising"] + re_["potts"]) * sweeps}
    kern = {}
    for kind in ("stream_ising", "stream_potts", "persist_ising", "persist_potts", "resident"):
        kms, nl = smp.profile_read(kind)
        if nl:
            kern[kind] = dict(ms=round(kms, 3), launches=nl, avg_us=round(kms / nl * 1e3, 2),
                              attempts_per_launch=total[kind] // nl)
    smp.profile(False)
    return kern


def ising_stream_probe(Sampler, torch, n_rep, sweeps, schedule=None):
    """The batched Ising sweep alone, streamed through HBM (n_rep replicas of
    256x256, the beta grid of the workload), timed per colour-pass launch;
    the stream schedule is autotuned unless given."""
    import synth
    reps = synth.batched_ising_potts(n_ising=n_rep, n_potts=0)
    smp = Sampler(reps, seed=2, init=True)
    if schedule:
        smp.set_schedule(mode="stream", **schedule)
        chosen = smp.get_schedule()
    else:
        chosen, _ = smp.autotune(trial_sweeps=10, mode="stream")
    smp.sweep(2)
    torch.cuda.synchronize()
    st_m, re_m = smp.schedule_sites(by_model=True)
    kern = profiled_kernels(smp, torch, sweeps)
    smp.close()
    kind = "persist_ising" if "persist_ising" in kern else "stream_ising"
    out = roofline(kind, kern[kind], f"ising_probe_{n_rep}")
    out["units"] = f"{n_rep} Ising 256x256 replicas, {sweeps} sweeps"
    if kind == "persist_ising":
        # one launch runs all passes of a chunk: per colour pass
        out["us_per_pass"] = round(out["avg_launch_us"] * k_launch_passes(kern[kind], sweeps), 2)
    out["schedule"] = chosen
    out["kernels"] = kern
    return out, dict(streamed_sites_by_model=st_m, resident_sites_by_model=re_m,
                     schedule=chosen)


def k_launch_passes(k, sweeps):
    """1 / colour passes per launch of a persistent kernel timed over
    `sweeps` sweeps (2 passes per sweep)."""
    return k["launches"] / (2.0 * sweeps)


def _events(torch, stream):
    a = torch.cuda.Event(enable_timing=True)
    b = torch.cuda.Event(enable_timing=True)
    a.record(stream)
    return a, b


def cpm_probe(Sampler, torch, mcs):
    """Cell sorting: 8 CPM replicas of 512x512 (1000 cells of 14x14, two
    types, A = 200, lambda = 1, T = 10), `mcs` Monte Carlo steps (4 colour
    passes each) timed per pass launch."""
    import synth
    ids, ctype, A, J, prm = synth.cpm_sorting()
    reps = [dict(model=2, Lx=ids.shape[2], Ly=ids.shape[1], q=len(ctype) - 1, rid=r, adhesion=J,
                 cell_type=ctype, target_area=A, lambda_area=prm["lambda_area"],
                 temperature=prm["temperature"]) for r in range(ids.shape[0])]
    smp = Sampler(reps, prm["seed"], init=False)
    for r in range(len(reps)):
        smp.set_state(r, ids[r])
    chosen, _ = smp.autotune(trial_sweeps=10)
    smp.sweep(mcs)  # warm-up at the timed length (captures its graph)
    torch.cuda.synchronize()
    e0, e1 = _events(torch, smp.stream)
    smp.sweep(mcs)
    e1.record(smp.stream)
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1)
    smp.profile(True)
    smp.sweep(mcs)
    torch.cuda.synchronize()
    kms, nl = smp.profile_read("cpm_pass")
    kind = {0: "k_cpm_pass_tile (two phases on LDS tiles, one launch per colour pass)",
            512: "k_cpm_pass_site (one site per lane, one launch per colour pass)"}.get(
                chosen.get("wg_threads", 0),
                "k_cpm_pass_quad (one quad per lane, one launch per colour pass)")
    per_launch = ids.size // 4
    if nl == 0:  # the tiled persistent passes: one launch for all passes of the call
        kms, nl = smp.profile_read("cpm_tiled")
        kind, per_launch = "k_cpm_tiled (one launch per chunk)", ids.size * mcs // nl
    smp.profile(False)
    smp.close()
    sites = ids.shape[0] * ids.shape[1] * ids.shape[2]
    avg_s = kms / nl * 1e-3
    return {"config": f"{ids.shape[0]} CPM replicas of {ids.shape[1]}x{ids.shape[2]}, "
                      f"1000 cells, {mcs} MCS (graph replays)", "schedule": chosen,
            "attempts_per_ns": round(sites * mcs / (ms * 1e6), 2),
            "kernel": kind, "bound": "alu", "launches": nl,
            "avg_launch_us": round(avg_s * 1e6, 2),
            "kernel_attempts_per_ns": round(per_launch / avg_s / 1e9, 2),
            "algorithmic_GBs": round(per_launch * 17 / avg_s / 1e9, 1)}


def cpm_paper_probe(Sampler, torch, n_rep=256, mcs=2000):
    """The paper's own CPM setting (Results, Table 2) batched: n_rep replicas
    of the 6 x 6 aggregate of 5 x 5 cells in 64 x 64, k_B T = 8, A = 25,
    lambda = 1, for `mcs` Monte Carlo steps; rate and mean boundary lengths
    (von Neumann bonds) by type pair at the start and the end."""
    import synth
    ids, types, A, J, prm = synth.cpm_paper_aggregate(n_rep=n_rep)
    reps = [dict(model=2, Lx=ids.shape[2], Ly=ids.shape[1], q=len(types[r]) - 1, rid=r,
                 adhesion=J, cell_type=types[r], target_area=A,
                 lambda_area=prm["lambda_area"], temperature=prm["temperature"])
            for r in range(n_rep)]
    smp = Sampler(reps, prm["seed"], init=False)
    for r in range(n_rep):
        smp.set_state(r, ids[r])
    b0, _ = smp.measure()
    b0 = b0.float().mean(0).cpu()
    smp.sweep(50)  # warm-up: captures the 50-step graph
    torch.cuda.synchronize()
    e0, e1 = _events(torch, smp.stream)
    smp.sweep(mcs)
    e1.record(smp.stream)
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1)
    b1, _ = smp.measure()
    b1 = b1.float().mean(0).cpu()
    smp.close()
    sites = n_rep * ids.shape[1] * ids.shape[2]
    names = {1: "light-medium", 2: "dark-medium", 4: "light-dark"}
    out = {"config": f"{n_rep} replicas of {ids.shape[1]}x{ids.shape[2]}, 36 cells of 5x5, "
                     f"Table 2 adhesion, kT 8, A 25, lambda 1, {mcs + 50} MCS",
           "attempts_per_ns": round(sites * mcs / (ms * 1e6), 2),
           "boundary_start": {v: round(float(b0[k]), 1) for k, v in names.items()},
           "boundary_end": {v: round(float(b1[k]), 1) for k, v in names.items()}}
    # the same aggregate with the 5x5 neighbourhood (66 x 66: multiples of 6)
    ids, types, A, J, prm = synth.cpm_paper_aggregate(n_rep=n_rep, L=66)
    reps = [dict(model=2, Lx=66, Ly=66, q=len(types[r]) - 1, rid=r, adhesion=J,
                 cell_type=types[r], target_area=A, lambda_area=prm["lambda_area"],
                 temperature=prm["temperature"], cpm_range=2) for r in range(n_rep)]
    smp = Sampler(reps, prm["seed"], init=False)
    for r in range(n_rep):
        smp.set_state(r, ids[r])
    smp.sweep(50)
    torch.cuda.synchronize()
    e0, e1 = _events(torch, smp.stream)
    smp.sweep(mcs // 4)
    e1.record(smp.stream)
    torch.cuda.synchronize()
    ms5 = e0.elapsed_time(e1)
    smp.close()
    out["range2_5x5"] = {"config": f"{n_rep} replicas of 66x66, {mcs // 4} MCS (9 passes each) "
                                   "after 50",
                         "attempts_per_ns": round(n_rep * 66 * 66 * (mcs // 4) / (ms5 * 1e6), 2)}
    return out


def tri_probe(Sampler, torch, n_rep=1024, L=96, sweeps=200):
    """Triangular-lattice Ising: n_rep replicas of L x L at the exact
    critical coupling beta_c = ln(3)/4 (J = 1), `sweeps` sweeps of three
    colour passes; algorithmic HBM bytes 4 per attempt (a pass reads the
    lattice once, 3 B per attempt of its colour, and writes the colour's
    sites, 1 B)."""
    import math
    reps = [dict(model=3, Lx=L, Ly=L, Jx=1.0, Jy=1.0, h=0.0, beta=math.log(3.0) / 4, rid=r)
            for r in range(n_rep)]
    smp = Sampler(reps, 11, init=True)
    smp.sweep(5)
    torch.cuda.synchronize()
    e0, e1 = _events(torch, smp.stream)
    smp.sweep(sweeps)
    e1.record(smp.stream)
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1)
    # recorded sweeps (statistics every sweep, still resident)
    rec = torch.empty((sweeps, n_rep, smp.width), dtype=torch.int32, device="cuda")
    e2, e3 = _events(torch, smp.stream)
    smp.sweep(sweeps, 1, stats=rec)
    e3.record(smp.stream)
    torch.cuda.synchronize()
    ms_rec = e2.elapsed_time(e3)
    # the streamed colour passes alone (the schedule for lattices beyond LDS)
    smp.set_schedule(mode="stream")
    smp.profile(True)
    smp.sweep(20)
    torch.cuda.synchronize()
    kms, nl = smp.profile_read("tri_pass")
    smp.profile(False)
    smp.close()
    sites = n_rep * L * L
    per_launch = sites / 3
    avg_s = kms / nl * 1e-3
    gbs = per_launch * 4 / avg_s / 1e9
    return {"config": f"{n_rep} triangular replicas of {L}x{L}, beta_c = ln(3)/4, {sweeps} sweeps",
            "attempts_per_ns": round(sites * sweeps / (ms * 1e6), 1),
            "recorded_attempts_per_ns": round(sites * sweeps / (ms_rec * 1e6), 1),
            "kernel": "k_plane_resident (lattices in LDS)",
            "stream_pass": {"kernel": "k_tri_pass4", "avg_launch_us": round(avg_s * 1e6, 2),
                            "attempts_per_ns": round(per_launch / avg_s / 1e9, 1),
                            "GBs_algorithmic": round(gbs, 1),
                            "frac_hbm": round(gbs / HBM_PEAK_GBS, 4)}}


def hc_probe(Sampler, torch, n_rep=256, L=32, sweeps=200):
    """Simple-cubic Ising: n_rep replicas of L^3 near the 3D critical
    coupling (beta 0.2216546, J = 1), `sweeps` sweeps of two colour passes;
    algorithmic HBM bytes 3 per attempt (a pass reads the lattice once, 2 B
    per attempt of its colour, and writes the colour's sites, 1 B)."""
    reps = [dict(model=4, Lx=L, Ly=L, Lz=L, Jx=1.0, Jy=1.0, h=0.0, beta=0.2216546, rid=r)
            for r in range(n_rep)]
    smp = Sampler(reps, 12, init=True)
    smp.sweep(5)
    torch.cuda.synchronize()
    e0, e1 = _events(torch, smp.stream)
    smp.sweep(sweeps)
    e1.record(smp.stream)
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1)
    rec = torch.empty((sweeps, n_rep, smp.width), dtype=torch.int32, device="cuda")
    e2, e3 = _events(torch, smp.stream)  # recorded sweeps, still resident
    smp.sweep(sweeps, 1, stats=rec)
    e3.record(smp.stream)
    torch.cuda.synchronize()
    ms_rec = e2.elapsed_time(e3)
    smp.set_schedule(mode="stream")
    smp.profile(True)
    smp.sweep(20)
    torch.cuda.synchronize()
    kms, nl = smp.profile_read("hc_pass")
    smp.profile(False)
    smp.close()
    sites = n_rep * L ** 3
    avg_s = kms / nl * 1e-3
    gbs = sites / 2 * 3 / avg_s / 1e9
    return {"config": f"{n_rep} simple-cubic replicas of {L}^3, beta 0.2216546, {sweeps} sweeps",
            "attempts_per_ns": round(sites * sweeps / (ms * 1e6), 1),
            "recorded_attempts_per_ns": round(sites * sweeps / (ms_rec * 1e6), 1),
            "kernel": "k_plane_resident (lattices in LDS)",
            "stream_pass": {"kernel": "k_hc_pass4", "avg_launch_us": round(avg_s * 1e6, 2),
                            "attempts_per_ns": round(sites / 2 / avg_s / 1e9, 1),
                            "GBs_algorithmic": round(gbs, 1),
                            "frac_hbm": round(gbs / HBM_PEAK_GBS, 4)}}


def msc_probe(Sampler, torch, n_groups=256, L=256, sweeps=200):
    """Multispin-coded Ising: n_groups groups of 32 replicas (8192 replicas
    of L x L for the defaults) at beta 0.4407, `sweeps` sweeps; the 32
    replicas of a group share each site's random word.  Groups that fit run
    resident in registers and LDS; a streamed pass has algorithmic HBM bytes
    0.375 per attempt (it reads the words once, 4 B per site, and writes the
    colour's words, 2 B per site, for 16 attempts per site)."""
    reps = [dict(model=5, Lx=L, Ly=L, Jx=1.0, Jy=1.0, h=0.0, beta=0.4407, rid=g)
            for g in range(n_groups)]
    smp = Sampler(reps, 13, init=True)
    smp.sweep(5)
    torch.cuda.synchronize()
    e0, e1 = _events(torch, smp.stream)
    smp.sweep(sweeps)
    e1.record(smp.stream)
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1)
    # the streamed colour passes alone (the schedule for lattices beyond a workgroup)
    smp.set_schedule(mode="stream")
    smp.profile(True)
    smp.sweep(20)
    torch.cuda.synchronize()
    kms, nl = smp.profile_read("msc_pass")
    smp.profile(False)
    smp.close()
    attempts = 32 * n_groups * L * L
    avg_s = kms / nl * 1e-3
    per_launch = attempts / 2
    gbs = per_launch * 0.375 / avg_s / 1e9
    return {"config": f"{n_groups} groups x 32 replicas of {L}x{L} (shared random words), "
                      f"beta 0.4407, {sweeps} sweeps",
            "attempts_per_ns": round(attempts * sweeps / (ms * 1e6), 1),
            "kernel": "k_msc_resident (lattices in registers)",
            "stream_pass": {"kernel": "k_msc_pass4", "avg_launch_us": round(avg_s * 1e6, 2),
                            "attempts_per_ns": round(per_launch / avg_s / 1e9, 1),
                            "GBs_algorithmic": round(gbs, 1),
                            "frac_hbm": round(gbs / HBM_PEAK_GBS, 4)}}


def grad_probe(Sampler, torch):
    """Differentiation workload: 256 Ising replicas of 128x128 (J ~ U(0.3,
    0.6), h ~ U(-0.05, 0.05), beta 1), 5000 recorded sweeps, then the
    covariance backward over the 4000 post-burn-in samples."""
    import synth
    reps = synth.differentiation()
    smp = Sampler(reps, 3, init=True)
    n, burn = 5000, 1000
    stats = torch.empty((n, len(reps), smp.width), dtype=torch.int32, device="cuda")
    smp.sweep(10)
    torch.cuda.synchronize()
    e0, e1 = _events(torch, smp.stream)
    smp.sweep(n, 1, stats=stats)
    e1.record(smp.stream)
    gout = torch.ones((len(reps), 2), dtype=torch.float64, device="cuda")
    smp.grad(stats, burn, grad_out=gout)
    torch.cuda.synchronize()
    ms_sweep = e0.elapsed_time(e1)
    ms_grad = float("inf")
    for _ in range(5):  # one launch per bracket, best of five
        e2, e3 = _events(torch, smp.stream)
        smp.grad(stats, burn, grad_out=gout)
        e3.record(smp.stream)
        torch.cuda.synchronize()
        ms_grad = min(ms_grad, e2.elapsed_time(e3))
    smp.close()
    sites = sum(r["Lx"] * r["Ly"] for r in reps)
    samples = (n - burn) * len(reps)
    return {"config": "256 Ising 128x128, 5000 recorded sweeps, burn-in 1000",
            "recorded_sweep_attempts_per_ns": round(sites * n / (ms_sweep * 1e6), 1),
            "kernel": "k_cov_partial + k_cov_final (chunk sums, then per replica)", "bound": "hbm",
            "grad_call_us": round(ms_grad * 1e3, 2),
            "samples": samples, "algorithmic_bytes": 12 * samples,
            "achieved_GBs": round(12 * samples / (ms_grad * 1e-3) / 1e9, 1)}


def mlp_probe(torch, steps=200, batch=1024, infer_batch=100_000):
    """Surrogate MLP 4-128-128-3: training steps (forward + backward + Adam)
    at batch 1024 and one forward over 10^5 points, timed with HIP events."""
    from paper_2304_01772_amd.surrogate import SurrogateMLP
    net = SurrogateMLP(seed=0)
    g = torch.Generator(device="cpu").manual_seed(0)
    xn = (torch.rand((batch, 4), generator=g) * 2 - 1).cuda().contiguous()
    tn = torch.randn((batch, 3), generator=g).cuda().contiguous()
    w = torch.ones(3, dtype=torch.float32, device="cuda")
    for _ in range(5):
        net.train_step(xn, tn, w)
    torch.cuda.synchronize()
    st = torch.cuda.current_stream()
    e0, e1 = _events(torch, st)
    for _ in range(steps):
        net.train_step(xn, tn, w)
    e1.record(st)
    xi = (torch.rand((infer_batch, 4), generator=g) * 2 - 1).cuda().contiguous()
    net.forward_normalised(xi)
    torch.cuda.synchronize()
    e2, e3 = _events(torch, st)
    net.forward_normalised(xi)
    e3.record(st)
    torch.cuda.synchronize()
    ms_train = e0.elapsed_time(e1) / steps
    ms_inf = e2.elapsed_time(e3)
    fwd = 2 * (4 * 128 + 128 * 128 + 128 * 3)
    train = 3 * fwd
    return {"config": "4-128-128-3 bf16 MFMA, fp32 accumulate and master weights",
            "train_step_us": round(ms_train * 1e3, 2), "train_batch": batch,
            "train_TFLOPs": round(train * batch / (ms_train * 1e-3) / 1e12, 3),
            "forward_points": infer_batch, "forward_ms": round(ms_inf, 3),
            "forward_TFLOPs": round(fwd * infer_batch / (ms_inf * 1e-3) / 1e12, 2),
            "bound": "mfma", "peak_TFLOPs": 2500.0}


def surrogate_probe(torch, n_points=100_000):
    """The learned surrogate's inverse problem against Monte Carlo alone
    (the learned-surrogate workload): labels for n_points parameter points
    (beta, Jx, Jy, h) by batched Monte Carlo on 64x64 Ising (1000 + 2000
    sweeps), training of the 4-128-128-3 network on the MLP kernels, then
    for each target <|m|> at beta 0.4 the wall time to Monte-Carlo-verified
    1 % error of the surrogate-steered solve and of the Monte-Carlo-only
    solve (the same bracketed Newton iteration from the same start; every
    evaluation resolved to a standard error of 0.25 % of the target)."""
    from paper_2304_01772_amd import surrogate as sg
    res = sg.experiment(n_points=n_points, log=lambda m: print(f"# surrogate: {m}",
                                                               file=sys.stderr, flush=True))
    rows = []
    for r in res["solves"]:
        t = r["target"]
        row = {"target": t}
        for k in ("mc_only", "surrogate"):
            v = r[k]
            row[k] = {"seconds": round(v["seconds"], 3), "absm_mc": round(v["absm"], 5),
                      "se_mc": round(v["se"], 5),
                      "rel_error_mc": round(abs(v["absm"] - t) / t, 5),
                      "mc_evaluations": v["iters"], "replicas": v["replicas"],
                      "converged": v["converged"], "Jx": round(v["Jx"], 5),
                      "Jy": round(v["Jy"], 5)}
        row["surrogate"]["fallback_mc_steps"] = r["surrogate"]["fallback_iters"]
        rows.append(row)
    tot = res["total_seconds"]
    return {"config": dict(res["config"], targets=[r["target"] for r in res["solves"]],
                           protocol="find (Jx, Jy) with <|m|>(beta 0.4, Jx, Jy, h 0) = target "
                                    "within 1 % relative, verified by Monte Carlo; both "
                                    "solvers start at (1, 1)"),
            "label_seconds": round(res["label_seconds"], 3),
            "train_seconds": round(res["train_seconds"], 3),
            "validation": {k: round(v, 5) for k, v in res["validation"].items()},
            "solves": rows,
            "all_converged": all(r["mc_only"]["converged"] and r["surrogate"]["converged"]
                                 for r in rows),
            "total_seconds": {k: round(v, 3) for k, v in tot.items()},
            "speedup_without_one_off": round(tot["mc_only"] / tot["surrogate"], 3),
            "speedup_with_labels_and_training": round(
                tot["mc_only"] / tot["surrogate_with_labels_and_training"], 3)}


def dmc_probe(torch, R=256, L=128, sweeps=10):
    """Differentiable Monte Carlo (relaxed chain of Algorithm 2): R replicas
    of L x L with per-bond couplings, `sweeps` sweeps forward and the reverse
    replay, timed with HIP events (best of five calls); algorithmic HBM bytes with the
    lattices resident: forward 4 per attempt (the saved spin) and 20 per site
    and call (spin and two couplings read, the final spin written to both
    outputs, the replay's and the caller's), backward 4 per
    attempt and 28 per site and call (output spin and its gradient, two
    couplings read; three gradients written)."""
    from paper_2304_01772_amd.dmc import relaxed_ising
    g = torch.Generator(device="cpu").manual_seed(0)
    s0 = (torch.rand((R, L, L), generator=g) * 2 - 1).cuda()
    jx = (torch.rand((R, L, L), generator=g) * 0.8 + 0.1).cuda().requires_grad_(True)
    jy = (torch.rand((R, L, L), generator=g) * 0.8 + 0.1).cuda().requires_grad_(True)
    for _ in range(2):  # warm-up at the timed size (allocator, first launches)
        out = relaxed_ising(s0, jx, jy, 0.5, 10.0, 0.0, sweeps, 1)
        out.sum().backward()
    torch.cuda.synchronize()
    st = torch.cuda.current_stream()
    fwd_ms = bwd_ms = float("inf")
    for _ in range(5):  # best of five calls: one call is short enough for host jitter to show
        e0, e1 = _events(torch, st)
        out = relaxed_ising(s0, jx, jy, 0.5, 10.0, 0.0, sweeps, 1)
        e1.record(st)
        e2, e3 = _events(torch, st)
        out.sum().backward()
        e3.record(st)
        torch.cuda.synchronize()
        fwd_ms, bwd_ms = min(fwd_ms, e0.elapsed_time(e1)), min(bwd_ms, e2.elapsed_time(e3))
    att = R * L * L * sweeps
    fwd_b, bwd_b = 4 + 20 / sweeps, 4 + 28 / sweeps
    return {"config": f"{R} Ising replicas of {L}x{L}, per-bond couplings, {sweeps} sweeps, "
                      "alpha 10, beta 0.5",
            "kernel": "k_dmc_resident_fwd / k_dmc_resident_bwd", "bound": "alu",
            "forward_attempts_per_ns": round(att / (fwd_ms * 1e6), 1),
            "backward_attempts_per_ns": round(att / (bwd_ms * 1e6), 1),
            "forward_GBs_algorithmic": round(fwd_b * att / (fwd_ms * 1e-3) / 1e9, 1),
            "forward_frac": round(fwd_b * att / (fwd_ms * 1e-3) / 1e9 / HBM_PEAK_GBS, 4),
            "backward_GBs_algorithmic": round(bwd_b * att / (bwd_ms * 1e-3) / 1e9, 1),
            "backward_frac": round(bwd_b * att / (bwd_ms * 1e-3) / 1e9 / HBM_PEAK_GBS, 4)}


def dmc_vs_covariance_probe(torch, R=4096, L=4):
    """d<e>/dJ for uniform couplings on R replicas of the L x L torus: the
    fluctuation (covariance) estimator of the library's backward kernel
    against the differentiable chain's pathwise derivative (alpha 10, 1 and
    5 sweeps after a discretised burn-in).  Exact values come from
    enumeration (2^16 states for 4 x 4) in the tests' helpers."""
    from paper_2304_01772_amd.differentiable import ising_observables
    from paper_2304_01772_amd.dmc import pathwise_energy_gradient
    out = {"config": f"{R} replicas of {L}x{L}, J = 1, h = 0"}
    for beta in (0.2, 0.44, 0.8):
        J = torch.ones(R, dtype=torch.float64, device="cuda", requires_grad=True)
        Jy = torch.ones(R, dtype=torch.float64, device="cuda", requires_grad=True)
        e, _ = ising_observables(J, Jy, torch.zeros(R, dtype=torch.float64, device="cuda"), L,
                                 beta, 2000, 500, 11, 0)
        e.sum().backward()
        d = (J.grad + Jy.grad).double()
        row = {"covariance": [round(float(d.mean()), 4), round(float(d.std() / R ** 0.5), 4)]}
        for n in (1, 5):
            _, m, se = pathwise_energy_gradient(L, R, beta, 10.0, n, 50, 11)
            row[f"pathwise_alpha10_{n}sweeps"] = [round(m, 4), round(se, 4)]
        out[f"beta_{beta}"] = row
    return out


def spinopt_probe(torch, R=64, L=64, steps=200):
    """Spin-value optimisation (Results): annealed Monte Carlo, gradient and
    differentiable Monte Carlo from the same random states over the same
    linear beta schedule 0.3 -> 3, on J = 1 and on +-J couplings; mean final
    and best energy per site and the time per step of each method."""
    from paper_2304_01772_amd.spinopt import SpinOptimiser, spin_glass_couplings
    g = torch.Generator(device="cpu").manual_seed(1)
    s0 = (torch.randint(0, 2, (R, L, L), generator=g).float() * 2 - 1).cuda()
    out = {"config": f"{R} replicas of {L}x{L}, {steps} steps, beta 0.3 -> 3, DMC alpha 20, "
                     "1 sweep per step, eta 0.05; gradient eta 1"}
    for kind in ("ferro", "glass"):
        if kind == "ferro":
            Jx = torch.ones((R, L, L), device="cuda")
            Jy = torch.ones((R, L, L), device="cuda")
        else:
            Jx, Jy = spin_glass_couplings(R, L, L, 7)
        o = SpinOptimiser(Jx, Jy, 0.0, seed=3)
        o.compare(s0, 2)  # warm-up (buffers, first launches)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        res = o.compare(s0, steps)
        torch.cuda.synchronize()
        wall = time.perf_counter() - t0
        out[kind] = {m: {"final": round(float(h[-1].mean()), 4), "best": round(float(b.mean()), 4)}
                     for m, (h, b) in res.items()}
        out[kind]["wall_s_all_methods"] = round(wall, 3)
    return out


def _oracle_rate(reps, seed, sweeps):
    """Wall time of the oracle over `sweeps` sweeps of every replica in
    reps (OpenMP over replicas); returns (attempts/ns, attempts, seconds)."""
    import numpy as np
    from oracle import chain as orc
    ising = [r for r in reps if r["model"] == 0]
    potts = [r for r in reps if r["model"] == 1]
    si = [orc.ising_init(r["Lx"], r["Ly"], seed, r["rid"]) for r in ising]
    sp = [orc.potts_init(r["Lx"], r["Ly"], r["q"], seed, r["rid"]) for r in potts]
    t0 = time.perf_counter()
    if ising:
        orc.ising_run_batch(si, [r["Jx"] for r in ising], [r["Jy"] for r in ising],
                            [r["h"] for r in ising], [r["beta"] for r in ising], seed,
                            np.array([r["rid"] for r in ising]), 0, sweeps)
    if potts:
        orc.potts_run_batch(sp, [r["q"] for r in potts], [r["Jx"] for r in potts],
                            [r["h"] for r in potts], [r["beta"] for r in potts], seed,
                            np.array([r["rid"] for r in potts]), 0, sweeps)
    dt = time.perf_counter() - t0
    att = sum(r["Lx"] * r["Ly"] for r in reps) * sweeps
    return att / dt / 1e9, att, dt


def cpu_baseline(reps, seed, sweeps, single_sweeps=20, single_stride=16):
    """The oracle on the host cores: every replica of the workload for a
    few sweeps on all threads (a bounded sample of the same chain), and
    every single_stride-th replica on one thread."""
    from oracle import chain as orc
    n_thr = orc.num_threads()
    v, att, dt = _oracle_rate(reps, seed, sweeps)
    sub = reps[::single_stride]
    orc.set_num_threads(1)
    try:
        v1, att1, dt1 = _oracle_rate(sub, seed, single_sweeps)
    finally:
        orc.set_num_threads(n_thr)
    return dict(value=v, unit="attempts/ns", cores=n_thr, kind="oracle",
                sample=f"all {len(reps)} replicas of the workload, {sweeps} sweeps "
                       f"({att:.3g} attempts, {dt:.1f} s wall)",
                single_thread=dict(value=v1, unit="attempts/ns", cores=1,
                                   sample=f"every {single_stride}th replica ({len(sub)}: "
                                          f"{sum(r['model'] == 0 for r in sub)} Ising, "
                                          f"{sum(r['model'] == 1 for r in sub)} Potts), "
                                          f"{single_sweeps} sweeps ({att1:.3g} attempts, "
                                          f"{dt1:.1f} s wall)"))


# ------------------------------------------------------------ counter summary
def _read_run(d):
    """One rocprofv3 --pmc run of this script: (bench JSON line, csv rows)."""
    with open(os.path.join(d, "bench.out")) as f:
        line = [ln for ln in f if ln.startswith("{")][-1]
    js = json.loads(line)
    rows = []
    for name in sorted(os.listdir(d)):
        if name.endswith("counter_collection.csv"):
            with open(os.path.join(d, name)) as f:
                rows += list(csv.DictReader(f))
    rows.sort(key=lambda r: int(r["Dispatch_Id"]))
    return js, rows


def summarize_counters(dirs):
    """Per-attempt FETCH / WRITE bytes and VALU lane-instructions of each
    lattice kernel from counter runs (bench.py --steps 0 --warmup 0 ...
    under rocprofv3 --pmc, one or several counters per run), calibrated by
    the plain device copy each run ends with."""
    modes, calib, cmds, hashes = {}, {}, [], set()
    for d in dirs:
        js, rows = _read_run(d)
        hashes.add(js["kernel_source_hash"])
        cfg = js["config"]
        mode = cfg["schedule_name"]
        sw = cfg["profiled_sweeps"]
        n_copy = cfg["copy_calibration_bytes"]
        counters = sorted({r["Counter_Name"] for r in rows})
        cmds.append(f"rocprofv3 --pmc {' '.join(counters)} --output-format csv -d <dir> -o pmc "
                    f"-- python3 bench.py {' '.join(js['argv'])}")
        for counter in counters:
            _summarize_counter(js, cfg, [r for r in rows if r["Counter_Name"] == counter],
                               counter, mode, sw, n_copy, calib, modes)
    if len(hashes) != 1:
        raise SystemExit(f"counter runs were taken on different kernel sources: {hashes}")
    # derived: VALU issue cycles per instruction and the 64-bit share
    for m in modes.values():
        for e in m.values():
            if e.get("valu_active_cycles_per_attempt") and e.get("valu_lane_instr_per_attempt"):
                e["valu_cycles_per_instr"] = round(
                    e["valu_active_cycles_per_attempt"] / (e["valu_lane_instr_per_attempt"] / 64.0), 3)
            if e.get("valu_int64_lane_instr_per_attempt") and e.get("valu_lane_instr_per_attempt"):
                e["valu_int64_share"] = round(
                    e["valu_int64_lane_instr_per_attempt"] / e["valu_lane_instr_per_attempt"], 4)
    out = {"kernel_source_hash": hashes.pop(), "copy_calibration": calib,
           "commands": cmds, "modes": modes}
    with open(COUNTERS, "w") as f:
        json.dump(out, f, indent=1)
    print(json.dumps(out, indent=1))


def _summarize_counter(js, cfg, rows, counter, mode, sw, n_copy, calib, modes):
    """Per-attempt figures of one counter of one run (rows in dispatch
    order) into modes[mode][kernel]."""
    copies = [float(r["Counter_Value"]) for r in rows if "copyBuffer" in r["Kernel_Name"]]
    scale = 1.0
    if counter in ("FETCH_SIZE", "WRITE_SIZE"):
        # counter reads KiB; the copy moves n_copy bytes each way
        scale = n_copy / (max(copies) * 1024.0)
        calib[counter] = round(scale, 4)
    st, re_ = cfg["streamed_sites_by_model"], cfg["resident_sites_by_model"]
    per_disp = {"k_stream_pass_ising": st["ising"] // 2, "k_stream_pass_potts": st["potts"] // 2}
    res_total = (re_["ising"] + re_["potts"]) * sw
    # persistent kernels: the profiled sweeps' launches come last
    kern = js.get("kernels") or js.get("ising_probe", {}).get("kernels") or {}
    n_pers = {"k_persist_ising": (kern.get("persist_ising") or {}).get("launches", 0),
              "k_persist_potts": (kern.get("persist_potts") or {}).get("launches", 0)}
    pers_total = {"k_persist_ising": st["ising"] * sw, "k_persist_potts": st["potts"] * sw}
    m = modes.setdefault(mode, {})
    for kname in ("k_stream_pass_ising", "k_stream_pass_potts", "k_persist_ising",
                  "k_persist_potts", "k_resident"):
        vals = [float(r["Counter_Value"]) for r in rows if kname in r["Kernel_Name"]]
        if not vals:
            continue
        if kname == "k_resident":
            att, v = res_total, sum(vals)
        elif kname in n_pers:
            if not n_pers[kname]:
                continue
            vals = vals[-n_pers[kname]:]
            # per dispatch: the mean over the profiled launches
            att, v = pers_total[kname] // len(vals), sum(vals) / len(vals)
        else:
            # the profiled sweeps come last: 2 launches per sweep
            vals = vals[-2 * sw:]
            att, v = per_disp[kname], statistics.median(vals)
        if att <= 0:
            continue
        e = m.setdefault(kname, {"dispatches": len(vals)})
        e["attempts_per_dispatch" if kname != "k_resident" else "attempts_total"] = att
        if counter == "FETCH_SIZE":
            e["fetch_bytes_per_attempt"] = round(v * 1024.0 * scale / att, 4)
        elif counter == "WRITE_SIZE":
            e["write_bytes_per_attempt"] = round(v * 1024.0 * scale / att, 4)
        elif counter == "SQ_INSTS_VALU":
            e["valu_lane_instr_per_attempt"] = round(v * 64.0 / att, 3)
        elif counter == "SQ_INSTS_VALU_INT64":
            e["valu_int64_lane_instr_per_attempt"] = round(v * 64.0 / att, 3)
        elif counter == "SQ_ACTIVE_INST_VALU":
            # cycles waves spend issuing VALU instructions, per attempt
            e["valu_active_cycles_per_attempt"] = round(v / att, 4)
        elif counter == "VALUBusy":
            e["valu_busy_pct"] = round(statistics.median(vals), 1)


def copy_calibration(torch, mib):
    """One plain device copy of mib MiB (the reference dispatch that scales
    rocprofv3 FETCH_SIZE / WRITE_SIZE); returns its size in bytes."""
    if mib <= 0:
        return 0
    n = mib << 20
    src = torch.ones(n, dtype=torch.uint8, device="cuda")
    dst = torch.empty_like(src)
    dst.copy_(src)
    torch.cuda.synchronize()
    del src, dst
    return n


PATH_PROBES = {
    "cpm": lambda S, torch: cpm_probe(S, torch, 50),
    "cpm_paper": lambda S, torch: cpm_paper_probe(S, torch),
    "grad": lambda S, torch: grad_probe(S, torch),
    "tri": lambda S, torch: tri_probe(S, torch),
    "hc": lambda S, torch: hc_probe(S, torch),
    # the streamed passes with more spins than the 256 MB last-level cache
    # holds (302 and 268 MB)
    "tri_large": lambda S, torch: tri_probe(S, torch, n_rep=8192, L=192, sweeps=50),
    "hc_large": lambda S, torch: hc_probe(S, torch, n_rep=8192, sweeps=50),
    "msc": lambda S, torch: msc_probe(S, torch),
    "mlp": lambda S, torch: mlp_probe(torch),
    "dmc": lambda S, torch: dmc_probe(torch),
    "dmc_vs_covariance": lambda S, torch: dmc_vs_covariance_probe(torch),
    "spinopt": lambda S, torch: spinopt_probe(torch),
    "surrogate": lambda S, torch: surrogate_probe(torch),
}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=2)
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--sweeps", type=int, default=10000, help="sweeps per step")
    ap.add_argument("--mode", default="tuned",
                    choices=["tuned", "auto", "resident", "stream", "hybrid"],
                    help="schedule; 'tuned' runs the library's autotuner first")
    ap.add_argument("--tune-sweeps", type=int, default=100,
                    help="sweeps per autotuner trial (trials of 20 sweeps misjudged the hybrid "
                         "schedule's long-run rate)")
    ap.add_argument("--prof-sweeps", type=int, default=200,
                    help="sweeps of the per-kernel timing run after the timed steps")
    ap.add_argument("--tile-rows", type=int, default=0)
    ap.add_argument("--threads", type=int, default=0)
    ap.add_argument("--nt", choices=["auto", "on", "off"], default="auto",
                    help="nontemporal own-plane access of the streamed passes")
    ap.add_argument("--rpb", type=int, default=0, help="replicas per resident workgroup")
    ap.add_argument("--persistent", action="store_true",
                    help="persistent streamed passes (one launch per chunk)")
    ap.add_argument("--cpu-sweeps", type=int, default=30)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-probes", action="store_true",
                    help="skip the Ising streaming probes (for counter collection runs)")
    ap.add_argument("--no-paths", action="store_true",
                    help="skip the CPM, covariance-backward, MLP and differentiable-MC "
                         "measurements")
    ap.add_argument("--no-surrogate", action="store_true",
                    help="skip the surrogate-vs-Monte-Carlo inverse problem")
    ap.add_argument("--copy-calibration-mib", type=int, default=0,
                    help="also run one plain device copy of this many MiB (the reference "
                         "dispatch that scales rocprofv3 FETCH_SIZE / WRITE_SIZE)")
    ap.add_argument("--ising-probe", type=int, default=0, metavar="N",
                    help="run only the streamed Ising probe with N replicas of 256x256 "
                         "(--prof-sweeps sweeps; for counter collection)")
    ap.add_argument("--path", choices=sorted(PATH_PROBES), default=None,
                    help="run only this measurement of the other paths and print it "
                         "(for profiling runs)")
    ap.add_argument("--summarize-counters", nargs="+", metavar="DIR",
                    help="write the counter summary from rocprofv3 --pmc runs of this script "
                         "(each DIR holds the run's counter csv and its stdout as bench.out)")
    args = ap.parse_args()
    if args.summarize_counters:
        summarize_counters(args.summarize_counters)
        return
    if args.gpus != 1:
        print(json.dumps({"error": "this benchmark runs on one GPU only: the workload is "
                                   "independent replicas, which shard by replica across GPUs "
                                   "with no communication; --gpus must be 1"}))
        sys.exit(2)

    import torch
    import synth
    from paper_2304_01772_amd.sampler import Sampler, MODES

    if args.path:
        res = PATH_PROBES[args.path](Sampler, torch)
        print(json.dumps({"path": args.path, "result": res, "argv": sys.argv[1:],
                          "kernel_source_hash": kernel_source_hash()}), flush=True)
        return

    if args.ising_probe:
        # the streamed Ising probe alone (counter collection for its roofline)
        sched = None
        if args.tile_rows or args.threads or args.nt != "auto" or args.persistent:
            sched = dict(tile_rows=args.tile_rows, wg_threads=args.threads,
                         nt={"auto": None, "on": True, "off": False}[args.nt],
                         persistent=args.persistent)
        res, cfg = ising_stream_probe(Sampler, torch, args.ising_probe, args.prof_sweeps, sched)
        n_copy = copy_calibration(torch, args.copy_calibration_mib)
        cfg.update(schedule_name=f"ising_probe_{args.ising_probe}",
                   profiled_sweeps=args.prof_sweeps, copy_calibration_bytes=n_copy)
        print(json.dumps({"ising_probe": res, "config": cfg, "argv": sys.argv[1:],
                          "kernel_source_hash": kernel_source_hash()}), flush=True)
        return

    reps = synth.batched_ising_potts()
    seed = 2
    sites = sum(r["Lx"] * r["Ly"] for r in reps)
    print(f"# workload: {len(reps)} replicas, {sites} sites/sweep, {args.sweeps} sweeps/step",
          file=sys.stderr, flush=True)
    smp = Sampler(reps, seed=seed, init=True)
    tuning = None
    if args.mode == "tuned":
        chosen, rates = smp.autotune(trial_sweeps=args.tune_sweeps)
        tuning = dict(chosen=chosen, candidate_rates=[round(r, 1) for r in rates])
        print(f"# autotune: {tuning}", file=sys.stderr, flush=True)
    else:
        smp.set_schedule(mode=args.mode, tile_rows=args.tile_rows, wg_threads=args.threads,
                         nt={"auto": None, "on": True, "off": False}[args.nt], rpb=args.rpb,
                         persistent=args.persistent)
    sched = smp.get_schedule()
    mode_name = {v: k for k, v in MODES.items()}[sched["mode"]]
    if mode_name == "auto":  # what it resolves to
        mode_name = "hybrid" if smp.schedule_sites()[0] else "resident"
    for w in range(args.warmup):
        smp.sweep(args.sweeps)
        torch.cuda.synchronize()
        print(f"# warmup step {w + 1}/{args.warmup} done", file=sys.stderr, flush=True)
    torch.cuda.synchronize()

    # timed steps: the production path (cached hipGraph replays)
    ms, value = None, None
    if args.steps > 0:
        e0 = torch.cuda.Event(enable_timing=True)
        e1 = torch.cuda.Event(enable_timing=True)
        e0.record(smp.stream)
        for k in range(args.steps):
            smp.sweep(args.sweeps)
        e1.record(smp.stream)
        torch.cuda.synchronize()
        ms = e0.elapsed_time(e1)
        print(f"# timed {args.steps} steps: {ms:.1f} ms", file=sys.stderr, flush=True)
        value = sites * args.sweeps * args.steps / (ms * 1e6)

    # per-kernel timing of the same workload right after the timed steps
    st_m, re_m = smp.schedule_sites(by_model=True)
    kern = profiled_kernels(smp, torch, args.prof_sweeps)
    print(f"# kernels over {args.prof_sweeps} profiled sweeps: {kern}", file=sys.stderr,
          flush=True)
    roof = None
    if kern:
        dom = max(kern, key=lambda k: kern[k]["ms"])
        roof = roofline(dom, kern[dom], mode_name)
        roof["units"] = f"{mode_name} schedule of the workload, {args.prof_sweeps} sweeps"
        if ms is not None:
            # the whole timed sweep against the VALU issue peak: VALU lane-
            # instructions per sweep from the counters of every kernel kind
            per = {"k_stream_pass_ising": st_m["ising"], "k_stream_pass_potts": st_m["potts"],
                   "k_persist_ising": st_m["ising"], "k_persist_potts": st_m["potts"],
                   "k_resident": re_m["ising"] + re_m["potts"]}
            ran = {KERNEL_NAMES[k] for k in kern}
            lanes, ok = 0.0, True
            for kname in ran:
                ce = counter_entry(mode_name, kname)
                if not ce or not ce.get("valu_lane_instr_per_attempt"):
                    ok = False
                    break
                lanes += ce["valu_lane_instr_per_attempt"] * per[kname]
            if ok and lanes > 0:
                sweep_s = ms * 1e-3 / (args.steps * args.sweeps)
                roof["sweep_alu"] = {
                    "lane_instr_per_sweep": round(lanes),
                    "achieved": round(lanes / sweep_s / 1e12, 2), "peak": round(VALU_PEAK / 1e12, 2),
                    "unit": "T lane-instr/s", "frac": round(lanes / sweep_s / VALU_PEAK, 4)}
    smp.close()

    n_copy = copy_calibration(torch, args.copy_calibration_mib)

    probes = {}
    for n_rep in (() if args.no_probes else (1024, 8192)):
        probes[f"ising_{n_rep}x256x256_stream"], _ = ising_stream_probe(Sampler, torch, n_rep, 100)
        print(f"# Ising stream probe {n_rep}: {probes[f'ising_{n_rep}x256x256_stream']}",
              file=sys.stderr, flush=True)

    paths = None
    if not args.no_paths:
        paths = {}
        paths["cpm_cell_sorting"] = cpm_probe(Sampler, torch, 50)
        print(f"# cpm: {paths['cpm_cell_sorting']}", file=sys.stderr, flush=True)
        paths["cpm_paper_setting"] = cpm_paper_probe(Sampler, torch)
        print(f"# cpm paper setting: {paths['cpm_paper_setting']}", file=sys.stderr, flush=True)
        paths["triangular_ising"] = tri_probe(Sampler, torch)
        print(f"# triangular: {paths['triangular_ising']}", file=sys.stderr, flush=True)
        paths["cubic_ising"] = hc_probe(Sampler, torch)
        print(f"# cubic: {paths['cubic_ising']}", file=sys.stderr, flush=True)
        paths["multispin_ising"] = msc_probe(Sampler, torch)
        print(f"# multispin: {paths['multispin_ising']}", file=sys.stderr, flush=True)
        paths["covariance_backward"] = grad_probe(Sampler, torch)
        print(f"# grad: {paths['covariance_backward']}", file=sys.stderr, flush=True)
        paths["surrogate_mlp"] = mlp_probe(torch)
        print(f"# mlp: {paths['surrogate_mlp']}", file=sys.stderr, flush=True)
        paths["differentiable_mc"] = dmc_probe(torch)
        print(f"# dmc: {paths['differentiable_mc']}", file=sys.stderr, flush=True)
        paths["dmc_vs_covariance"] = dmc_vs_covariance_probe(torch)
        print(f"# dmc vs covariance: {paths['dmc_vs_covariance']}", file=sys.stderr, flush=True)
        paths["spin_value_optimisation"] = spinopt_probe(torch)
        print(f"# spinopt: {paths['spin_value_optimisation']}", file=sys.stderr, flush=True)
    surrogate = None
    if not args.no_surrogate:
        surrogate = surrogate_probe(torch)
        print(f"# surrogate vs Monte Carlo: {surrogate}", file=sys.stderr, flush=True)

    cpu = None
    if not args.no_cpu_baseline:
        print("# cpu baseline (oracle on host cores)...", file=sys.stderr, flush=True)
        cpu = cpu_baseline(reps, seed, args.cpu_sweeps)

    out = {
        "metric": "spin-update attempts/ns",
        "value": round(value, 2) if value is not None else None,
        "unit": "attempts/ns",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(ms / args.steps, 2) if ms is not None else None,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "u8",
        "data": "synthetic",
        "config": {
            "workload": "1024 Ising 256x256 (beta grid 0.30-0.60) + 512 Potts L in "
                        "{64..1024}, q in {3,4,6,8}, beta in [0.9,1.1] ln(1+sqrt q); "
                        f"{args.sweeps} checkerboard sweeps per step",
            "replicas": len(reps),
            "sites_per_sweep": sites,
            "sweeps_per_step": args.sweeps,
            "schedule": sched,
            "schedule_name": mode_name,
            "autotune": tuning,
            "streamed_sites_by_model": st_m,
            "resident_sites_by_model": re_m,
            "profiled_sweeps": args.prof_sweeps,
            "copy_calibration_bytes": n_copy,
        },
        "roofline": roof,
        "kernels": kern,
        "ising_stream_roofline": probes,
        "other_paths": paths,
        "surrogate_vs_mc": surrogate,
        "cpu_baseline": cpu,
        "argv": sys.argv[1:],
        "kernel_source_hash": kernel_source_hash(),
    }
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
