"""Throughput of batched r-cell MD (and of the learned stress surrogate) on one MI355X.

Workloads (``--workload``; every run prints one JSON line):

  cu_element  one hex8 element of copper: 8 FCC r-cells x 4000 atoms, Sutton-Chen EAM,
              300 K Langevin, dt = 1 fs, mixed precision.  A step is one finite-element load step:
              the device-resident F of every cell is QR-decomposed and the boxes remapped, 100 MD
              steps run (neighbour builds, two-pass EAM forces fused with the Langevin
              velocity-Verlet update, per-cell stress reduction), and the window-averaged stress is
              rotated to the FE frame into device memory.
  cu_batched  the same copper element batched 32 times (256 cells, 1.02 M atoms): the EAM kernels
              with the GPU full.
  kg_single   one Kremer-Grest cell of 20 x 50 beads in FP64; F ramped to a 20 % uniaxial
              isochoric stretch over 1000 MD steps (a new F before every step), stress read every
              100 steps.  A step is one MD step; latency bound.
  kg_batched  512 Kremer-Grest cells of 2k-20k beads (chains of 50-200), each under its own
              rotation x symmetric stretch; mixed precision; a step is 100 MD steps of the whole
              batch followed by the stress read.
  kg_glassy   100 glassy Kremer-Grest cells of 100 x 100 beads (10^6 beads, the size of the paper's
              production run) with the LJ attraction to 2.5 sigma at T = 0.1.
  fe_bar      (default) the explicit hex8 bar (8 x 2 x 2 elements, 2 x 2 x 2 Gauss points = 256 r-cells of
              400 x 100 beads, ~10.2 M beads) under uniaxial tension; a step is one FE load step
              (host FE update, F to the cells, 500 MD steps, stress back).
  fe_tet      the paper's polymer specimen (Sec. 3.2): a cube of 100 C3D4 tetrahedra with one
              quadrature point each = 100 r-cells of 100 x 100 beads (10^6 beads), uniaxial tension;
              a step is one FE load step with 500 MD steps.
  fe_scaling  the system of the paper's scaling test on one GPU: 1000 C3D4 tetrahedra = 1000 r-cells
              of 100 x 100 beads (10^7 beads); a step is one FE load step with 100 MD steps.
  glassy_rates  direct MD of glassy cells at the constant strain rates 0.01, 0.015, 0.02 / tau of
              the paper's direct-MD comparison (a new F before every MD step), beside the r-cell's
              load-step protocol at the same mean rates; a step is one MD step.
  surrogate   the stress surrogate network (153 -> 4 x 256 -> 6, ensemble of 5, BF16 matrix cores
              with FP32 accumulation): ensemble evaluations per second at the bar's batch (256
              Gauss points) and at a large batch, and training samples per second.

Inputs are resident in HBM before the timed region; timings bracket K steps with device
synchronisation.  The roofline object describes the dominant kernel, timed in a separate pass with
the start and stop events of its own dispatches on the library's stream, and, after the timed
region, the copy bandwidth and FP32 FMA rate this GPU delivers (measured_peaks).  The CPU baseline
is the FP64 oracle on a bounded sample of the same workload (about ORACLE_SECONDS of CPU time), on
this host's cores.

  python bench.py [--workload W] [--gpus 1] [--steps K] [--warmup W] [--no-cpu-baseline]
"""
import argparse
import hashlib
import json
import math
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

PEAK_FP32 = 157.3e12          # MI355X FP32 vector, FLOP/s (published)
PEAK_HBM = 8.0e12             # MI355X HBM3E, bytes/s (published)
PEAK_BF16 = 2.5e15            # MI355X dense BF16 matrix, FLOP/s (published)
# Sutton-Chen: algorithmic FLOPs per unique pair inside the cutoff of an MD step that does not
# report the energy (FMA = 2, every other arithmetic op 1), for a half-list evaluation from Cartesian
# coordinates.  Force pass: separation d = x_j - x_i 3, r^2 5, 1/r 1, powers r^-2, r^-3, r^-6 3,
# pair scalar g/r = -r^-2 r^-6 (eps n a^9 r^-3 + F'_i + F'_j) 5, t = (g/r) d 3, f_i += t and
# f_j -= t 6, virial W += t (x) d 12: 38.  Density pass: separation 3, r^2 5, 1/r 1, r^-3 2,
# r^-6 1, (a/r)^m 1, shift 1, both densities 2: 16.
FLOP_FORCE_PER_PAIR = 38
FLOP_DENSITY_PER_PAIR = 16
PAIRS_PER_ATOM = 67           # unique neighbours within 1.95 a in FCC copper
# Kremer-Grest: the least HBM traffic an MD step needs per bead: x and v in FP64, read and
# written (96 B), plus the two chain partners as 32-bit indices (8 B)
BYTES_PER_BEAD_STEP = 104

ORACLE_SECONDS = 10.0     # CPU time the oracle baseline runs for (bounded sample of the workload)
DEFAULTS = {"cu_element": (50, 3), "cu_batched": (10, 2), "kg_single": (1000, 100), "kg_batched": (10, 1),
            "kg_glassy": (10, 1),
            "fe_bar": (10, 2), "fe_tet": (4, 1), "fe_scaling": (3, 1), "glassy_rates": (4000, 100),
            "surrogate": (200, 20), "fe_bar_surrogate": (1, 0)}


def kernel_source_hash():
    h = hashlib.sha256()
    for f in ("md_device.h", "rcell_md.hip"):
        with open(os.path.join(ROOT, "paper_1902_09171_amd", "csrc", f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


def traffic_from_profiles(kernel, workload):
    """HBM bytes per launch from the committed rocprofv3 PMC summary, if it matches the source."""
    path = os.path.join(ROOT, "profiles", f"traffic_{kernel}_{workload}.json")
    if not os.path.exists(path):
        return None
    with open(path) as fh:
        rec = json.load(fh)
    if rec.get("source_hash") != kernel_source_hash():
        return None
    return rec.get("bytes_per_launch")


def fro(s):
    import numpy as np
    s = np.asarray(s)
    return np.sqrt((s[..., :3] ** 2).sum(-1) + 2 * (s[..., 3:] ** 2).sum(-1))


def log(msg):
    print(f"[bench] {msg}", file=sys.stderr, flush=True)


# ------------------------------------------------------------------ MD helpers
def oracle_sample(params, cells, F, nsteps, label, seconds=None):
    """The FP64 oracle on the host cores: MD steps of the given cells after set_deformation(F).  The
    stress window of the first nsteps is returned for the comparison with the GPU; the oracle then
    runs on until about `seconds` of CPU time (ORACLE_SECONDS) have been spent, and the rate is taken
    over every step.  Returns (cpu_baseline dict, oracle stress after nsteps)."""
    from oracle import core
    seconds = ORACLE_SECONDS if seconds is None else seconds
    threads = core.threads(min(len(cells), host_threads()))
    ob = core.OracleBatch(params, cells)
    ob.set_deformation(F)
    ob.get_stress()
    t0 = time.perf_counter()
    ob.run(nsteps)
    dt = time.perf_counter() - t0
    s_ora = ob.get_stress()
    extra = min(100 * nsteps, max(0, math.ceil((seconds - dt) / (dt / nsteps))))
    if extra:
        t1 = time.perf_counter()
        ob.run(extra)
        dt += time.perf_counter() - t1
    natoms = sum(len(c["x"]) for c in cells)
    total = nsteps + extra
    value = natoms * total / dt
    # the same sample on one core, for a bounded third of the time (the all-core rate is `value`)
    single = value
    if threads > 1:
        core.threads(1)
        n1, t2 = 0, time.perf_counter()
        while n1 == 0 or time.perf_counter() - t2 < seconds / 3:
            ob.run(max(1, nsteps // 4))
            n1 += max(1, nsteps // 4)
        single = natoms * n1 / (time.perf_counter() - t2)
        core.threads(threads)
    return dict(value=value, unit="atom-steps/s", cores=threads, kind="oracle",
                sample=f"{len(cells)} cells, {natoms} atoms, {total} MD steps in {dt:.1f} s ({label}; "
                       f"stress compared with the GPU after the first {nsteps})",
                single_core_value=single, host_threads=host_threads(), cpu_model=cpu_model()), s_ora


def host_threads():
    """Hardware threads this process may use: the CPU affinity mask, capped by OMP_NUM_THREADS."""
    try:
        n = len(os.sched_getaffinity(0))
    except AttributeError:
        n = os.cpu_count() or 1
    omp = os.environ.get("OMP_NUM_THREADS", "")
    if omp.isdigit() and int(omp) > 0:
        n = min(n, int(omp))
    return max(1, n)


def cpu_model():
    try:
        with open("/proc/cpuinfo") as fh:
            for line in fh:
                if line.startswith("model name"):
                    return line.split(":", 1)[1].strip()
    except OSError:
        pass
    import platform
    return platform.processor() or "unknown"


def gpu_sample_error(rcell, params, cells, F, nsteps, s_ora, lanes, bin_factor=1):
    """The same sample on the GPU from the same initial state: max relative stress deviation."""
    import numpy as np
    g = rcell.RCellBatch(params, cells)
    g.set_lanes(lanes)
    g.set_bin_factor(bin_factor)
    g.set_deformation(F)
    g.get_stress()
    g.run(nsteps)
    s_gpu = g.get_stress()
    g.close()
    return float((np.abs(s_gpu - s_ora).max(1) / fro(s_ora)).max())


def kernel_avg(g, slot, run_again):
    """Average HIP-event duration (s) of the force kernel (slot 0) or density pass (slot 1)
    over a separate pass of run_again(), so that the events do not perturb the timed region."""
    g.prof_enable(True)
    g.prof_read(0); g.prof_read(1)
    run_again()
    ms, n = g.prof_read(slot)
    ms1, n1 = g.prof_read(1 - slot)
    g.prof_enable(False)
    return (ms / 1e3 / max(n, 1), n), (ms1 / 1e3 / max(n1, 1), n1)


def tune(g, args):
    """The batch engine's knobs: rcell_autotune (bin factor, then lanes per atom) unless --lanes
    fixes the lanes; returns (lanes, bin_factor)."""
    if args.lanes == 0:
        return g.autotune(use_cache=True)
    g.set_lanes(args.lanes)
    return g.lanes(), g.bin_factor()


def md_line(args, workload, value, elapsed, natoms, config, roofline, extra=None, dtype=None):
    out = {"metric": "atom-steps/s batched r-cell MD", "value": value, "unit": "atom-steps/s",
           "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
           "ms_per_step": elapsed / args.steps * 1e3, "higher_is_better": True, "scaling": "weak",
           "vs_baseline": None, "dtype": dtype or "f32 pair forces, f64 positions/integration/stress",
           "data": "synthetic", "config": dict(workload=workload, **config), "roofline": roofline}
    if extra:
        out.update(extra)
    return out


def check_status(g):
    import numpy as np
    st = g.status()
    if np.any(st != 0):
        raise SystemExit(f"cell status errors during the bench: {st.tolist()}")


# ------------------------------------------------------------------ workloads
def bench_cu_element(args, torch, rcell, configs, ncells=8):
    import numpy as np
    MD_PER_LOAD = 100
    cfg = configs.cu_element(ncells=ncells)
    ncells = len(cfg["cells"])
    natoms = sum(len(c["x"]) for c in cfg["cells"])
    dev = torch.device("cuda:0")
    stream = torch.cuda.current_stream(dev)
    g = rcell.RCellBatch(cfg["params"], cfg["cells"], stream=stream.cuda_stream)
    nload = len(cfg["F_path"])
    F_dev = torch.tensor(np.ascontiguousarray(cfg["F_path"]), dtype=torch.float64, device=dev)
    sig_dev = torch.zeros((ncells, 6), dtype=torch.float64, device=dev)
    P_dev = torch.zeros((ncells, 9), dtype=torch.float64, device=dev)
    g.set_deformation_dev(F_dev[0].data_ptr())
    lanes, binf = tune(g, args)

    def load_step(k):
        g.set_deformation_dev(F_dev[k % nload].data_ptr())
        g.run(MD_PER_LOAD)
        g.get_stress_dev(sig_dev.data_ptr(), P_dev.data_ptr())

    for k in range(args.warmup):
        load_step(k)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for k in range(args.steps):
        load_step(args.warmup + k)
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    nprof = min(args.steps, 10)
    (avg_s, force_n), (rho_s, _) = kernel_avg(
        g, 0, lambda: [load_step(args.warmup + args.steps + k) for k in range(nprof)])
    check_status(g)
    value = natoms * MD_PER_LOAD * args.steps / elapsed
    flop_launch = FLOP_FORCE_PER_PAIR * PAIRS_PER_ATOM * natoms
    achieved = flop_launch / avg_s
    name = "cu_element" if ncells == 8 else "cu_batched"
    roofline = {"bound": "alu", "achieved": achieved / 1e12, "peak": PEAK_FP32 / 1e12, "unit": "TFLOP/s",
                "frac": achieved / PEAK_FP32, "traffic": traffic_from_profiles("k_force_eam", name),
                "kernel": "k_force_eam", "avg_us": avg_s * 1e6, "launches": force_n,
                "density_pass_avg_us": rho_s * 1e6, "flop_per_launch": flop_launch}
    what = ("8 FCC copper r-cells x 4000 atoms (one hex8 element, 2x2x2 Gauss points)" if ncells == 8 else
            f"{ncells} FCC copper r-cells x 4000 atoms (the copper element batched {ncells // 8} times)")
    out = md_line(args, name, value, elapsed, natoms,
                  {"description": what + ", Sutton-Chen EAM, 300 K, dt 1 fs, rotated uniaxial F ramp to 5 %, "
                                         "100 MD steps per load step",
                   "cells": ncells, "atoms": natoms, "md_steps_per_step": MD_PER_LOAD,
                   "lanes_per_atom": lanes, "bin_factor": binf}, roofline)
    if not args.no_cpu_baseline:
        sub = list(range(min(ncells, max(8, host_threads()))))
        cells8, F8 = [cfg["cells"][c] for c in sub], cfg["F_path"][0][sub]
        cb, s_ora = oracle_sample(cfg["params"], cells8, F8, args.cpu_sample_steps,
                                  f"first load step of the first {len(sub)} cells")
        out["cpu_baseline"] = cb
        out["stress_rel_err_vs_oracle"] = gpu_sample_error(rcell, cfg["params"], cells8, F8,
                                                           args.cpu_sample_steps, s_ora, lanes, binf)
    return out


def bench_cu_batched(args, torch, rcell, configs):
    return bench_cu_element(args, torch, rcell, configs, ncells=256)


def bench_kg_single(args, torch, rcell, configs):
    import numpy as np
    cfg = configs.kg_single()
    natoms = len(cfg["cells"][0]["x"])
    dev = torch.device("cuda:0")
    stream = torch.cuda.current_stream(dev)
    g = rcell.RCellBatch(cfg["params"], cfg["cells"], stream=stream.cuda_stream)
    F_dev = torch.tensor(np.ascontiguousarray(cfg["F_path"]), dtype=torch.float64, device=dev)
    sig_dev = torch.zeros((1, 6), dtype=torch.float64, device=dev)
    nF = len(cfg["F_path"])
    lanes, binf = tune(g, args)

    def md_step(k):                                   # F of step k, one MD step, stress every 100
        g.set_deformation_dev(F_dev[k % nF].data_ptr())
        g.run(1)
        if (k + 1) % 100 == 0:
            g.get_stress_dev(sig_dev.data_ptr(), None)

    for k in range(args.warmup):
        md_step(k)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for k in range(args.steps):
        md_step(k)
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    # plain MD of the same cell (no deformation between steps), graph-captured blocks
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    g.run(1000)
    torch.cuda.synchronize()
    plain_us = (time.perf_counter() - t1) / 1000 * 1e6
    (avg_s, n), _ = kernel_avg(g, 0, lambda: g.run(100))
    check_status(g)
    achieved = BYTES_PER_BEAD_STEP * natoms / avg_s
    roofline = {"bound": "hbm", "achieved": achieved / 1e9, "peak": PEAK_HBM / 1e9, "unit": "GB/s",
                "frac": achieved / PEAK_HBM, "traffic": None, "kernel": "k_force_kg", "avg_us": avg_s * 1e6,
                "launches": n, "note": "1000 beads cannot fill 256 CUs: latency bound"}
    out = md_line(args, "kg_single", natoms * args.steps / elapsed, elapsed, natoms,
                  {"description": "one Kremer-Grest cell, 20 chains x 50 beads, FP64, F ramped to a 20 % "
                                  "uniaxial isochoric stretch over 1000 MD steps (new F before every step), "
                                  "stress every 100 steps", "cells": 1, "atoms": natoms,
                   "md_steps_per_step": 1, "lanes_per_atom": lanes, "bin_factor": binf}, roofline,
                  extra={"us_per_md_step_with_new_F": elapsed / args.steps * 1e6,
                         "us_per_md_step_plain_run": plain_us}, dtype="f64")
    if not args.no_cpu_baseline:
        cb, s_ora = oracle_sample(cfg["params"], cfg["cells"], cfg["F_path"][0], 1000,
                                  "the cell at the first F of the ramp")
        out["cpu_baseline"] = cb
        out["stress_rel_err_vs_oracle"] = gpu_sample_error(rcell, cfg["params"], cfg["cells"], cfg["F_path"][0],
                                                           1000, s_ora, lanes, binf)
    return out


def make_cells(fn, arg_list):
    """Generate the KG melts in this process (host-side input preparation, untimed; the melt
    relaxation is itself multithreaded), with a progress line every 32 cells."""
    out = []
    for k, a in enumerate(arg_list):
        out.append(fn(a))
        if (k + 1) % 32 == 0 or k + 1 == len(arg_list):
            log(f"  {k + 1}/{len(arg_list)} cells")
    return out


def _kg_batched_cell(c):
    from synth import configs
    out = configs.kg_batched(cells_subset=[c])
    return out["cells"][0], out["F"][0]


def _fe_bar_cell(c):
    from synth import configs
    return configs.fe_bar_cells(cells_subset=[c])["cells"][0]


def _fe_tet_cell(c):
    from synth import configs
    return configs.fe_tet_cells(cells_subset=[c])["cells"][0]


def _fe_scaling_cell(c):
    from synth import configs
    return configs.fe_tet_cells(cells_subset=[c], stream=8)["cells"][0]


def _kg_glassy_cell(c):
    from synth import configs
    out = configs.kg_glassy(cells_subset=[c])
    return out["cells"][0], out["F"][0]


def bench_kg_batched(args, torch, rcell, configs, glassy=False):
    import numpy as np
    MD_PER_STEP = 100
    ncells = 100 if glassy else 512
    log(f"generating {ncells} Kremer-Grest cells")
    res = make_cells(_kg_glassy_cell if glassy else _kg_batched_cell, list(range(ncells)))
    cells = [r[0] for r in res]
    F = np.stack([r[1] for r in res])
    params = (configs.kg_glassy_params(precision="mixed") if glassy else
              configs.kg_params(precision="mixed", skin=0.55))      # the fastest skin of a sweep
    natoms = sum(len(c["x"]) for c in cells)
    dev = torch.device("cuda:0")
    stream = torch.cuda.current_stream(dev)
    log(f"creating the batch: {natoms} beads")
    g = rcell.RCellBatch(params, cells, stream=stream.cuda_stream)
    g.set_deformation(F)
    lanes, binf = tune(g, args)
    sig_dev = torch.zeros((ncells, 6), dtype=torch.float64, device=dev)

    def step():
        g.run(MD_PER_STEP)
        g.get_stress_dev(sig_dev.data_ptr(), None)

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for k in range(args.steps):
        step()
        if k % 5 == 4:
            torch.cuda.synchronize()
            log(f"step {k + 1}/{args.steps}")
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    (avg_s, n), _ = kernel_avg(g, 0, lambda: g.run(100))
    check_status(g)
    achieved = BYTES_PER_BEAD_STEP * natoms / avg_s
    name = "kg_glassy" if glassy else "kg_batched"
    roofline = {"bound": "hbm", "achieved": achieved / 1e9, "peak": PEAK_HBM / 1e9, "unit": "GB/s",
                "frac": achieved / PEAK_HBM, "traffic": traffic_from_profiles("k_force_kg", name),
                "kernel": "k_force_kg", "avg_us": avg_s * 1e6, "launches": n,
                "bytes_per_launch": BYTES_PER_BEAD_STEP * natoms}
    what = ("100 glassy Kremer-Grest cells of 100 chains x 100 beads (LJ cut and shifted at 2.5 sigma, "
            "T = 0.1), each under a small isochoric uniaxial stretch, dt 0.005" if glassy else
            "512 Kremer-Grest cells of 2k-20k beads (chains 50-200, density 0.85), each under its own "
            "rotation x symmetric stretch (eigenvalues 0.9-1.1), Langevin T = 1, dt 0.005")
    out = md_line(args, name, natoms * MD_PER_STEP * args.steps / elapsed, elapsed, natoms,
                  {"description": what + "; 100 MD steps per step",
                   "cells": ncells, "atoms": natoms, "md_steps_per_step": MD_PER_STEP,
                   "lanes_per_atom": lanes, "bin_factor": binf, "skin": params["skin"], "rebuilds": g.rebuilds()}, roofline)
    if not args.no_cpu_baseline:
        sub = list(range(min(ncells, max(16, host_threads()))))
        cb, s_ora = oracle_sample(params, [cells[c] for c in sub], F[sub], 20,
                                  f"the first {len(sub)} cells of the batch")
        out["cpu_baseline"] = cb
        out["stress_rel_err_vs_oracle"] = gpu_sample_error(rcell, params, [cells[c] for c in sub], F[sub], 20,
                                                           s_ora, lanes, binf)
    return out


def bench_kg_glassy(args, torch, rcell, configs):
    return bench_kg_batched(args, torch, rcell, configs, glassy=True)


def bench_glassy_rates(args, torch, rcell, configs):
    """Direct MD under a constant engineering strain rate (a new isochoric uniaxial F before every
    MD step) at the three rates of the paper's direct-MD comparison (Fig. 6a), next to the r-cell
    protocol at the same mean rates (the strain of a 100-step load step applied at once, then the
    window-averaged stress): one glassy cell of 100 x 100 beads per rate, same initial state."""
    import numpy as np
    from synth import uniaxial_isochoric
    RATES, N = (0.01, 0.015, 0.02), 100
    cfg = configs.kg_glassy(ncells=1)
    params, cell0 = cfg["params"], cfg["cells"][0]
    cells = [dict(cell0) for _ in RATES]
    natoms = len(cell0["x"]) * len(RATES)
    dt = params["dt"]
    dev = torch.device("cuda:0")
    stream = torch.cuda.current_stream(dev)
    A = rcell.RCellBatch(params, cells, stream=stream.cuda_stream)      # continuous
    B = rcell.RCellBatch(params, cells, stream=stream.cuda_stream)      # load steps
    lanes, binf = tune(A, args)
    B.set_lanes(lanes)
    B.set_bin_factor(binf)
    nst = args.steps                  # timed MD steps of the direct path, each with its own F
    nld = max(1, nst // N)            # load steps of N MD steps on the r-cell path
    F_cont = np.stack([np.stack([uniaxial_isochoric(r * dt * (t + 1)) for r in RATES]) for t in range(nst)])
    F_load = np.stack([np.stack([uniaxial_isochoric(r * dt * N * (k + 1)) for r in RATES]) for k in range(nld)])
    F_cont_dev = torch.tensor(F_cont, dtype=torch.float64, device=dev)
    F_load_dev = torch.tensor(F_load, dtype=torch.float64, device=dev)
    sig_a = torch.zeros((nst, len(RATES), 6), dtype=torch.float64, device=dev)
    sig_b = torch.zeros((nld, len(RATES), 6), dtype=torch.float64, device=dev)
    for g in (A, B):                                  # untimed equilibration at F = I
        g.run(args.warmup)
        g.get_stress()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for t in range(nst):
        A.set_deformation_dev(F_cont_dev[t].data_ptr())
        A.run(1)
        A.get_stress_dev(sig_a[t].data_ptr(), None)
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    t1 = time.perf_counter()
    for k in range(nld):
        B.set_deformation_dev(F_load_dev[k].data_ptr())
        B.run(N)
        B.get_stress_dev(sig_b[k].data_ptr(), None)
    torch.cuda.synchronize()
    elapsed_b = time.perf_counter() - t1
    (avg_s, n), _ = kernel_avg(A, 0, lambda: A.run(100))
    check_status(A)
    check_status(B)
    sa, sb = sig_a.cpu().numpy(), sig_b.cpu().numpy()
    tens = lambda s: s[..., 0] - 0.5 * (s[..., 1] + s[..., 2])       # uniaxial along x, tension +
    nwin = nst // N                                                     # whole load-step windows
    wa = tens(sa[:nwin * N]).reshape(nwin, N, len(RATES)).mean(1)       # continuous, per load-step window
    wb = tens(sb)
    curves = {}
    for c, r in enumerate(RATES):
        rows = []
        for eps in (0.05, 0.1, 0.15, 0.2):
            k = int(round(eps / (r * dt * N))) - 1
            if 0 <= k < nwin:
                rows.append([round(r * dt * N * (k + 1), 4), float(wa[k, c]), float(wb[k, c])])
        curves[str(r)] = rows
    achieved = BYTES_PER_BEAD_STEP * natoms / avg_s
    roofline = {"bound": "hbm", "achieved": achieved / 1e9, "peak": PEAK_HBM / 1e9, "unit": "GB/s",
                "frac": achieved / PEAK_HBM, "traffic": None, "kernel": "k_force_kg", "avg_us": avg_s * 1e6,
                "launches": n, "note": "a new F before every MD step: bound by the deformation's latency"}
    out = md_line(args, "glassy_rates", natoms * nst / elapsed, elapsed, natoms,
                  {"description": "direct MD at constant engineering strain rates 0.01, 0.015, 0.02 / tau (new "
                                  "isochoric uniaxial F before every MD step), one glassy Kremer-Grest cell of "
                                  "100 x 100 beads per rate (LJ to 2.5 sigma, T = 0.1, dt 0.005)",
                   "cells": len(RATES), "atoms": natoms, "md_steps_per_step": 1, "lanes_per_atom": lanes, "bin_factor": binf},
                  roofline,
                  extra={"load_step_path_atom_steps_per_s": natoms * nld * N / elapsed_b,
                         "tensile_stress_curves": {"columns": ["strain", "direct MD (mean over the load step's "
                                                               "window)", "r-cell load steps of 100 MD steps"],
                                                   "by_rate": curves}})
    if not args.no_cpu_baseline:
        F1 = np.stack([uniaxial_isochoric(0.01)])
        cb, _ = oracle_sample(params, [cell0], F1, 20, "one of the glassy cells")
        out["cpu_baseline"] = cb
    return out


# The FE workloads: mesh, r-cell generator, MD steps per load step, neighbour skin and the text of
# the line.  The skin changes speed only (never the pairs within rc); the values are the fastest of a
# sweep on one MI355X (0.3 - 0.8 sigma): the bar's 40 000-bead cells rebuild more often than smaller
# ones (the largest displacement is taken over more atoms), so a wider skin pays there.
FE_WORKLOADS = {
    "fe_bar": dict(mesh=("hex8", (8, 2, 2), (200.0, 50.0, 50.0), 0.95), cell=_fe_bar_cell, md=500, skin=0.7,
                   text="explicit hex8 bar 8x2x2 elements x 8 Gauss points = 256 Kremer-Grest r-cells of 400 "
                        "chains x 100 beads, imperfection-seeded neck"),
    "fe_tet": dict(mesh=("tet4", (5, 2, 2), (150.0, 150.0, 150.0), 1.0), cell=_fe_tet_cell, md=500, skin=0.55,
                   text="the paper's cubic polymer specimen: 100 C3D4 tetrahedra, one quadrature point each = 100 "
                        "Kremer-Grest r-cells of 100 chains x 100 beads (10^6 beads)"),
    "fe_scaling": dict(mesh=("tet4", (8, 5, 5), (200.0, 200.0, 200.0), 1.0), cell=_fe_scaling_cell, md=100,
                       skin=0.55,
                       text="the paper's scaling system on one GPU: 1000 C3D4 tetrahedra = 1000 Kremer-Grest "
                            "r-cells of 100 chains x 100 beads (10^7 beads)"),
}


def bench_fe(args, torch, rcell, configs, name):
    import numpy as np
    from paper_1902_09171_amd import fe
    spec = FE_WORKLOADS[name]
    MD_PER_LOAD = spec["md"]
    kind, nel, size, imp = spec["mesh"]
    mesh = (fe.Hex8Bar if kind == "hex8" else fe.Tet4Bar)(nel=nel, size=size, rho0=0.85, imperfection=imp)
    log(f"generating {mesh.ngp} r-cells")
    cells = make_cells(spec["cell"], list(range(mesh.ngp)))
    params = configs.kg_params(precision="mixed", skin=spec["skin"])
    natoms = sum(len(c["x"]) for c in cells)
    log(f"creating the batch: {natoms} beads")
    md = fe.MDStress(params, cells, MD_PER_LOAD)
    lanes, binf = tune(md.g, args)
    dt = MD_PER_LOAD * params["dt"]
    # 1 % nominal strain per load step
    bar = fe.ExplicitBar(mesh, md, dt=dt, pull_velocity=0.01 * mesh.size[0] / dt, damping=0.2)
    for _ in range(args.warmup):
        bar.step()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    step_s = []                    # each load step ends with the stress on the host (synchronised)
    for k in range(args.steps):
        ts = time.perf_counter()
        bar.step()
        step_s.append(time.perf_counter() - ts)
        log(f"load step {k + 1}/{args.steps}: tensile stress {bar.history[-1]['tensile']:.4f}")
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    (avg_s, n), _ = kernel_avg(md.g, 0, lambda: md.g.run(100))
    check_status(md.g)
    achieved = BYTES_PER_BEAD_STEP * natoms / avg_s
    roofline = {"bound": "hbm", "achieved": achieved / 1e9, "peak": PEAK_HBM / 1e9, "unit": "GB/s",
                "frac": achieved / PEAK_HBM, "traffic": traffic_from_profiles("k_force_kg", name),
                "kernel": "k_force_kg", "avg_us": avg_s * 1e6, "launches": n,
                "bytes_per_launch": BYTES_PER_BEAD_STEP * natoms}
    out = md_line(args, name, natoms * MD_PER_LOAD * args.steps / elapsed, elapsed, natoms,
                  {"description": spec["text"] + f", 1 % nominal strain per load step, {MD_PER_LOAD} MD steps "
                                                 "per load step",
                   "cells": mesh.ngp, "atoms": natoms, "md_steps_per_step": MD_PER_LOAD,
                   "lanes_per_atom": lanes, "bin_factor": binf, "skin": params["skin"], "rebuilds": md.g.rebuilds()}, roofline,
                  extra={"fe_wall_s_per_load_step": elapsed / args.steps,
                         "load_step_ms": {"median": float(np.median(step_s)) * 1e3, "min": min(step_s) * 1e3,
                                          "max": max(step_s) * 1e3}})
    if not args.no_cpu_baseline:
        sub = list(range(min(len(cells), host_threads())))
        F = np.stack([np.eye(3)] * len(sub))
        cb, s_ora = oracle_sample(params, [cells[c] for c in sub], F, 20,
                                  f"{len(sub)} of the r-cells (one per host thread), from rest")
        out["cpu_baseline"] = cb
        out["stress_rel_err_vs_oracle"] = gpu_sample_error(rcell, params, [cells[c] for c in sub], F, 20,
                                                           s_ora, lanes, binf)
    return out


def bench_surrogate(args, torch, rcell, configs):
    import numpy as np
    from paper_1902_09171_amd import rsur
    from synth.surrogate import init_params
    DIN, WIDTH, DEPTH, DOUT, K = 153, 256, 4, 6, 5
    B_BAR, B_BIG, B_TRAIN = 256, 65536, 4096
    dev = torch.device("cuda:0")
    stream = torch.cuda.Stream(device=dev)            # an explicit stream: the events below time it
    net = rsur.Surrogate(din=DIN, width=WIDTH, depth=DEPTH, dout=DOUT, ensemble=K, max_batch=B_BIG,
                         stream=stream.cuda_stream)
    for k in range(K):
        net.set_params(k, init_params(net.dims, 7, k))
    macs = DIN * WIDTH + (DEPTH - 1) * WIDTH * WIDTH + WIDTH * DOUT
    flop_eval = 2 * macs                              # per evaluation per member
    gen = torch.Generator(device=dev).manual_seed(1)
    X = torch.randn((B_BIG, DIN), generator=gen, device=dev, dtype=torch.float32)
    Y = torch.randn((B_BIG, DOUT), generator=gen, device=dev, dtype=torch.float32)
    mean = torch.zeros((B_BIG, DOUT), device=dev)
    var = torch.zeros_like(mean)
    torch.cuda.synchronize()
    net.fit_norm(X.data_ptr(), Y.data_ptr(), B_BIG)

    def timed(fn, reps):
        for _ in range(max(1, reps // 10)):
            fn()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        e0.record(stream)
        for _ in range(reps):
            fn()
        e1.record(stream)
        torch.cuda.synchronize()
        return (time.perf_counter() - t0) / reps, e0.elapsed_time(e1) / 1e3 / reps

    fwd_bar = lambda: net.forward(X.data_ptr(), B_BAR, mean.data_ptr(), var.data_ptr())
    fwd_big = lambda: net.forward(X.data_ptr(), B_BIG, mean.data_ptr(), var.data_ptr())
    trn = lambda: net.train_step(X.data_ptr(), Y.data_ptr(), B_TRAIN, 1e-4, want_loss=False)
    for _ in range(args.warmup):
        fwd_bar()
    t_bar, ev_bar = timed(fwd_bar, args.steps)
    t_big, ev_big = timed(fwd_big, max(10, args.steps // 10))
    t_trn, ev_trn = timed(trn, max(10, args.steps // 4))
    achieved = flop_eval * K * B_BIG / ev_big
    roofline = {"bound": "mfma", "achieved": achieved / 1e12, "peak": PEAK_BF16 / 1e12, "unit": "TFLOP/s",
                "frac": achieved / PEAK_BF16, "traffic": None,
                "kernel": "forward pass (k_mlp_forward over the ensemble, k_ensemble)",
                "avg_us": ev_big * 1e6, "batch": B_BIG, "flop_per_launch": flop_eval * K * B_BIG}
    out = {"metric": "surrogate stress-evals/s (ensemble of 5)", "value": B_BAR / t_bar, "unit": "evals/s",
           "n_gpus": 1, "steps": args.steps, "warmup": args.warmup, "ms_per_step": t_bar * 1e3,
           "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
           "dtype": "bf16 matrix products, f32 accumulation and master weights", "data": "synthetic",
           "config": {"workload": "surrogate", "description": "MLP 153 -> 4 x 256 -> 6, ensemble of 5, "
                      "random-init weights; a step is one ensemble evaluation of the FE bar's 256 Gauss "
                      "points", "batch": B_BAR, "params_per_member": macs + 4 * WIDTH + DOUT},
           "gpu_us_per_call_at_batch": ev_bar * 1e6,
           "evals_per_s_large_batch": B_BIG / t_big, "large_batch": B_BIG,
           "train_samples_per_s": B_TRAIN / t_trn, "train_batch": B_TRAIN,
           "roofline": roofline}
    if not args.no_cpu_baseline:
        from oracle import surrogate as osur
        Ws = [net.get_params(k) for k in range(K)]
        Xh = X[:B_BAR].double().cpu().numpy()
        reps = 0
        t0 = time.perf_counter()
        while time.perf_counter() - t0 < 2.0:
            for k in range(K):
                osur.forward(Ws[k], net.dims, Xh)
            reps += 1
        dt = (time.perf_counter() - t0) / reps
        out["cpu_baseline"] = {"value": B_BAR / dt, "unit": "evals/s", "cores": 1, "kind": "oracle",
                               "sample": f"FP64 numpy forward of the 5 members on {B_BAR} inputs, {reps} repeats"}
    return out


SUR_CHAINS = 40                   # chains of 100 beads per training r-cell


def _sur_melt(c):
    from synth import configs
    from synth.rng import cell_seed
    return configs.kg_cell([100] * SUR_CHAINS, cell_seed(1902 + 31, c))


def bench_fe_bar_surrogate(args, torch, rcell, configs):
    """The FE bar of fe_bar driven by the learned stress surrogate (153 -> 4 x 256 -> 6, ensemble of
    5), with batched MD as its fallback:
      (1) training data from MD-driven bars of the same mesh stepped in lockstep in one batched
          r-cell context (cells of --sur-chains x 100 beads, 500 MD steps per load step, other
          imperfections and pull rates), one (history, sigma_MD) pair per Gauss point per load step;
      (2) the ensemble trained by the library's BF16 kernels; the OOD threshold is the largest
          ensemble spread met on the held-out bars;
      (3) the bar of 256 r-cells of 40 000 beads driven by the surrogate for the evaluation load
          steps, while two shadow MD batches of the same cells (two Langevin seeds) follow its
          deformation: the surrogate's stress error per Gauss point and load step against shadow MD
          beside the seed-to-seed spread, the fallback fraction, and the time per load step against
          the MD load step.  The value (ensemble evaluations per second at the bar's 256 Gauss
          points) is reported only when the error bound holds."""
    import numpy as np
    from paper_1902_09171_amd import fe, rsur, surrogate as SU
    from synth.rng import generator
    from synth.surrogate import init_params
    global SUR_CHAINS
    MD, WARM, NGP = 500, 2000, 256
    params = configs.kg_params(precision="mixed")
    NB, NDIST, NLOAD, NEVAL = args.sur_bars, args.sur_melts, args.sur_load, args.sur_eval_load
    SUR_CHAINS = args.sur_chains
    NBEAD = 100 * SUR_CHAINS
    # stress-magnitude floor of the error measure: the thermal pressure scale rho k_B T of the melt;
    # below it the window stress of one r-cell is dominated by its own fluctuations
    S_FLOOR = 0.85 * params["kB"] * params["temperature"]
    rng = generator(1902 + 32, 0)
    log(f"generating {NDIST} training melts of {SUR_CHAINS} x 100 beads")
    melts = make_cells(_sur_melt, list(range(NDIST)))
    meshes, cells, rates = [], [], []
    for b in range(NB):
        meshes.append(fe.Hex8Bar(nel=(8, 2, 2), size=(200.0, 50.0, 50.0), rho0=0.85,
                                 imperfection=float(rng.uniform(0.9, 1.0))))
        rates.append(float(rng.uniform(0.006, 0.014)))
        cells.append([melts[(b * NGP + g) % NDIST] for g in range(NGP)])
    log(f"training data: {NB} bars x {NGP} Gauss points x {NLOAD} load steps of {MD} MD steps")
    net = rsur.Surrogate(din=SU.FEATURES, width=256, depth=4, dout=6, ensemble=5, max_batch=4096)
    for k in range(5):
        net.set_params(k, init_params(net.dims, 41, k))
    c_wave = fe.md_wave_speed(params, melts[:8], 0.85, MD, warmup_steps=WARM)
    tr = SU.train_on_bars(torch, net, params, meshes, cells, NLOAD, MD, rates, WARM, args.sur_train_steps,
                          holdout=max(1, NB // 8), wave_speed=c_wave,
                          progress=lambda k: (k % 10 == 9) and log(f"  load step {k + 1}/{NLOAD}"))
    atom_steps_gen = NB * NGP * NBEAD * (WARM + NLOAD * MD)
    ntrain = int((~tr["held"]).sum())
    losses = tr["losses"]
    log(f"  {len(tr['X'])} pairs in {tr['t_gen']:.1f} s ({atom_steps_gen / tr['t_gen']:.3e} atom-steps/s); "
        f"trained on {ntrain} in {tr['t_train']:.1f} s, loss {losses[0][1]:.4f} -> {losses[-1][1]:.4f}")

    # the bar of fe_bar, driven by the surrogate; shadow MD of its own cells follows its deformation
    log("generating the bar's 256 r-cells of 40 000 beads")
    bcells = make_cells(_fe_bar_cell, list(range(NGP)))
    mesh = fe.Hex8Bar(nel=(8, 2, 2), size=(200.0, 50.0, 50.0), rho0=0.85, imperfection=0.95)
    sur = SU.SurrogateStress(torch, net, tr["y_sd"], tr["tau"], params, bcells, MD, warmup_steps=WARM)

    def progress(k, o):
        if k % 10 == 9:
            log(f"  eval load step {k + 1}/{NEVAL}: median error {np.median(o['rel'][-1]):.4f} "
                f"(MD seed-to-seed {np.median(o['floor'][-1]):.4f}), |sigma| {np.median(o['mags'][-1]):.3f}, "
                f"flagged {sur.flag_log[-1]}")
    ev = SU.shadow_evaluation(torch, sur, params, mesh, bcells, MD, NEVAL, 0.01, WARM, S_FLOOR, wave_speed=c_wave,
                              progress=progress)
    rel, floor, mags, dev, dev_floor = ev["rel"], ev["floor"], ev["mags"], ev["dev"], ev["dev_floor"]
    t_sur, t_md, bar = ev["t_provider"], ev["t_md"], ev["bar"]
    med, flo = np.median(rel, 1), np.median(floor, 1)
    ok = bool(np.all(med <= 0.05))
    err_ho = tr["err_ho"]
    tau = tr["tau"]
    dt = MD * params["dt"]
    # ensemble evaluations per second at the bar's batch, device time of the forward calls
    Xd = torch.tensor(sur.hist.features().astype(np.float32), device="cuda:0")
    m = torch.zeros((NGP, 6), device="cuda:0")
    v = torch.zeros_like(m)
    for _ in range(20):
        net.forward(Xd.data_ptr(), NGP, m.data_ptr(), v.data_ptr())
    torch.cuda.synchronize()
    reps = 200
    t0 = time.perf_counter()
    for _ in range(reps):
        net.forward(Xd.data_ptr(), NGP, m.data_ptr(), v.data_ptr())
    torch.cuda.synchronize()
    t_fwd = (time.perf_counter() - t0) / reps
    if args.dump:
        np.savez_compressed(args.dump, rel=rel, floor=floor, mags=mags, t_sur=t_sur, t_md=t_md,
                            flags=np.array(sur.flag_log), err_ho=err_ho, losses=np.array(losses),
                            spread_ho=tr["spread_ho"], strain=np.array([h["strain"] for h in bar.history]),
                            dev=dev, dev_floor=dev_floor, tensile=np.array([h["tensile"] for h in bar.history]))
    value = NGP / t_fwd
    flagged = float(np.sum(sur.flag_log)) / (NEVAL * NGP)
    out = {"metric": "surrogate stress-evals/s at <=5% stress error", "value": value if ok else None,
           "unit": "evals/s", "n_gpus": 1, "steps": NEVAL, "warmup": 0, "ms_per_step": float(np.mean(t_sur)) * 1e3,
           "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
           "dtype": "bf16 matrix products, f32 accumulation; MD f32 pair forces, f64 integration/stress",
           "data": "synthetic",
           "config": {"workload": "fe_bar_surrogate",
                      "description": "the fe_bar bar (8x2x2 hex8, 256 Gauss points, r-cells of 400 x 100 beads, "
                                     "1 % nominal strain and 500 MD steps per load step) driven by the surrogate "
                                     "153 -> 4 x 256 -> 6, ensemble of 5, batched MD fallback above the OOD "
                                     "threshold; a step is one FE load step",
                      "training_pairs": ntrain, "training_bars": NB, "training_cell_beads": NBEAD,
                      "training_melts": NDIST, "load_steps_per_bar": NLOAD, "md_steps_per_load_step": MD,
                      "warmup_md_steps": WARM, "eval_load_steps": NEVAL},
           "error_gate": {"held": ok, "rule": "at every load step, the median over the 256 Gauss points of "
                                              "|sigma_sur - sigma_MD|_F / max(|sigma_MD|_F, rho kB T) <= 0.05, "
                                              "sigma_MD from shadow MD of the same cells following the surrogate "
                                              "bar's deformation; rho kB T = 0.85 eps/sigma^3",
                          "stress_floor": S_FLOOR,
                          "median_per_load_step_max": float(med.max()), "median_per_load_step_mean": float(med.mean()),
                          "p95_all": float(np.quantile(rel, 0.95)),
                          "md_seed_to_seed_median_per_load_step_max": float(flo.max()),
                          "md_seed_to_seed_median_mean": float(flo.mean()),
                          "deviatoric_median_per_load_step_max": float(np.median(dev, 1).max()),
                          "deviatoric_md_seed_to_seed_median_max": float(np.median(dev_floor, 1).max()),
                          "per_load_step": {"strain": [round(float(h["strain"]), 4) for h in bar.history],
                                            "median": [round(float(v), 5) for v in med],
                                            "md_seed_to_seed_median": [round(float(v), 5) for v in flo],
                                            "median_sigma_md": [round(float(v), 4) for v in np.median(mags, 1)]},
                          "held_out_bars_median_vs_training_cells": float(np.median(err_ho)),
                          "held_out_bars_p95_vs_training_cells": float(np.quantile(err_ho, 0.95))},
           "fallback_fraction": flagged, "ood_threshold": tau,
           "time_per_load_step_s": {"surrogate": float(np.mean(t_sur)), "md": float(np.mean(t_md)),
                                    "speedup": float(np.mean(t_md) / np.mean(t_sur)),
                                    "surrogate_median": float(np.median(t_sur)),
                                    "speedup_median": float(np.median(t_md) / np.median(t_sur))},
           "ensemble_forward_us_at_256": t_fwd * 1e6,
           "generation": {"pairs": int(len(tr["X"])), "seconds": tr["t_gen"],
                          "atom_steps_per_s": atom_steps_gen / tr["t_gen"]},
           "training": {"steps": args.sur_train_steps, "batch": 4096, "seconds": tr["t_train"],
                        "loss_first": losses[0][1], "loss_last": losses[-1][1]},
           "cfl": {"wave_speed": c_wave, "dt_fe": dt, "limit": fe.cfl_limit(mesh, c_wave)},
           "roofline": {"bound": "mfma", "achieved": 2 * 237312 * 5 * NGP / t_fwd / 1e12, "peak": PEAK_BF16 / 1e12,
                        "unit": "TFLOP/s", "frac": 2 * 237312 * 5 * NGP / t_fwd / PEAK_BF16, "traffic": None,
                        "kernel": "ensemble forward at batch 256 (latency bound)", "avg_us": t_fwd * 1e6}}
    if not ok:
        out["note"] = "the error bound did not hold: value withheld"
    return out


WORKLOADS = {"cu_element": bench_cu_element, "cu_batched": bench_cu_batched, "kg_single": bench_kg_single,
             "kg_batched": bench_kg_batched, "kg_glassy": bench_kg_glassy,
             "fe_bar": lambda *a: bench_fe(*a, name="fe_bar"), "fe_tet": lambda *a: bench_fe(*a, name="fe_tet"),
             "fe_scaling": lambda *a: bench_fe(*a, name="fe_scaling"), "glassy_rates": bench_glassy_rates,
             "surrogate": bench_surrogate, "fe_bar_surrogate": bench_fe_bar_surrogate}


def main():
    global ORACLE_SECONDS
    ap = argparse.ArgumentParser()
    ap.add_argument("--workload", default="fe_bar", choices=sorted(WORKLOADS))
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=None)
    ap.add_argument("--warmup", type=int, default=None)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--cpu-sample-steps", type=int, default=25)
    ap.add_argument("--no-peak-probe", action="store_true",
                    help="skip the copy / FMA probe that reports measured peaks")
    ap.add_argument("--cpu-seconds", type=float, default=ORACLE_SECONDS,
                    help="CPU time of the oracle baseline sample")
    ap.add_argument("--lanes", type=int, default=0, help="lanes per atom (0 = autotune)")
    ap.add_argument("--skin", type=float, default=None,
                    help="neighbour skin override for the MD workloads (changes speed, never the pairs within rc)")
    ap.add_argument("--sur-bars", type=int, default=32, help="fe_bar_surrogate: training bars")
    ap.add_argument("--sur-melts", type=int, default=512, help="fe_bar_surrogate: distinct training melts")
    ap.add_argument("--sur-load", type=int, default=125, help="fe_bar_surrogate: load steps per training bar")
    ap.add_argument("--sur-eval-load", type=int, default=100, help="fe_bar_surrogate: evaluated load steps")
    ap.add_argument("--sur-train-steps", type=int, default=30000, help="fe_bar_surrogate: Adam steps")
    ap.add_argument("--sur-chains", type=int, default=40, help="fe_bar_surrogate: 100-bead chains per training cell")
    ap.add_argument("--dump", default=None, help="fe_bar_surrogate: write the per-step errors to this .npz")
    ap.add_argument("--copy-probe-mb", type=int, default=0,
                    help="first run one plain device copy of this many MiB (calibrates HBM counters)")
    args = ap.parse_args()
    if args.gpus != 1:
        print(json.dumps({"error": "the r-cell library runs on one GPU; sharding the cells "
                                   "over several GPUs is not implemented", "n_gpus": args.gpus}))
        sys.exit(2)
    ORACLE_SECONDS = args.cpu_seconds
    d_steps, d_warm = DEFAULTS[args.workload]
    args.steps = d_steps if args.steps is None else args.steps
    args.warmup = d_warm if args.warmup is None else args.warmup
    if args.steps < 1 or args.warmup < 0:
        print(json.dumps({"error": "--steps must be at least 1 and --warmup at least 0",
                          "steps": args.steps, "warmup": args.warmup}))
        sys.exit(2)

    import torch
    from paper_1902_09171_amd import rcell
    from synth import configs
    rcell.load()

    if args.copy_probe_mb > 0:
        n = args.copy_probe_mb * (1 << 20) // 4
        src = torch.ones(n, dtype=torch.float32, device="cuda:0")
        dst = torch.empty_like(src)
        dst.copy_(src)
        torch.cuda.synchronize()
        del src, dst

    if args.skin is not None:
        for name in ("kg_params", "cu_params"):
            base = getattr(configs, name)
            setattr(configs, name, (lambda b: lambda **over: dict(b(**over), skin=args.skin))(base))
    out = WORKLOADS[args.workload](args, torch, rcell, configs)
    if args.skin is not None:
        out["config"]["skin"] = args.skin
    if not args.no_peak_probe:
        # after the timed region: the peaks this GPU delivers, beside the published ones
        gbs, tf = rcell.probe_peaks(1 << 30, torch.cuda.current_stream().cuda_stream)
        r = out["roofline"]
        r["measured_peaks"] = {"copy_GBs": gbs, "fp32_fma_TFLOPs": tf,
                               "probe": "1 GiB device copy (read + write) and FP32 FMA chains on every CU, "
                                        "non-packed as in the MD kernels"}
        meas = {"hbm": gbs, "alu": tf}.get(r["bound"])
        if meas:
            r["frac_of_measured_peak"] = r["achieved"] / meas
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
