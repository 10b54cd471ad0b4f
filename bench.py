"""Throughput of the N-component free-energy LBM update on one MI355X.

Workload: D3Q19 quaternary phase separation with a fifth component that is
exactly zero (the reduction-consistency check), 256^3 periodic nodes,
C_i = 0.25 + U(-0.02, 0.02) renormalised (seed 0), sigma = 0.01 for every
pair, tau = tau_g = 1, m = 0.1.  One "step" is one full time step of the
method over the whole lattice (concentration reconstruction + the fused
stencil / force / collide / stream launch).

Prints ONE JSON line.  value = MLUPS (million lattice-node updates per second)
of the FP32-storage form; the FP16S and FP64 forms are timed the same way and
reported under "forms".  roofline: the update kernel's algorithmic HBM bytes
per launch divided by its mean launch time (HIP events on the stream the
kernel runs on), against the 8 TB/s HBM3E peak.  cpu_baseline: the FP64 NumPy
oracle on a 64^3 sample of the same recipe.
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

METRIC = "MLUPS at N components (FP32/FP16-store vs FP64) and % of HBM roofline"
HBM_PEAK_GBS = 8000.0
Q = 19


def update_bytes_per_node(N, fs, g0s, ts, rs, form, fform="populations"):
    """Algorithmic HBM bytes of one update launch per node (halo re-reads of
    C and E_B not counted).  Every form reads the N-1 reconstructed
    concentrations and E_B (ts bytes each).  f as populations: the Q-1 moving
    f are read and written (fs each); f as node records: the four moments of
    the streamed f are read and (fB, F) written (rs each).  The population
    form of g writes all Q populations of the N-1 evolved components, the
    moment form the records mu~ and (v, -3/2 v.v) (rs each)."""
    NE = N - 1
    fpart = 8 * rs if fform == "records" else 2 * (Q - 1) * fs
    common = fpart + (NE + 1) * ts
    if form == "moments":
        return common + (NE + 4) * rs
    return common + NE * ((Q - 1) * fs + g0s)


def conc_bytes_per_node(N, fs, g0s, ts, rs, form, fform="populations"):
    """Population form: read all Q populations of the N-1 evolved components,
    write C and E_B.  Moment form: read the node record C (ts), mu~ and
    (v, -3/2 v.v) (rs), write C and E_B (ts); with f as node records also
    read (fB, F) and write the four f moments (rs; neighbour records re-read
    from cache not counted)."""
    NE = N - 1
    if form == "moments":
        b = NE * ts + (NE + 4) * rs + (NE + 1) * ts
        return b + 8 * rs if fform == "records" else b
    return NE * ((Q - 1) * fs + g0s) + (NE + 1) * ts


# bytes of a stored value: moving population, rest population, compute
# value (C, E_B), node record (mu~, v, f records)
SIZES = {"fp64": (8, 8, 8, 8), "fp32": (4, 4, 4, 4), "fp16s": (2, 4, 4, 2)}
# bench form name -> (storage precision, extra creation flags)
FORMS = {"fp32": ("fp32", 0), "fp16s": ("fp16s", 0), "fp64": ("fp64", 0),
         "fp32_f_populations": ("fp32", 32), "fp32_populations": ("fp32", 4 | 32)}

# Per node of one launch at 256^3, from rocprofv3 on the kernel sources with
# the hash below: HBM bytes (FETCH_SIZE and WRITE_SIZE, each scaled by what
# the counter reads for a 1 GiB device copy: x2.0 and x1.0) and VALU
# instructions per lane (SQ_INSTS_VALU x 64 / nodes).  The committed summary
# under profiles/ gives the commands and the raw figures.
COUNTERS = {
    "sources_sha256": "3934672bb8852847e23efa0d1c33cb69a56ded3dbb3a899cafaeb783296748ab",
    "n": 256,
    "k_update": {"fp32": (85.0, 382.5), "fp16s": (53.0, 409.5), "fp64": (170.4, 433.3)},
    "k_conc_m": {"fp32": (104.0, 461.6), "fp16s": (71.5, 515.7), "fp64": (232.8, 559.4)},
}
# VALU issue peak: 256 CUs x 4 SIMDs x 16 lanes x 2.4 GHz (one lane-op per
# lane and cycle; packed FP32 is not generated by these builds).
VALU_PEAK_LANE_OPS = 256 * 4 * 16 * 2.4e9
KERNEL_SOURCES = ("paper_2605_22214_amd/csrc/kernels.hip", "paper_2605_22214_amd/csrc/device.h",
                  "paper_2605_22214_amd/csrc/internal.h")


def kernel_sources_sha256():
    h = hashlib.sha256()
    for rel in KERNEL_SOURCES:
        with open(os.path.join(ROOT, rel), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()


def run_form(nf, w, form, steps, warmup, timing_steps):
    import torch
    precname, flags = FORMS[form]
    prec = nf.PRECISIONS[precname]
    sim = nf.Simulation.from_workload(w, precision=prec, implicit=0, flags=flags)
    storage = sim.storage_form()
    fstorage = sim.f_storage_form()
    sim.set_fields(w["C0"])
    d0 = sim.diagnostics(vcm_component=0)
    sim.step(warmup)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    ms_events = sim.step_timed(steps)
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    # separate pass: events around every reconstruction and update launch
    # (the library's stream)
    ms_conc, ms_upd = sim.step_timed_kernels(timing_steps)
    d1 = sim.diagnostics(vcm_component=0)
    n = w["C0"][0].size
    mlups = n * steps / wall / 1e6
    fs, g0s, ts, rs = SIZES[precname]
    N = w["sigma"].shape[0]
    ub = update_bytes_per_node(N, fs, g0s, ts, rs, storage, fstorage)
    cb = conc_bytes_per_node(N, fs, g0s, ts, rs, storage, fstorage)
    upd_ms = ms_upd / timing_steps
    conc_ms = ms_conc / timing_steps
    out = {
        "storage_of_g": storage,
        "storage_of_f": fstorage,
        "mlups": mlups,
        "ms_per_step": wall / steps * 1e3,
        "ms_per_step_events": ms_events / steps,
        "update_ms": upd_ms,
        "update_bytes_per_node": ub,
        "step_bytes_per_node": ub + cb,
        "update_gbs": n * ub / (upd_ms * 1e-3) / 1e9,
        "conc_ms": conc_ms,
        "conc_bytes_per_node": cb,
        "conc_gbs": n * cb / (conc_ms * 1e-3) / 1e9,
        "step_gbs": n * (ub + cb) / (wall / steps) / 1e9,
        "absent_max_abs": d1["max_abs_c"][4],
        "mass_rel_drift": max(abs(a - b) / abs(b) for a, b in zip(d1["mass"][:4], d0["mass"][:4])),
        "momentum_drift": [a - b for a, b in zip(d1["momentum"], d0["momentum"])],
        "nan": d1["nan"],
    }
    out["step_frac_of_peak"] = out["step_gbs"] / HBM_PEAK_GBS
    # the usual LBM figure: every population of f (Q-1) and g (N Q) read and
    # written once per node update, priced at this form's storage size
    pop_model = 2 * fs * ((Q - 1) + N * Q)
    out["effective_gbs_population_model"] = mlups * 1e6 * pop_model / 1e9
    sim.close()
    return out


def run_batch(nf, count, steps, per_sim_steps, seed=0):
    """Batch of independent D2Q9 N=3 lens / Janus problems (sides 64..512 in
    steps of 32, sigma_13 and sigma_23 drawn from U[0.0025, 0.01]), FP32
    storage: whole-batch steps (the library's graph mode, in which these
    members take two steps a launch and no graph is replayed) against each
    member's own launch sequence.  MLUPS counts the nodes of all members."""
    import workloads as W
    ws = W.batch_members(count=count, seed=seed)
    b = nf.Batch.from_workloads(ws, precision=nf.FP32)
    for i, w in enumerate(ws):
        b.members[i].set_fields(w["C0"])
    nodes = b.nodes()
    tx, graph_steps, blocks = b.autotune()
    b.step(2 * graph_steps, "graph")
    ms_graph = b.step_timed(steps, "graph")
    ms_launch = b.step_timed(max(2, steps // 10), "launch")
    b.step(2, "per_sim")
    ms_per = b.step_timed(per_sim_steps, "per_sim")
    absent_nan = max(m.diagnostics(check=False)["nan"] for m in b.members[:8])
    b.close()
    graph = nodes * steps / (ms_graph * 1e-3) / 1e6
    per = nodes * per_sim_steps / (ms_per * 1e-3) / 1e6
    return {"workload": f"{count} independent D2Q9 N=3 lens/Janus problems, sides 64..512, FP32",
            "nodes": nodes, "tile_x": 1 << tx, "graph_steps": graph_steps, "workgroups": blocks,
            "graph_mlups": graph, "graph_steps_timed": steps,
            "launch_mlups": nodes * max(2, steps // 10) / (ms_launch * 1e-3) / 1e6,
            "per_sim_mlups": per, "per_sim_steps_timed": per_sim_steps,
            "speedup_graph_vs_per_sim": graph / per, "nan_in_first_8": absent_nan}


def run_variants(nf, side, steps, warmup=20):
    """The diffusive-only runs of Sec. IV B (Fig. 3 c, d) on a side^2 D2Q9
    lattice, N = 4, C_i from U[0, 2/N] renormalised (seed 0), FP32 storage:
    the constant mobility (m = 1/50, g in the moment form) and the
    concentration-dependent mobility of Appendix C (m* = 10, populations).
    MLUPS over `steps` timed steps.  They are taken several a launch, with
    the intermediate steps in LDS, so no bandwidth is derived from the library's
    count of what a separate step's kernels read and write."""
    import torch
    import workloads as W
    out = {}
    for name, m, flags in (("diffusive_constant_alpha", 1.0 / 50.0, nf.FLAG_NO_HYDRO),
                           ("diffusive_c2c2_alpha", 10.0, nf.FLAG_NO_HYDRO | nf.FLAG_C2C2_MOBILITY)):
        w = W.coarsening_2d(side, 4, seed=0, m=m)
        with nf.Simulation.from_workload(w, precision=nf.FP32, flags=flags) as sim:
            sim.set_fields(w["C0"])
            sim.step(warmup)
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            sim.step(steps)
            torch.cuda.synchronize()
            wall = time.perf_counter() - t0
            form = sim.storage_form()
        mlups = side * side * steps / wall / 1e6
        out[name] = {"mlups": mlups, "ms_per_step": wall / steps * 1e3, "storage_of_g": form}
    out["workload"] = f"D2Q9 N=4 {side}^2 periodic, U[0, 2/N] mixture, diffusive-only, FP32"
    return out


def run_small_configs(nf, steps, warmup=20):
    """Throughput of the smaller workloads of the parity tests, each stepped
    alone on the GPU as the library takes its steps (launch-bound at these sizes):
    the 64^2 liquid lens (D2Q9, N = 3, FP64), the 512^2 quaternary phase
    separation (D2Q9, N = 4, FP64 and FP32) and the 16 x 16 x 192 layered
    channel (D3Q19, N = 6, walls on z, FP32)."""
    import torch
    import workloads as W
    cases = (("lens_64sq_fp64", W.lens_2d(), nf.FP64),
             ("quaternary_512sq_fp64", W.quaternary_2d(512), nf.FP64),
             ("quaternary_512sq_fp32", W.quaternary_2d(512), nf.FP32),
             ("layered_16x16x192_fp32", W.layered_3d(), nf.FP32))
    out = {}
    for name, w, prec in cases:
        nodes = int(np.prod(w["shape"]))
        with nf.Simulation.from_workload(w, precision=prec) as sim:
            sim.set_fields(w["C0"], w.get("v0"))
            sim.step(warmup)
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            sim.step(steps)
            torch.cuda.synchronize()
            wall = time.perf_counter() - t0
        out[name] = {"mlups": nodes * steps / wall / 1e6, "ms_per_step": wall / steps * 1e3,
                     "nodes": nodes}
    return out


def run_boundaries(nf, steps, warmup=10):
    """Throughput with the boundary conditions of Sec. III C at a lattice that
    fills the GPU: a 256 x 128 x 128 D3Q19 channel, N = 4 mixture, FP32 storage,
    walls on x, y and z periodic: (a) an inlet on x- (u = 0.01, fixed C_b) and
    the convective outflow on x+, in the default storage form (node records
    of g and f) and with g and f as populations; (b) the same lattice with a
    square array of solid posts (8 x 8 nodes every 32 nodes in x and y,
    through z), node records.  Bytes per node are the library's count of what
    one step's kernels read and write."""
    import torch
    import workloads as W
    shape = (256, 128, 128)
    out = {}
    w = W.noise("D3Q19", shape, 4, seed=3)
    w["walls"] = (True, False, False)
    nx, ny, nz = shape
    post = np.zeros((nz, ny, nx), dtype=bool)
    for x0 in range(16, nx, 32):
        for y0 in range(12, ny, 32):
            post[:, y0:y0 + 8, x0:x0 + 8] = True
    for name in ("inlet_outflow", "inlet_outflow_populations", "solid_posts"):
        flags = nf.FLAG_G_POPULATIONS | nf.FLAG_F_POPULATIONS if name.endswith("populations") else 0
        with nf.Simulation.from_workload(w, precision=nf.FP32, flags=flags) as sim:
            if name.startswith("inlet"):
                sim.set_open_face(0, (0.01, 0.0, 0.0), (0.25, 0.25, 0.25, 0.25))
                sim.set_outflow(1)
            else:
                sim.set_solid(post)
            sim.set_fields(w["C0"])
            sim.step(warmup)
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            sim.step(steps)
            torch.cuda.synchronize()
            wall = time.perf_counter() - t0
            bpn = sim.bytes_per_node()
            form = (sim.storage_form(), sim.f_storage_form())
        mlups = nx * ny * nz * steps / wall / 1e6
        out[name] = {"mlups": mlups, "ms_per_step": wall / steps * 1e3, "bytes_per_node": bpn,
                     "step_gbs": mlups * 1e6 * bpn / 1e9, "storage_of_g": form[0], "storage_of_f": form[1]}
    out["workload"] = "D3Q19 N=4 256x128x128, walls on x, FP32"
    return out


def cpu_baseline(sample_n=64, steps=60):
    """The FP64 oracle (not tuned) on a sample_n^3 lattice of the same recipe."""
    import workloads as W
    from oracle import step as S
    from oracle.lattice import D3Q19
    w = W.quaternary_3d(sample_n)
    par = S.Params(D3Q19, w["shape"], w["sigma"], w["tau"], m=w["m"], implicit=0)
    f, g = S.initial_state(par, w["C0"])
    f, g, _ = S.step(f, g, par)
    t0 = time.perf_counter()
    for _ in range(steps):
        f, g, _ = S.step(f, g, par)
    dt = time.perf_counter() - t0
    return {"value": sample_n ** 3 * steps / dt / 1e6, "unit": "MLUPS", "cores": 1,
            "kind": "oracle",
            "sample": f"{sample_n}^3 D3Q19 N=5 (same recipe), {steps} steps, NumPy FP64 on one "
                      f"core ({len(os.sched_getaffinity(0))} visible), {dt:.1f} s"}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=1000)
    ap.add_argument("--warmup", type=int, default=20)
    ap.add_argument("--n", type=int, default=256, help="lattice side")
    ap.add_argument("--forms", default="fp32,fp16s,fp64,fp32_populations")
    ap.add_argument("--timing-steps", type=int, default=50)
    ap.add_argument("--no-cpu", action="store_true")
    ap.add_argument("--batch-count", type=int, default=256,
                    help="members of the batch measurement (0 skips it)")
    ap.add_argument("--batch-steps", type=int, default=2000)
    ap.add_argument("--variant-side", type=int, default=4096,
                    help="D2Q9 side of the diffusive-only / mobility-variant measurement (0 skips it)")
    ap.add_argument("--variant-steps", type=int, default=200)
    ap.add_argument("--small-steps", type=int, default=2000,
                    help="steps for the smaller workloads (0 skips them)")
    ap.add_argument("--boundary-steps", type=int, default=200,
                    help="steps for the boundary-condition runs (0 skips them)")
    ap.add_argument("--calibrate-copy", action="store_true",
                    help="only run a plain device copy of 1 GiB, 3 times (for scaling the "
                         "FETCH_SIZE / WRITE_SIZE counters)")
    args = ap.parse_args()
    if args.calibrate_copy:
        import torch
        a = torch.ones(1 << 28, dtype=torch.float32, device="cuda")
        b = torch.empty_like(a)
        for _ in range(3):
            b.copy_(a)
        torch.cuda.synchronize()
        print(json.dumps({"copy_bytes_per_launch": 4 * (1 << 28)}))
        return
    if args.gpus != 1:
        print(f"bench.py: this workload runs on one GPU; --gpus {args.gpus} is not supported "
              "(the library advances each lattice on a single GPU and has no domain decomposition)",
              file=sys.stderr)
        sys.exit(2)
    import torch
    if not torch.cuda.is_available():
        print("bench.py: no GPU visible", file=sys.stderr)
        sys.exit(1)
    import paper_2605_22214_amd as nf
    import workloads as W
    nf.lib()
    w = W.quaternary_3d(args.n)
    forms = [f for f in args.forms.split(",") if f]
    results = {}
    for form in forms:
        print(f"bench: timing {form} ({args.n}^3, {args.steps} steps)", file=sys.stderr, flush=True)
        results[form] = run_form(nf, w, form, args.steps, args.warmup, args.timing_steps)
        print(f"bench: {form} {results[form]['mlups']:.1f} MLUPS", file=sys.stderr, flush=True)
    batch = None
    if args.batch_count > 0:
        print(f"bench: batch of {args.batch_count} D2Q9 problems", file=sys.stderr, flush=True)
        batch = run_batch(nf, args.batch_count, args.batch_steps, max(2, args.batch_steps // 10))
        print(f"bench: batch {batch['graph_mlups']:.0f} MLUPS vs {batch['per_sim_mlups']:.0f} "
              "(per simulation)", file=sys.stderr, flush=True)
    variants = None
    if args.variant_side > 0:
        print(f"bench: diffusive-only variants on {args.variant_side}^2", file=sys.stderr, flush=True)
        variants = run_variants(nf, args.variant_side, args.variant_steps)
        print("bench: " + ", ".join(f"{k} {v['mlups']:.0f} MLUPS" for k, v in variants.items()
                                     if isinstance(v, dict)), file=sys.stderr, flush=True)
    small = None
    if args.small_steps > 0:
        print("bench: the smaller workloads", file=sys.stderr, flush=True)
        small = run_small_configs(nf, args.small_steps)
        print("bench: " + ", ".join(f"{k} {v['mlups']:.0f} MLUPS" for k, v in small.items()),
              file=sys.stderr, flush=True)
    bounds = None
    if args.boundary_steps > 0:
        print("bench: boundary conditions at 256x128x128", file=sys.stderr, flush=True)
        bounds = run_boundaries(nf, args.boundary_steps)
        print("bench: " + ", ".join(f"{k} {v['mlups']:.0f} MLUPS" for k, v in bounds.items()
                                     if isinstance(v, dict)), file=sys.stderr, flush=True)
    main_form = forms[0]
    r = results[main_form]
    # the dominant kernel: the one of the two launches of a step that takes
    # longer
    dom = "k_update" if r["update_ms"] >= r["conc_ms"] else "k_conc_m"
    dms, dgbs, dbpn = ((r["update_ms"], r["update_gbs"], r["update_bytes_per_node"]) if dom == "k_update"
                       else (r["conc_ms"], r["conc_gbs"], r["conc_bytes_per_node"]))
    traffic = None
    valu_frac = None
    if (kernel_sources_sha256() == COUNTERS["sources_sha256"] and args.n == COUNTERS["n"]
            and main_form in COUNTERS[dom]):
        b_node, valu_node = COUNTERS[dom][main_form]
        traffic = b_node * args.n ** 3
        valu_frac = valu_node * args.n ** 3 / (dms * 1e-3) / VALU_PEAK_LANE_OPS
    roof = {"bound": "hbm", "achieved": dgbs, "peak": HBM_PEAK_GBS, "unit": "GB/s",
            "frac": dgbs / HBM_PEAK_GBS, "traffic": traffic,
            "traffic_unit": "bytes per launch (FETCH_SIZE x2.0 + WRITE_SIZE x1.0)",
            "valu_issue_frac": valu_frac,
            "kernel": dom, "bytes_per_node": dbpn, "mean_launch_ms": dms,
            "step_frac": r["step_frac_of_peak"]}
    cpu = None
    if not args.no_cpu:
        print("bench: timing the CPU oracle sample", file=sys.stderr, flush=True)
        cpu = cpu_baseline()
    line = {
        "metric": METRIC,
        "value": r["mlups"],
        "unit": "MLUPS",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": r["ms_per_step"],
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": {"fp32": "f32", "fp16s": "f16-store/f32", "fp64": "f64"}[FORMS[main_form][0]],
        "data": "synthetic",
        "config": {"workload": f"D3Q19 quaternary phase separation + absent 5th component, "
                               f"{args.n}^3 periodic, {main_form} storage",
                   "lattice": "D3Q19", "shape": [args.n] * 3, "ncomp": 5, "precision": main_form},
        "roofline": roof,
        "cpu_baseline": cpu,
        "forms": results,
        "batch": batch,
        "variants": variants,
        "small_workloads": small,
        "boundaries": bounds,
    }
    print(json.dumps(line), flush=True)


if __name__ == "__main__":
    main()
