"""Benchmark: restricted power diagram + fractional chi + beta0 of 2,000 weighted sites over the ~132k-tet solid
torus (64^3 voxel grid, Kuhn tets), on one MI355X (the default workload; --workload genus3 and batch256 run the
2.1M-tet CAD-like solid and the 256-shape batch).

One step = one rpd_build call: candidate search, clipping, chi/beta0 reductions, sorted element lists copied to
the host. Inputs (the prepared mesh and the sites) are resident in HBM before the timed region. Prints one JSON
line; metric: tet-site clips/sec (nonempty pieces per second) with ms per RPD+chi beside it, for the FP32 path
with FP64/exact fallback (the reported value) and the all-FP64 path.
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

# MI355X published peaks (dense): FP32 vector 157.3 TFLOP/s (packed issue), FP64 vector 78.6 TFLOP/s; without
# packed FP32 instructions (the build disables them) the FP32 vector rate is that of FP64, 78.6 TFLOP/s
PEAK_FP32_TFLOPS = 157.3
PEAK_FP32_NONPACKED_TFLOPS = 78.6

# Algorithmic FLOPs of one nonempty piece with v vertices and f bisector faces: each bounding bisector is
# evaluated at the piece's vertices (8 v f), every vertex is constructed once (30 v) and enters the volume and
# moment fans (25 v). The mean over the pieces of each workload comes from the oracle's piece statistics
# (tests/golden/piece_stats.py writes tests/golden/piece_stats.json).
PIECE_STATS_FILE = os.path.join(ROOT, "tests", "golden", "piece_stats.json")


def flop_per_piece(workload: str) -> float:
    with open(PIECE_STATS_FILE) as fh:
        return float(json.load(fh)[workload]["flop_per_piece"])


# HBM traffic of the clipping kernels from rocprofv3 FETCH_SIZE / WRITE_SIZE runs (scaled by a plain copy of known
# size), valid only for the kernel sources it was measured on.
TRAFFIC_FILE = os.path.join(ROOT, "profiles", "traffic_clip.json")
KERNEL_SOURCES = ("clip.hip", "rpd_device.h", "rpd_common.h")


def kernel_source_hash() -> str:
    h = hashlib.sha256()
    for f in KERNEL_SOURCES:
        with open(os.path.join(ROOT, "paper_2403_18761_amd", "csrc", f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


def measured_counters(workload: str, kernel: str, launch: dict):
    """The committed counter summary of `kernel` on `workload` (HBM bytes and executed VALU FLOPs per launch), or
    None when there is none, it was taken with another launch shape, or the kernel sources changed since."""
    try:
        with open(TRAFFIC_FILE) as fh:
            d = json.load(fh)
    except (OSError, ValueError):
        return None
    e = d.get(workload, {})
    if e.get("source_hash") != kernel_source_hash() or e.get("kernel") != kernel or e.get("launch") != launch:
        return None
    return e


WORKLOADS = {
    "torus2000": dict(desc="solid torus R0.6 r0.25 (seed 2 jitter), 64^3 grid, 131838 Kuhn tets, 2000 sites uniform "
                           "inside with r = 0.9|sdf|", cpu_frac=1.0),
    "genus3": dict(desc="genus-3 CAD-like solid (three boxes minus three cylinders), 128^3 grid, 2142000 Kuhn tets, "
                        "20000 sites, 30% within 0.02 of sharp edges", cpu_frac=0.005),
    "batch256": dict(desc="256 seeded shapes (tori, box unions, metaballs), log-uniform 5k-200k tets and 100-5k sites "
                          "each, one rpd_build call", cpu_frac=0.002),
    "envelope": dict(desc="geometric-error metric: distance from 1M surface samples of the torus2000 shape to the "
                          "enveloping spheres, cones and slabs of its thinned (sigma 0.3) dual medial mesh",
                     cpu_frac=0.02),
    "repair": dict(desc="topology repair: 5 metaball blobs joined by thin handles (genus 2), 128^3 grid, 975462 Kuhn "
                        "tets, 500 initial sites, up to 64 insertions per round from a per-tet sphere table, one "
                        "captured graph per round (a step is one round)", cpu_frac=0.25),
}


def workload(name):
    from paper_2403_18761_amd import synth

    if name == "torus2000":
        return [synth.torus_inside(N=64, n_sites=2000, seed=2)]
    if name == "genus3":
        return [synth.genus3_cad(N=128, n_sites=20000, seed=3)]
    if name == "batch256":
        return synth.batch_problems(256, 4)
    if name == "repair":
        return [synth.repair_problem(N=128, n_sites=500, seed=5)]
    if name == "envelope":
        return [synth.torus_inside(N=64, n_sites=2000, seed=2)]
    raise SystemExit(f"unknown workload {name}")


def time_builds(meshes, sites, precision, steps, warmup, stream, block=0, clip_budget=0, flags=0, slots=0):
    """Times `steps` rpd_build calls (each returns with its results on the host, its stream synchronised).
    Returns a dict: mean ms per call over the timed region, median and p90 of the per-call times, the mean
    HIP-event time of the clipping kernels (group lists, candidates, pieces), the pieces and the last call's statistics."""
    import torch

    from paper_2403_18761_amd import rpd

    flags |= rpd.RPD_TIMING
    kw = dict(precision=precision, flags=flags, stream=stream, block=block, clip_budget=clip_budget, slots=slots)
    for _ in range(warmup):
        rpd.build(meshes, sites, **kw)
    torch.cuda.synchronize()
    clip_ms, per_call = [], []
    n_pairs = None
    t0 = time.perf_counter()
    for _ in range(steps):
        c0 = time.perf_counter()
        res = rpd.build(meshes, sites, **kw)
        per_call.append((time.perf_counter() - c0) * 1e3)
        st = res.stats()
        clip_ms.append(st["ms_clip"])
        n_pairs = st["n_pairs"]
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    return dict(ms=(t1 - t0) * 1e3 / steps, ms_median=float(np.median(per_call)),
                ms_p90=float(np.percentile(per_call, 90)), clip_ms=float(np.mean(clip_ms)), n_pairs=n_pairs,
                stats=st)


def batch_comparison(args, stream):
    """The 256-shape batch in one rpd_build call, FP32 + fallback (autotuned launch) against all-FP64, so that one
    benchmark line shows whether the batched FP32 path beats the all-FP64 one (no oracle leg)."""
    import torch

    from paper_2403_18761_amd import rpd

    t0 = time.perf_counter()
    probs = workload("batch256")
    dev = torch.device("cuda:0")

    def t(a, dt=torch.float32):
        return torch.as_tensor(np.ascontiguousarray(a), dtype=dt, device=dev)

    meshes = [rpd.Mesh(t(p.vx), t(p.vy), t(p.vz), t(p.tv.reshape(-1), torch.int32), stream=stream) for p in probs]
    sites = [(t(p.sx), t(p.sy), t(p.sz), t(p.sr)) for p in probs]
    torch.cuda.synchronize()
    prep_s = time.perf_counter() - t0
    tuned = rpd.autotune(meshes, sites, stream=stream)
    steps = args.batch_steps
    a = time_builds(meshes, sites, rpd.RPD_FP32_FALLBACK, steps, 1, stream, tuned["block"], tuned["clip_budget"],
                    slots=tuned["slots"])
    b = time_builds(meshes, sites, rpd.RPD_FP64, steps, 1, stream)
    assert a["n_pairs"] == b["n_pairs"]
    out = {"workload": WORKLOADS["batch256"]["desc"], "n_tets": sum(p.n_tets for p in probs),
           "n_sites": sum(p.n_sites for p in probs), "n_pairs": a["n_pairs"], "launch": tuned, "steps": steps,
           "fp32_ms": {"mean": a["ms"], "median": a["ms_median"], "p90": a["ms_p90"], "clip_kernel": a["clip_ms"]},
           "fp64_ms": {"mean": b["ms"], "median": b["ms_median"], "p90": b["ms_p90"], "clip_kernel": b["clip_ms"]},
           "fp32_clips_per_s": a["n_pairs"] / (a["ms"] * 1e-3), "fp32_speedup_over_fp64": b["ms"] / a["ms"],
           "input_prep_s": prep_s}
    print(f"# batch256: fp32+fallback {a['ms']:.2f} ms, all-fp64 {b['ms']:.2f} ms per call "
          f"({out['fp32_speedup_over_fp64']:.2f}x), launch {tuned}", file=sys.stderr, flush=True)
    return out


def invariants(meshes, sites, tuned):
    """One more (untimed) build in the timed launch shape, checked for properties that hold at any size: cell volumes
    partition each mesh, Euler additivity over the diagram equals the mesh's chi, every live element has beta0 >= 1."""
    from paper_2403_18761_amd import rpd

    res = rpd.build(meshes, sites, block=tuned["block"], clip_budget=tuned["clip_budget"], slots=tuned["slots"])
    worst_vol, bad = 0.0, 0
    medial = {"chi_mismatch_after_thinning": 0, "thin_ms": 0.0, "tets_left": 0}
    for k, m in enumerate(meshes):
        info = m.info()
        _, chi = res.euler(k, rpd.RPD_CELL)
        _, b0 = res.components(k, rpd.RPD_CELL)
        _, fchi = res.euler(k, rpd.RPD_FACE)
        _, echi = res.euler(k, rpd.RPD_EDGE)
        nrpv = len(res.adjacency(k, rpd.RPD_VERTEX))
        vol, _ = res.geometry(k)
        worst_vol = max(worst_vol, abs(vol.sum() - info["volume"]) / info["volume"])
        additive = int(chi.sum()) - int(fchi.sum()) + int(echi.sum()) - nrpv == info["euler"]
        bad += int(not additive) + int(np.any(b0[vol > 0] < 1))
        # dual medial mesh and its thinning (host), sigma 0.3: the removals keep the medial chi
        (V, E, F, T), mchi = res.medial_euler(k)
        if k == 0:
            medial.update(V=V, E=E, F=F, T=T, chi=mchi)
        _, alpha = res.edge_geometry(k)
        t0 = time.perf_counter()
        ke, kf, kt = rpd.thin(len(chi), res.adjacency(k, rpd.RPD_FACE), res.adjacency(k, rpd.RPD_EDGE), alpha,
                              res.adjacency(k, rpd.RPD_VERTEX), 0.3)
        medial["thin_ms"] += 1e3 * (time.perf_counter() - t0)
        medial["tets_left"] += int(kt.sum())
        medial["chi_mismatch_after_thinning"] += int(V - int(ke.sum()) + int(kf.sum()) - int(kt.sum()) != mchi)
    return {"volume_partition_rel_err_max": worst_vol, "shapes_failing_euler_or_beta0": bad, "shapes": len(meshes),
            "medial": medial}


def run_repair(args, prob, table):
    """One step = one round of the incremental session; value = (tet, site) pairs clipped per second in the timed
    rounds (removal and re-insertion passes of the dirty blocks). A from-scratch rebuild with the final sites is
    timed beside it."""
    import torch

    from paper_2403_18761_amd import rpd

    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)

    def t(a, dt=torch.float32):
        return torch.as_tensor(np.ascontiguousarray(a), dtype=dt, device=dev)

    max_insert = 64
    mesh = rpd.Mesh(t(prob.vx), t(prob.vy), t(prob.vz), t(prob.tv.reshape(-1), torch.int32))
    shrink = args.insertion == "shrink"
    t_create = time.perf_counter()
    sess = rpd.Session(mesh, (t(prob.sx), t(prob.sy), t(prob.sz), t(prob.sr)),
                       None if shrink else tuple(t(x) for x in table),
                       max_sites=prob.n_sites + max_insert * (args.steps + args.warmup), max_insert=max_insert,
                       insertion=rpd.RPD_INSERT_SHRINK if shrink else rpd.RPD_INSERT_TABLE)
    ms_create = (time.perf_counter() - t_create) * 1e3
    sess.run(args.warmup)
    i0 = sess.info()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    sess.run(args.steps)
    torch.cuda.synchronize()
    dt = time.perf_counter() - t0
    i1 = sess.info()
    res = sess.result()
    st = res.stats()
    _, chi = res.euler(0, rpd.RPD_CELL)
    _, b0 = res.components(0, rpd.RPD_CELL)
    vol, _ = res.geometry(0)
    live = vol > 0
    bad = int(np.sum(live & ((chi != 1) | (b0 > 1))))
    s = sess.sites()
    sites = tuple(t(s[:, k]) for k in range(4))
    full = time_builds([mesh], [sites], rpd.RPD_FP32_FALLBACK, 5, 1, None)
    ms_full = full["ms"]
    assert full["n_pairs"] == st["n_pairs"]
    clipped = i1["n_clipped"] - i0["n_clipped"]
    ms_round = dt * 1e3 / args.steps
    print(f"# repair: {ms_round:.3f} ms/round, {i1['n_inserted'] - i0['n_inserted']} inserted, "
          f"{i1['n_dirty_blocks'] - i0['n_dirty_blocks']} dirty blocks of {i1['n_blocks']} x {args.steps}, "
          f"rebuild {ms_full:.3f} ms, violating cells left {bad}, insertion {args.insertion}, session creation "
          f"{ms_create:.1f} ms", file=sys.stderr, flush=True)
    return dict(value=clipped / dt, ms_per_step=ms_round, n_pairs=st["n_pairs"], n_sites=int(s.shape[0]),
                extra={"ms_per_round": ms_round, "ms_full_rebuild_final_sites": ms_full,
                       "rounds_timed": args.steps, "inserted_timed": i1["n_inserted"] - i0["n_inserted"],
                       "dirty_blocks_timed": i1["n_dirty_blocks"] - i0["n_dirty_blocks"], "n_blocks": i1["n_blocks"],
                       "pairs_clipped_timed": clipped, "violating_cells_left": bad,
                       "sites_final": int(s.shape[0]), "insertion": args.insertion,
                       "ms_session_create": ms_create})


# Algorithmic FLOPs of one (sample, element) evaluation of the geometric-error kernel: d = q - c (3), then
# sphere: |d| (5 + sqrt) - r = 10; cone: u = d.axis (5), d x axis (9), |.|^2 (5), sqrt, t = u + c h (2),
# value (4) = 29; slab: H, g.d, two barycentric dots with their |H| terms (5 + 5 + 7 + 7), value (3) = 30.
FLOP_SPHERE, FLOP_CONE, FLOP_SLAB = 10, 29, 30


def run_envelope(args, prob):
    """One step = one rpd_envelope_distance call over every sample (inputs resident on the device; distances only,
    as the insertion test of Sec. 4.3 uses); value = (sample, element) pairs decided per second (evaluated, or passed
    over by their bounding spheres)."""
    import torch

    from paper_2403_18761_amd import rpd, synth

    dev = torch.device("cuda:0")

    def t(a, dt=torch.float32):
        return torch.as_tensor(np.ascontiguousarray(a), dtype=dt, device=dev)

    mesh = rpd.Mesh(t(prob.vx), t(prob.vy), t(prob.vz), t(prob.tv.reshape(-1), torch.int32))
    res = rpd.build([mesh], [(t(prob.sx), t(prob.sy), t(prob.sz), t(prob.sr))])
    S, E, F = res.medial_mesh(0, np.stack([prob.sx, prob.sy, prob.sz, prob.sr], axis=1), 0.3)
    q = synth.surface_samples(prob, 1_000_000, seed=4)
    dS, dE, dF, dq = t(S), t(E, torch.int32), t(F, torch.int32), t(q)
    for _ in range(args.warmup):
        rpd.envelope_distance(dS, dE, dF, dq, nearest=False)
    torch.cuda.synchronize()
    kms = []
    t0 = time.perf_counter()
    for _ in range(args.steps):
        d, _, k = rpd.envelope_distance(dS, dE, dF, dq, timing=True, nearest=False)
        kms.append(k)
    torch.cuda.synchronize()
    ms = (time.perf_counter() - t0) * 1e3 / args.steps
    kernel_ms = float(np.mean(kms))
    n_el = len(S) + len(E) + len(F)
    flops = len(q) * (FLOP_SPHERE * len(S) + FLOP_CONE * len(E) + FLOP_SLAB * len(F))
    achieved = flops / (kernel_ms * 1e-3) / 1e12
    print(f"# envelope: {len(S)} spheres {len(E)} cones {len(F)} slabs, {len(q)} samples: {ms:.3f} ms/call, "
          f"kernels {kernel_ms:.3f} ms", file=sys.stderr, flush=True)
    dist = d.cpu().numpy()
    return dict(value=len(q) * n_el / (ms * 1e-3), ms_per_step=ms, kernel_ms=kernel_ms, achieved=achieved,
                counts=dict(spheres=len(S), cones=len(E), slabs=len(F), samples=len(q)),
                checks=dict(finite=bool(np.all(np.isfinite(dist))), max_over_diag=float(dist.max() / np.sqrt(12.0)),
                            mean=float(dist.mean())),
                elements=(S, E, F), samples=q)


def cpu_baseline_envelope(S, E, F, q, frac):
    import oracle.envelope as env

    rng = np.random.default_rng(0)
    pick = rng.choice(len(q), max(1, int(frac * len(q))), replace=False)
    t0 = time.perf_counter()
    env.envelope_distance(S, E, F, q[pick])
    dt = time.perf_counter() - t0
    n_el = len(S) + len(E) + len(F)
    return dict(value=len(pick) * n_el / dt, unit="evaluations/s", cores=1, kind="oracle",
                sample=f"{len(pick)} of {len(q)} samples (random, seed 0) against all {n_el} elements, FP64 numpy "
                       f"in {dt:.2f} s")


def cpu_baseline(probs, frac):
    """The oracle (brute force over all sites, exact predicates) on a random sample of every shape's tets;
    clips/sec on the host."""
    import oracle

    oracle.build(force=False)
    threads = min(16, os.cpu_count() or 1)
    rng = np.random.default_rng(0)
    pieces = 0
    tets = 0
    dt = 0.0
    for prob in probs:
        sel = np.sort(rng.choice(prob.n_tets, max(1, int(frac * prob.n_tets)), replace=False))
        t0 = time.perf_counter()
        r = oracle.tet_pieces(prob, sel, threads=threads)
        dt += time.perf_counter() - t0
        pieces += len(r["pieces"])
        tets += len(sel)
    total = sum(p.n_tets for p in probs)
    # the per-core rate: one thread on a smaller random sample of the first shape
    sel1 = np.sort(rng.choice(probs[0].n_tets, max(1, int(frac * probs[0].n_tets / 20)), replace=False))
    t0 = time.perf_counter()
    r1 = oracle.tet_pieces(probs[0], sel1, threads=1)
    dt1 = time.perf_counter() - t0
    return dict(value=pieces / dt, unit="clips/s", cores=threads, kind="oracle",
                sample=f"{tets} of {total} tets (random {frac:g} of every shape, seed 0), each clipped against all "
                       f"sites of its shape; {pieces} nonempty pieces in {dt:.2f} s",
                one_thread={"value": len(r1["pieces"]) / dt1, "unit": "clips/s", "cores": 1,
                            "sample": f"{len(sel1)} tets of shape 0, {len(r1['pieces'])} pieces in {dt1:.2f} s"})


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--no-fp64", action="store_true", help="skip the all-FP64 comparison")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-estimated", action="store_true",
                    help="no effect (there is one dispatch order: nothing is learned from earlier builds)")
    ap.add_argument("--no-autotune", action="store_true", help="use the default launch shape (64 threads, k=28, 16 vertex slots)")
    ap.add_argument("--launch", default=None, metavar="BLOCK,K[,SLOTS]",
                    help="use this launch shape (threads per workgroup, clip budget, vertex slots: 16 if not given) "
                         "instead of autotuning")
    ap.add_argument("--cpu-frac", type=float, default=None)
    ap.add_argument("--no-batch", action="store_true",
                    help="torus workload: skip the 256-shape batch comparison of FP32 + fallback against all-FP64")
    ap.add_argument("--batch-steps", type=int, default=5)
    ap.add_argument("--workload", default="torus2000", choices=sorted(WORKLOADS))
    ap.add_argument("--insertion", default="table", choices=("table", "shrink"),
                    help="repair workload: spheres from the per-tet table, or shrunk at the furthest surface face")
    ap.add_argument("--calibrate-copy", type=int, default=0, metavar="MIB",
                    help="only run a plain device-to-device copy of MIB MiB (the reference kernel that scales the "
                         "FETCH_SIZE / WRITE_SIZE counters to bytes) and exit")
    args = ap.parse_args()
    if args.gpus != 1:
        print("the benchmark runs on one GPU only: sharding across GPUs is described, not implemented",
              file=sys.stderr)
        sys.exit(2)

    import torch

    from paper_2403_18761_amd import rpd

    if args.calibrate_copy:
        n = args.calibrate_copy * (1 << 20) // 4
        src = torch.ones(n, dtype=torch.float32, device="cuda:0")
        dst = torch.empty_like(src)
        for _ in range(3):
            dst.copy_(src)
        torch.cuda.synchronize()
        print(json.dumps({"calibrate_copy_bytes": 4 * n, "launches": 3}), flush=True)
        return

    probs = workload(args.workload)
    if args.workload == "repair":
        probs, table = [probs[0][0]], probs[0][1]
    print(f"# workload {args.workload}: {len(probs)} shape(s), {sum(p.n_tets for p in probs)} tets, "
          f"{sum(p.n_sites for p in probs)} sites", file=sys.stderr, flush=True)
    if args.workload == "envelope":
        r = run_envelope(args, probs[0])
        line = {
            "metric": "sample-element pairs decided/sec of the geometric-error metric, 1 MI355X",
            "value": r["value"], "unit": "evaluations/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
            "ms_per_step": r["ms_per_step"], "higher_is_better": True, "scaling": "strong", "vs_baseline": None,
            "dtype": "f32", "data": "synthetic",
            "config": {"workload": WORKLOADS[args.workload]["desc"], "name": args.workload, **r["counts"]},
            # the pairs that bounding spheres decide are not evaluated, so the work done is not known from the sizes
            # and no rate of the ALUs follows from them
            "roofline": {"bound": "alu", "achieved": None, "peak": PEAK_FP32_TFLOPS, "unit": "TFLOP/s", "frac": None,
                         "traffic": None, "kernel": "k_env_near", "kernel_ms": r["kernel_ms"],
                         "flop_per_evaluation": {"sphere": FLOP_SPHERE, "cone": FLOP_CONE, "slab": FLOP_SLAB},
                         "tflops_if_all_pairs_were_evaluated": r["achieved"]},
            "checks": r["checks"],
        }
        if not args.no_cpu_baseline:
            frac = args.cpu_frac if args.cpu_frac is not None else WORKLOADS[args.workload]["cpu_frac"]
            line["cpu_baseline"] = cpu_baseline_envelope(*r["elements"], r["samples"], frac)
        print(json.dumps(line), flush=True)
        return
    if args.workload == "repair":
        r = run_repair(args, probs[0], table)
        line = {
            "metric": "tet-site clips/sec in the incremental repair loop (dirty blocks only) + ms per round, 1 MI355X",
            "value": r["value"], "unit": "clips/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
            "ms_per_step": r["ms_per_step"], "higher_is_better": True, "scaling": "strong", "vs_baseline": None,
            "dtype": "f32", "data": "synthetic",
            "config": {"workload": WORKLOADS[args.workload]["desc"], "name": args.workload, "n_shapes": 1,
                       "n_tets": probs[0].n_tets, "n_sites_initial": probs[0].n_sites,
                       "n_pairs_final": r["n_pairs"]},
            "repair": r["extra"],
        }
        if not args.no_cpu_baseline:
            frac = args.cpu_frac if args.cpu_frac is not None else WORKLOADS[args.workload]["cpu_frac"]
            line["cpu_baseline"] = cpu_baseline(probs, frac)
        print(json.dumps(line), flush=True)
        return
    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)
    stream = torch.cuda.current_stream(dev)

    def t(a, dt=torch.float32):
        return torch.as_tensor(np.ascontiguousarray(a), dtype=dt, device=dev)

    meshes = [rpd.Mesh(t(p.vx), t(p.vy), t(p.vz), t(p.tv.reshape(-1), torch.int32), stream=stream) for p in probs]
    sites = [(t(p.sx), t(p.sy), t(p.sz), t(p.sr)) for p in probs]
    torch.cuda.synchronize()
    # the autotuner picks the launch shape for this bucket of shapes (untimed); rpd_build then uses it
    if args.launch:
        v = [int(x) for x in args.launch.split(",")]
        tuned = {"block": v[0], "clip_budget": v[1], "slots": v[2] if len(v) > 2 else 16}
    elif args.no_autotune:
        tuned = {"block": 64, "clip_budget": 28, "slots": 16}
    else:
        tuned = rpd.autotune(meshes, sites, stream=stream)
    print(f"# autotuned launch shape: {tuned}", file=sys.stderr, flush=True)

    f32 = time_builds(meshes, sites, rpd.RPD_FP32_FALLBACK, args.steps, args.warmup, stream, tuned["block"],
                      tuned["clip_budget"], slots=tuned["slots"])
    pairs, st32 = f32["n_pairs"], f32["stats"]
    print(f"# fp32+fallback: {f32['ms']:.3f} ms/RPD (median {f32['ms_median']:.3f}, p90 {f32['ms_p90']:.3f}), clip "
          f"kernel {f32['clip_ms']:.3f} ms, pairs {pairs}", file=sys.stderr, flush=True)
    # the same builds with whole blocks as work items of the candidate kernel
    ns_ = time_builds(meshes, sites, rpd.RPD_FP32_FALLBACK, args.steps, 1, stream, tuned["block"],
                      tuned["clip_budget"], flags=rpd.RPD_NO_SPLIT, slots=tuned["slots"])
    nosplit = {"ms_per_rpd": ns_["ms"], "ms_median": ns_["ms_median"], "clip_kernel_ms": ns_["clip_ms"]}
    print(f"# fp32+fallback, whole blocks as work items: {ns_['ms']:.3f} ms/RPD, clip kernel {ns_['clip_ms']:.3f} ms",
          file=sys.stderr, flush=True)
    out64 = None
    if not args.no_fp64:
        d = time_builds(meshes, sites, rpd.RPD_FP64, args.steps, args.warmup, stream)
        assert d["n_pairs"] == pairs
        out64 = dict(ms_per_rpd=d["ms"], ms_median=d["ms_median"], ms_p90=d["ms_p90"],
                     clips_per_s=pairs / (d["ms"] * 1e-3), clip_kernel_ms=d["clip_ms"],
                     fp32_speedup=d["ms"] / f32["ms"])
        print(f"# all-fp64: {d['ms']:.3f} ms/RPD, clip kernel {d['clip_ms']:.3f} ms", file=sys.stderr, flush=True)

    fpp = flop_per_piece(args.workload)
    achieved = fpp * pairs / (f32["clip_ms"] * 1e-3) / 1e12
    # ms_clip covers the group lists, the candidate kernel and the piece kernel
    kernel = f"k_candidates + k_clip_pieces<float,{tuned['slots'] if tuned['block'] == 64 else 16}>"
    cnt = measured_counters(args.workload, kernel, tuned) if len(probs) == 1 else None
    roof = {"bound": "alu", "achieved": achieved, "peak": PEAK_FP32_TFLOPS, "unit": "TFLOP/s",
            "frac": achieved / PEAK_FP32_TFLOPS, "traffic": cnt["bytes_per_launch"] if cnt else None,
            "kernel": kernel, "kernel_ms": f32["clip_ms"], "flop_per_piece": fpp,
            "frac_of_nonpacked_peak": achieved / PEAK_FP32_NONPACKED_TFLOPS}
    if cnt:  # executed work and HBM rate from the committed counter summary of this kernel and launch shape
        roof["executed_fp32_tflops"] = cnt["fp32_flop_per_launch"] / (f32["clip_ms"] * 1e-3) / 1e12
        roof["executed_fp32_frac"] = roof["executed_fp32_tflops"] / PEAK_FP32_TFLOPS
        roof["executed_fp64_tflops"] = cnt["fp64_flop_per_launch"] / (f32["clip_ms"] * 1e-3) / 1e12
        roof["valu_busy"] = cnt["valu_busy"]
        roof["hbm_gbps"] = cnt["bytes_per_launch"] / (f32["clip_ms"] * 1e-3) / 1e9
        roof["counters"] = cnt["summary"]
    line = {
        "metric": "tet-site clips/sec (nonempty pieces/s) + ms per RPD+chi, FP32/FP64-fallback vs all-FP64, 1 MI355X",
        "value": pairs / (f32["ms"] * 1e-3),
        "unit": "clips/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": f32["ms"],
        "higher_is_better": True,
        "scaling": "strong",
        "vs_baseline": None,
        "dtype": "f32",
        "data": "synthetic",
        "config": {"workload": WORKLOADS[args.workload]["desc"], "name": args.workload, "n_shapes": len(probs),
                   "n_tets": sum(p.n_tets for p in probs), "n_sites": sum(p.n_sites for p in probs),
                   "n_pairs": pairs, "launch": tuned},
        "ms_per_rpd": {"mean": f32["ms"], "median": f32["ms_median"], "p90": f32["ms_p90"]},
        "estimated_order": None,
        "all_fp64": out64,
        "stats": {k: st32[k] for k in ("n_candidates", "n_deferred", "n_fp64", "n_exact", "n_faces", "n_edges",
                                       "n_rpv", "n_defer_block", "n_defer_kmax", "n_defer_clip", "n_split", "n_items", "n_big",
                                       "ms_clip", "ms_deferred", "ms_reduce", "ms_total")},
        "no_split": nosplit,
        "roofline": roof,
    }
    if args.workload == "torus2000" and not args.no_batch:
        line["batch256"] = batch_comparison(args, stream)
    line["checks"] = invariants(meshes, sites, tuned)
    if not args.no_cpu_baseline:
        frac = args.cpu_frac if args.cpu_frac is not None else WORKLOADS[args.workload]["cpu_frac"]
        line["cpu_baseline"] = cpu_baseline(probs, frac)
    print(json.dumps(line), flush=True)


if __name__ == "__main__":
    main()
