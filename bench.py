"""Benchmark: node-tet pair evaluations per second on one MI355X.

One step = one bs_eval_velocity on the two-ring workload (a [-1.5,1.5]^3
box, 80^3 Kuhn-split cells: 531,441 nodes, 3,072,000 tetrahedra, jitter
0.2 h; two coaxial Gaussian-core rings, radii 1.0 and 0.8, sigma 0.08) with
the learned rule selector (trained first on the GPU by the library's own
kernels, outside the timed region), 16 x 16 angular rule, FP32 with
compensated accumulation.  Inputs are resident in HBM before the timed
region; the output goes to device memory.

Besides the headline, the same JSON line carries:
  fixed       the fixed distance rule (RT < 2 hbar, G11 < 4, G4 < 8, else G1)
              on the same mesh;
  accuracy    rel-L2 error of each policy at stored probe nodes against the
              exact velocity of the piecewise-linear vorticity
              (tests/golden/probe_exact_<workload>.json, written by a script
              that runs the FP64 oracle's references), and a ladder of fixed
              settings (cuts, lines) timed beside the learned policy: the
              speed ratio to the fastest fixed setting whose error is not
              above the learned policy's is "vs_fixed_equal_accuracy";
  treecode    the fixed and learned policies with the treecode far field
              (BS_FAR_TREECODE, theta 0.3, order 4: the fast-multipole-like
              evaluation of the 1-point pairs): time, error at the probes,
              speed against the same policy summing every pair, the far
              field's roofline; and at theta 0.2, order 6 its deviation from
              the all-pairs velocities at every node (within 1e-6);
  valu_far    the fixed rule with the far field on the vector ALUs
              (k_gauss_all, the design without matrix cores) and its roofline;
  c2, c3      the vortex-ring workload (97,175 nodes x 540,672 tets; the
              selector's training distribution) and the Fourier-curl box
              (117,649 x 663,552; held out): fixed, learned and learned with
              the treecode far field, timings and errors;
  lagrangian  Heun steps of the two-ring run with the learned policy
              (bs_advect_heun: mesh rebuild, two evaluations per step), and
              step 1 against the FP64 oracle's Heun step at sampled nodes
              (tests/golden/c5_heun_step1.json, an oracle-only script's
              output), with the fixed rule and with the learned policy;
  roofline    the longest kernel of the headline step alone (HIP events on
              its launch stream in a pass with every kernel on one stream),
              "roofline_kernels" lists far field, band and ray tracing;
  cpu_baseline  the FP64 oracle on a bounded sample of nodes x all tets.
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

import numpy as np  # noqa: E402

FP32_PEAK_TFLOPS = 157.3  # MI355X FP32 vector: 256 CUs x 2.4 GHz x 256 flop/clk
FLOPS_PER_POINT = 26.0     # one Gauss point: 3 sub, |r|^2 (5), rsqrt (1), r^-3 (2), W x r / r^3 + acc (15)
DEFAULT_CUTS = (2.0, 4.0, 8.0)
# fixed settings (near cut, G11 cut, G4 cut, lines per angle) timed for the
# equal-accuracy comparison: narrower ray-traced zones and more lines are
# more accurate at 16 x 16 and above
LADDER = ((1.5, 4.0, 8.0, 24), (1.5, 4.0, 8.0, 32), (1.0, 4.0, 8.0, 24), (2.0, 4.0, 8.0, 32), (2.0, 4.0, 8.0, 48))
TREE_THETA, TREE_ORDER = 0.3, 4  # the treecode leg's opening ratio and expansion order
TREE_EQUIV = (0.2, 6)             # a setting whose velocities equal the all-pairs sum within 1e-6


def expansion_flops(P):
    """Flops of one (node, cluster) expansion term as formulated: the
    offset from the centre's hi/lo split (9), |r|^2 (5), reciprocal and
    reciprocal square root (2), two scalings per degree (4 per degree), per
    Taylor coefficient of degree 1..P+1 the recurrence (2 per r_c term less 1,
    one add per further a_(m-2e_c) term, 1 mul, 2 for the second sum's FMA)
    and 6 for the contraction with the curl moments."""
    D = P + 1
    fl = 9 + 5 + 2 + 4 * D
    for n in range(1, D + 1):
        for i in range(n, -1, -1):
            for j in range(n - i, -1, -1):
                m = (i, j, n - i - j)
                k1 = sum(1 for c in m if c >= 1)
                k2 = sum(1 for c in m if c >= 2)
                fl += 2 * k1 - 1 + 1 + ((k2 - 1) + 2 if k2 else 0) + 6
    return fl


def algorithmic_flops(st, nm):
    """Method flop count of one evaluation: 26 per Gauss point, ray tracing
    9 per pair + 7 per line (the precheck) + 156 per line that hits."""
    g1, g4, g11, rt = st["pairs_by_rule"]
    return (FLOPS_PER_POINT * (g1 + 4 * g4 + 11 * g11) + rt * (9.0 + 7.0 * nm) + 156.0 * st["rt_hit_lines"])


WORKLOAD_TEXT = {
    "C1": "Gaussian swirl, [-1,1]^3, 10^3 Kuhn cells",
    "C2": "vortex ring, [-1.5,1.5]^2 x [-0.5,0.5], 64x64x22 Kuhn cells",
    "C3": "random Fourier curl field, [-1,1]^3, 48^3 Kuhn cells",
    "C5": "two coaxial rings, [-1.5,1.5]^3, 80^3 Kuhn cells",
}


def measured_traffic(kernel, workload, policy, precision):
    """HBM bytes per launch of `kernel` from the committed counter summary
    of this workload and policy, or None when the kernel source has changed
    since the counters were taken (the summary records the sha256 of that
    source) or the run is not a profiled configuration."""
    import hashlib

    if precision != 1:
        return None
    path = os.path.join(ROOT, "profiles", f"bs_eval_velocity_{workload}_hbm_traffic.md")
    src = os.path.join(ROOT, "paper_0712_1695_amd", "csrc",
                       "bs_tree.hip" if kernel.startswith("k_tree") else "bs_kernels.hip")
    try:
        lines = open(path).read().split("\n")
        sha = hashlib.sha256(open(src, "rb").read()).hexdigest()
    except OSError:
        return None
    for ln in lines:
        f = ln.split()
        if len(f) == 5 and f[0] == "traffic" and f[1] == policy and f[2] == kernel and f[4] == sha:
            return float(f[3])
    return None


def copy_calibration(mib):
    """A plain device-to-device copy of a known size, so that the HBM byte
    counters of a profiler can be scaled: it reads and writes mib MiB."""
    import torch

    n = mib * (1 << 20) // 4
    src = torch.ones(n, dtype=torch.float32, device="cuda")
    dst = torch.empty_like(src)
    torch.cuda.synchronize()
    dst.copy_(src)
    torch.cuda.synchronize()
    print(json.dumps({"copy_bytes_read": n * 4, "copy_bytes_written": n * 4}), flush=True)


def cpu_baseline(mesh, target_seconds=15.0):
    import oracle

    pol = oracle.make_policy("fixed")
    rng = np.random.default_rng(123)
    k = 8
    while True:
        tg = rng.choice(mesh.n_nodes, size=k, replace=False)
        t0 = time.perf_counter()
        oracle.evaluate(mesh.xyz, mesh.omega, mesh.tets, pol, targets=tg)
        dt = time.perf_counter() - t0
        if dt >= target_seconds / 2 or k >= mesh.n_nodes // 2:
            break
        k = min(mesh.n_nodes // 2, int(k * max(2.0, target_seconds / max(dt, 1e-3))))
    pairs = k * mesh.n_tets
    return {"value": pairs / dt, "unit": "pairs/s", "cores": oracle.num_threads(), "kind": "oracle",
            "sample": f"{k} random nodes x all {mesh.n_tets} tets of the same workload (FP64, fixed rule), "
                      f"{dt:.1f} s"}


def load_probes(workload):
    """Probe nodes and their exact velocities (stored reference), or None."""
    path = os.path.join(ROOT, "tests", "golden", f"probe_exact_{workload}.json")
    if not os.path.exists(path):
        return None
    doc = json.load(open(path))
    return np.array(doc["nodes"], dtype=np.int64), np.array(doc["velocity"], dtype=np.float64)


class Bench:
    """One uploaded workload with helpers that time evaluations on it."""

    def __init__(self, bs, torch, mesh, precision):
        self.bs, self.torch, self.mesh, self.precision = bs, torch, mesh, precision
        dev = torch.device("cuda", 0)
        self.h = bs.bs_mesh_upload(torch.tensor(mesh.xyz, device=dev), torch.tensor(mesh.omega, device=dev),
                                   torch.tensor(mesh.tets, device=dev))
        self.out = torch.empty((mesh.n_nodes, 3), dtype=torch.float64, device=dev)
        self.pairs = mesh.n_nodes * mesh.n_tets
        self.probes = None

    def set_policy(self, **kw):
        self.bs.bs_set_policy(self.h, precision=self.precision, **kw)

    def time(self, steps, warmup, **flags):
        """Wall time per evaluation over `steps` after `warmup` (seconds)."""
        bs, torch = self.bs, self.torch
        for _ in range(warmup):
            bs.bs_eval_velocity(self.h, out=self.out, **flags)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(steps):
            bs.bs_eval_velocity(self.h, out=self.out, **flags)
        torch.cuda.synchronize()
        return (time.perf_counter() - t0) / max(steps, 1)

    def kernels(self, steps, **flags):
        """Mean per-kernel seconds [far, band, ray tracing, sum] with every
        kernel on one stream, the stats of the last pass and its wall time
        per evaluation."""
        bs, torch = self.bs, self.torch
        kern = np.zeros(4)
        st = None
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(max(steps, 1)):
            _, st = bs.bs_eval_velocity(self.h, out=self.out, stats=True, serial=True, **flags)
            kern += np.array(st["t_kernel_s"])
        torch.cuda.synchronize()
        return kern / max(steps, 1), st, (time.perf_counter() - t0) / max(steps, 1)

    def stats(self, **flags):
        return self.bs.bs_eval_velocity(self.h, out=self.out, stats=True, **flags)[1]

    def error(self):
        """rel-L2 error of the last evaluation at the probe nodes."""
        if self.probes is None:
            return None
        nodes, exact = self.probes
        v = self.out[self.torch.as_tensor(nodes, device=self.out.device)].cpu().numpy()
        return float(np.linalg.norm(v - exact) / np.linalg.norm(exact))

    def free(self):
        self.bs.bs_mesh_free(self.h)


def roof_entry(name, what, bound, kflops, t, workload, policy, precision, extra=None):
    r = {"kernel": f"{name} ({what})", "bound": bound, "achieved": kflops / t / 1e12,
         "peak": FP32_PEAK_TFLOPS, "unit": "TFLOP/s", "frac": kflops / t / 1e12 / FP32_PEAK_TFLOPS,
         "traffic": measured_traffic(name, workload, policy, precision),
         "traffic_unit": "bytes per launch (rocprofv3 FETCH_SIZE + WRITE_SIZE, copy-calibrated)",
         "avg_duration_ms": t * 1e3,
         "measured": "kernel alone: the serial pass (every kernel on one stream), HIP events on its stream"}
    if extra:
        r.update(extra)
    return r


def kernel_rooflines(st, kern, nm, workload, policy, precision, valu_far=False):
    g1, g4, g11, rtp = st["pairs_by_rule"]
    far_name = "k_gauss_all" if (valu_far or precision == 2) else "k_far_split"
    band_name = "k_band" if far_name == "k_gauss_all" else "k_band_piece"
    rt_what = ("learned selection pass and ray tracing by walking face neighbours; the method's flops of "
               "the ray-traced pairs" if policy == "learned"
               else "ray tracing by walking face neighbours; the method's flops of its pairs")
    rt_name = "k_select+k_rt_walk" if policy == "learned" else "k_rt_walk"
    return [
        roof_entry(far_name, "far field, 1-point rule on every pair, vector ALUs" if far_name == "k_gauss_all"
                   else "far field, the G1 pairs, matrix-core contractions on 16-bit pieces, binary32 accuracy",
                   "alu" if far_name == "k_gauss_all" else "mfma", FLOPS_PER_POINT * g1, kern[0],
                   workload, policy, precision),
        roof_entry(band_name, "the G4 and G11 pairs, vector ALUs", "alu", FLOPS_PER_POINT * (4 * g4 + 11 * g11),
                   kern[1], workload, policy, precision),
        roof_entry(rt_name, rt_what, "alu", rtp * (9.0 + 7.0 * nm) + 156.0 * st["rt_hit_lines"], kern[2],
                   workload, policy, precision, extra=walk_executed(st, kern[2])),
    ]


def walk_executed(st, t):
    """The ray-tracing flops the walk executes beside those the method's
    count credits: it never runs the per-line precheck (7 flops per line and
    pair), only the pair set-up and the chords of the lines that hit."""
    kflops = 9.0 * st["pairs_by_rule"][3] + 156.0 * st["rt_hit_lines"]
    return {"executed_tflop": kflops / 1e12, "executed_achieved": kflops / t / 1e12,
            "executed_frac": kflops / t / 1e12 / FP32_PEAK_TFLOPS,
            "executed_what": "9 per ray-traced pair + 156 per (line, tet) hit: the precheck term the walk skips "
                             "is left out"}


def load_heun_reference(workload):
    """The FP64 oracle's Heun step 1 of the workload at sampled nodes, if one
    is stored (written by tests/golden/make_c5_heun_reference.py)."""
    path = os.path.join(ROOT, "tests", "golden", "c5_heun_step1.json")
    if workload != "C5" or not os.path.exists(path):
        return None
    with open(path) as f:
        ref = json.load(f)
    ref["nodes"] = np.asarray(ref["nodes"], dtype=np.int64)
    ref["x1"] = np.asarray(ref["x1"])
    return ref


def heun_drift(pos, ref, mesh):
    """Largest position error at the reference's nodes after one step."""
    nodes = ref["nodes"]
    err = float(np.abs(pos[nodes] - ref["x1"]).max())
    step = float(np.abs(ref["x1"] - mesh.xyz[nodes]).max())
    return {"max_abs": err, "max_rel_to_step": err / step}


def tree_roofline(st, kern, order, workload, policy, precision):
    """The treecode far field (moments, expansions and direct leaves
    together, one duration): 26 flops per 1-point pair of the direct leaves,
    expansion_flops per expansion term."""
    direct_g1 = st["pairs_by_rule"][0] - st["tree_covered"]
    kflops = FLOPS_PER_POINT * direct_g1 + expansion_flops(order) * st["tree_expansions"]
    return roof_entry("k_tree_direct+k_tree_m2p", "treecode far field: direct leaves and expansions, vector ALUs, "
                      "with the moment passes", "alu", kflops, kern[0], workload, "treecode-" + policy, precision)


def train_selector(W):
    """The learned policy's network, trained on the GPU (outside any timed
    region) on 10 million pairs of the swirl box and the ring box, and
    evaluated on pairs of the held-out Fourier-curl box."""
    from paper_0712_1695_amd import selector

    return selector.train_selector(W.make_config)


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=5)
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--workload", default="C5")
    ap.add_argument("--policy", default="learned", choices=["learned", "fixed"],
                    help="policy of the headline step")
    ap.add_argument("--precision", type=int, default=1)
    ap.add_argument("--quick", action="store_true",
                    help="the headline steps and their per-kernel pass only (profiling runs)")
    ap.add_argument("--serial", action="store_true", help="time the headline steps with every kernel on one stream")
    ap.add_argument("--valu-far", action="store_true",
                    help="headline far field on the vector ALUs instead of the matrix cores")
    ap.add_argument("--far", default="all_pairs", choices=["all_pairs", "treecode"],
                    help="far field of the headline step (treecode: the profiling runs of the treecode kernels)")
    ap.add_argument("--heun-steps", type=int, default=10, help="Heun steps of the Lagrangian leg (0: skip)")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--copy-calibration", type=int, default=0, metavar="MIB",
                    help="only run a plain copy of MIB MiB (profiler byte-counter calibration)")
    args = ap.parse_args()
    if args.gpus != 1:
        print(f"bench.py runs on one GPU only (--gpus {args.gpus} requested); multi-GPU sharding is not built",
              file=sys.stderr)
        sys.exit(2)

    if args.copy_calibration:
        copy_calibration(args.copy_calibration)
        return

    import torch

    import paper_0712_1695_amd as bs
    import workloads as W

    torch.cuda.set_device(0)
    nm = 16 * 16
    t_start = time.perf_counter()
    blob, sel_info = train_selector(W) if (args.policy == "learned" or not args.quick) else (None, None)
    learned_pol = dict(kind=bs.BS_POLICY_LEARNED, n_phi=16, n_theta=16, mlp_bf16=blob, conf_min=0.9)
    fixed_pol = dict(kind=bs.BS_POLICY_FIXED, n_phi=16, n_theta=16)
    head_pol = dict(learned_pol if args.policy == "learned" else fixed_pol)
    tree_kw = dict(far_field=bs.BS_FAR_TREECODE, tree_theta=TREE_THETA, tree_order=TREE_ORDER)
    if args.far == "treecode":
        head_pol.update(tree_kw)
    flags = dict(valu_far=args.valu_far)

    mesh = W.make_config(args.workload)
    B = Bench(bs, torch, mesh, args.precision)
    B.probes = load_probes(args.workload)
    print(f"bench: {args.workload} {mesh.n_nodes} nodes x {mesh.n_tets} tets, {args.policy} policy", flush=True)

    # ---- the timed steps (the headline)
    B.set_policy(**head_pol)
    t_head = B.time(args.steps, args.warmup, serial=args.serial, **flags)
    err_head = B.error()
    st_head = B.stats(**flags)
    kern, st_k, t_serial = B.kernels(args.steps, **flags)
    value = B.pairs / t_head
    print(f"bench: headline {t_head * 1e3:.2f} ms per evaluation", flush=True)

    flops = algorithmic_flops(st_head, nm)
    kernels = kernel_rooflines(st_head, kern, nm, args.workload, args.policy, args.precision, args.valu_far)
    if args.far == "treecode":
        kernels[0] = tree_roofline(st_head, kern, TREE_ORDER, args.workload, args.policy, args.precision)
    roof = dict(max(kernels, key=lambda r: r["avg_duration_ms"]))
    cuts = "RT < 2 hbar, G11 < 4, G4 < 8, else G1"
    line = {
        "metric": "node-tet pair evals/s (+ % FP32 peak)",
        "value": value,
        "unit": "pairs/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": t_head * 1e3,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32",
        "data": "synthetic",
        "config": {
            "workload": f"{args.workload}: {WORKLOAD_TEXT.get(args.workload, mesh.name)}, {mesh.n_nodes} nodes x "
                        f"{mesh.n_tets} tets, {args.policy} policy "
                        f"({'selector on the pairs the fixed rule ray-traces, ' if args.policy == 'learned' else ''}"
                        f"{cuts}), 16x16 lines, "
                        f"{'treecode far field (theta %.1f, order %d), ' % (TREE_THETA, TREE_ORDER) if args.far == 'treecode' else ''}"
                        f"{['fp32 naive', 'fp32 compensated', 'fp64 accumulation'][args.precision]}",
            "pairs_per_step": B.pairs,
            "pairs_by_rule": st_head["pairs_by_rule"],
            "rt_hit_lines": st_head["rt_hit_lines"],
            "algorithmic_tflop_per_step": flops / 1e12,
            "path_fp32_peak_frac": flops / t_head / 1e12 / FP32_PEAK_TFLOPS,
            "ms_per_step_serial": t_serial * 1e3,
            "kernel_ms_serial": {"far": kern[0] * 1e3, "band": kern[1] * 1e3, "rt": kern[2] * 1e3,
                                 "sum": kern[3] * 1e3},
            "probe_error": err_head,
        },
        "roofline": roof,
        "roofline_kernels": kernels,
    }
    if sel_info is not None:
        line["config"]["selector"] = sel_info

    # ---- the fixed rule on the same mesh
    steps2 = max(2, args.steps // 2 + 1)
    if args.policy == "learned" and not args.quick:
        B.set_policy(**fixed_pol)
        t_fix = B.time(args.steps, args.warmup, **flags)
        err_fix = B.error()
        st_fix = B.stats(**flags)
        kf, _, _ = B.kernels(steps2, **flags)
        line["fixed"] = {"ms_per_step": t_fix * 1e3, "value": B.pairs / t_fix, "probe_error": err_fix,
                         "pairs_by_rule": st_fix["pairs_by_rule"], "rt_hit_lines": st_fix["rt_hit_lines"],
                         "kernel_ms_serial": {"far": kf[0] * 1e3, "band": kf[1] * 1e3, "rt": kf[2] * 1e3},
                         "learned_vs_fixed_speed": t_fix / t_head,
                         "roofline_kernels": kernel_rooflines(st_fix, kf, nm, args.workload, "fixed",
                                                              args.precision, args.valu_far)}
        print(f"bench: fixed {t_fix * 1e3:.2f} ms", flush=True)

    if not args.quick:
        # ---- equal accuracy: a ladder of fixed settings against the learned policy
        if args.policy == "learned" and B.probes is not None:
            ladder = [{"near_cut": DEFAULT_CUTS[0], "d_g11": DEFAULT_CUTS[1], "d_g4": DEFAULT_CUTS[2], "lines": 16,
                       "ms_per_step": t_fix * 1e3, "probe_error": err_fix}]
            for a, b, c, nl in LADDER:
                B.set_policy(kind=bs.BS_POLICY_FIXED, near_cut=a, d_g11=b, d_g4=c, n_phi=nl, n_theta=nl)
                t = B.time(steps2, 1, **flags)
                ladder.append({"near_cut": a, "d_g11": b, "d_g4": c, "lines": nl, "ms_per_step": t * 1e3,
                               "probe_error": B.error()})
                print(f"bench: fixed {a}/{b}/{c} {nl}x{nl}: {t * 1e3:.2f} ms, error {ladder[-1]['probe_error']:.3e}",
                      flush=True)
            ok = [r for r in ladder if r["probe_error"] <= err_head]
            best = min(ok, key=lambda r: r["ms_per_step"]) if ok else min(ladder, key=lambda r: r["probe_error"])
            line["accuracy"] = {
                "reference": f"exact velocity at {len(B.probes[0])} probe nodes (tests/golden/probe_exact_"
                             f"{args.workload}.json: cone decomposition within 4 hbar, 11-point rule beyond)",
                "learned": {"ms_per_step": t_head * 1e3, "probe_error": err_head},
                "fixed_ladder": ladder,
                "equal_accuracy_fixed": best,
                "fixed_reaches_learned_error": bool(ok),
                "vs_fixed_equal_accuracy": best["ms_per_step"] / (t_head * 1e3),
            }

        # ---- the treecode far field with both policies
        if args.policy == "learned" and args.far == "all_pairs":
            tree = {"theta": TREE_THETA, "order": TREE_ORDER,
                    "what": "BS_FAR_TREECODE: the 1-point pairs by a batched Barnes-Hut treecode (clusters of the "
                            "k-d tree of the centroids, Cartesian expansions, 64-node target blocks), every other "
                            "pair as in the all-pairs evaluation"}
            for name, pol, t_ref in (("fixed", fixed_pol, t_fix), ("learned", learned_pol, t_head)):
                t0 = time.perf_counter()
                B.set_policy(**pol, **tree_kw)
                t_plan = time.perf_counter() - t0
                t = B.time(steps2, 1)
                err = B.error()
                kt, st_t, _ = B.kernels(steps2)
                tree[name] = {"ms_per_step": t * 1e3, "probe_error": err, "vs_all_pairs_speed": t_ref / t,
                              "plan_s": t_plan, "tree_expansions": st_t["tree_expansions"],
                              "tree_direct": st_t["tree_direct"], "tree_covered": st_t["tree_covered"],
                              "kernel_ms_serial": {"far": kt[0] * 1e3, "band": kt[1] * 1e3, "rt": kt[2] * 1e3},
                              "roofline_far": tree_roofline(st_t, kt, TREE_ORDER, args.workload, name,
                                                            args.precision)}
                print(f"bench: treecode {name} {t * 1e3:.2f} ms (error {err:.3e}, {t_ref / t:.2f}x all pairs)",
                      flush=True)
            # the setting whose result is the all-pairs sum within 1e-6:
            # its deviation from this mesh's all-pairs evaluation, every node
            B.set_policy(**fixed_pol)
            B.time(1, 0)
            v_all = B.out.cpu().numpy()
            B.set_policy(**fixed_pol, far_field=bs.BS_FAR_TREECODE, tree_theta=TREE_EQUIV[0],
                         tree_order=TREE_EQUIV[1])
            t = B.time(steps2, 1)
            v_t = B.out.cpu().numpy()
            dev = float(np.linalg.norm(v_t - v_all) / np.linalg.norm(v_all))
            worst = float(np.linalg.norm(v_t - v_all, axis=1).max() / np.linalg.norm(v_all, axis=1).max())
            tree["all_pairs_equivalent"] = {
                "theta": TREE_EQUIV[0], "order": TREE_EQUIV[1], "policy": "fixed", "ms_per_step": t * 1e3,
                "vs_all_pairs_speed": t_fix / t, "rel_l2_vs_all_pairs": dev, "worst_node_vs_max_speed": worst,
                "probe_error": B.error(), "all_pairs_result_rate": B.pairs / t,
                "all_pairs_result_rate_what": "n x T node-tet pairs of the all-pairs result delivered per second "
                                              "(the far 1-point pairs are summed by expansions, not pair by pair)",
                "what": "the treecode at a setting whose velocities equal the all-pairs evaluation's within 1e-6 "
                        "(rel-L2 over every node, and the largest node error over the largest speed)"}
            print(f"bench: treecode at theta {TREE_EQUIV[0]}, order {TREE_EQUIV[1]}: {t * 1e3:.2f} ms "
                  f"({t_fix / t:.2f}x all pairs), rel-L2 {dev:.2e} from the all-pairs velocities", flush=True)
            ok = [r for r in line["accuracy"]["fixed_ladder"] if r["probe_error"] <= tree["learned"]["probe_error"]] \
                if "accuracy" in line else []
            if ok:
                best = min(ok, key=lambda r: r["ms_per_step"])
                tree["learned_vs_fixed_all_pairs_equal_accuracy"] = best["ms_per_step"] / tree["learned"]["ms_per_step"]
            line["treecode"] = tree

        # ---- the far field on the vector ALUs (the design without matrix cores)
        B.set_policy(**fixed_pol)
        t_valu = B.time(steps2, 1, valu_far=True)
        err_valu = B.error()
        kv, st_v, _ = B.kernels(steps2, valu_far=True)
        line["valu_far"] = {"ms_per_step": t_valu * 1e3, "value": B.pairs / t_valu, "probe_error": err_valu,
                            "policy": "fixed",
                            "roofline_kernels": kernel_rooflines(st_v, kv, nm, args.workload, "fixed",
                                                                 args.precision, valu_far=True)}
        print(f"bench: vector-ALU far field {t_valu * 1e3:.2f} ms", flush=True)

        # ---- the Lagrangian run (moves this mesh: last on it)
        if args.heun_steps > 0:
            drift = None
            ref = load_heun_reference(args.workload)
            if ref is not None:
                # step 1 with the fixed rule against the FP64 oracle's own
                # step, then back to the initial positions
                B.set_policy(**fixed_pol)
                pos, _ = bs.bs_advect_heun(B.h, ref["dt"], 1)
                drift = {"fixed": heun_drift(pos, ref, mesh)}
                bs.bs_mesh_update(B.h, xyz=mesh.xyz)
            B.set_policy(**head_pol)
            pos, secs1 = bs.bs_advect_heun(B.h, 0.005, 1)
            if ref is not None:
                drift[args.policy + "_policy"] = heun_drift(pos, ref, mesh)
            secs = list(secs1)
            if args.heun_steps > 1:
                secs += list(bs.bs_advect_heun(B.h, 0.005, args.heun_steps - 1)[1])
            line["lagrangian"] = {"steps": args.heun_steps, "dt": 0.005, "policy": args.policy,
                                  "seconds_per_step": [float(s) for s in secs],
                                  "median_s_per_step": float(np.median(secs)),
                                  "evaluations_per_step": 2,
                                  "what": "bs_advect_heun: per step two device-mesh rebuilds on the host and two "
                                          "evaluations, connectivity and nodal vorticity kept"}
            if drift is not None:
                drift["what"] = ("positions after step 1 at %d sampled nodes against the same Heun step taken by "
                                 "the FP64 oracle with the fixed rule (tests/golden/c5_heun_step1.json): largest "
                                 "error, absolute and over the largest displacement of the step; the learned "
                                 "policy's figure also holds the rule changes the selector makes" % len(ref["nodes"]))
                line["lagrangian"]["step1_vs_oracle"] = drift
                print(f"bench: Heun step 1 against the oracle: fixed {drift['fixed']['max_rel_to_step']:.3e}, "
                      f"{args.policy} {drift[args.policy + '_policy']['max_rel_to_step']:.3e} of the step", flush=True)
            print(f"bench: Heun {np.median(secs):.3f} s per step", flush=True)
            if args.policy == "learned" and args.far == "all_pairs":
                # three steps from the initial positions with the treecode far
                # field (continuing the run, the ring cores' shear inverts
                # tetrahedra a few steps later: a Lagrangian mesh needs
                # re-meshing by then)
                bs.bs_mesh_update(B.h, xyz=mesh.xyz)
                B.set_policy(**head_pol, **tree_kw)
                _, secs_t = bs.bs_advect_heun(B.h, 0.005, 3)
                line["lagrangian"]["treecode"] = {
                    "steps": 3, "seconds_per_step": [float(s) for s in secs_t],
                    "median_s_per_step": float(np.median(secs_t)),
                    "what": "the same run from the initial positions with the treecode far field (theta %.1f, "
                            "order %d): per step two rebuilds of the device mesh and of the treecode plan on the "
                            "host, two evaluations" % (TREE_THETA, TREE_ORDER)}
                print(f"bench: Heun with the treecode {np.median(secs_t):.3f} s per step", flush=True)
    B.free()

    if not args.quick:
        # ---- the vortex ring (in the selector's training distribution) and
        # the Fourier-curl box (held out from it) as further legs
        for wl in ("C2", "C3"):
            if wl == args.workload:
                continue
            m2 = W.make_config(wl)
            B2 = Bench(bs, torch, m2, args.precision)
            B2.probes = load_probes(wl)
            leg = {"workload": f"{wl}: {WORKLOAD_TEXT[wl]}, {m2.n_nodes} nodes x {m2.n_tets} tets"}
            for name, pol in (("fixed", fixed_pol), ("learned", learned_pol),
                              ("learned_treecode", dict(learned_pol, **tree_kw))):
                B2.set_policy(**pol)
                t = B2.time(args.steps * 2, args.warmup, **flags)
                leg[name] = {"ms_per_step": t * 1e3, "value": B2.pairs / t, "probe_error": B2.error()}
            B2.free()
            line[wl.lower()] = leg
            print(f"bench: {wl} fixed {leg['fixed']['ms_per_step']:.2f} ms (error {leg['fixed']['probe_error']:.3e}), "
                  f"learned {leg['learned']['ms_per_step']:.2f} ms (error {leg['learned']['probe_error']:.3e}), "
                  f"learned + treecode {leg['learned_treecode']['ms_per_step']:.2f} ms "
                  f"(error {leg['learned_treecode']['probe_error']:.3e})", flush=True)

    if not args.no_cpu_baseline and not args.quick:
        line["cpu_baseline"] = cpu_baseline(mesh)
    line["config"]["bench_wall_s"] = time.perf_counter() - t_start
    print(json.dumps(line), flush=True)


if __name__ == "__main__":
    main()
