"""The work this library is used for, as cases that can be timed and compared.

A case is a dict of plain values.  kind says which entry points it takes:

  eval       bs_eval_velocity (or, with noalloc, bs_eval_velocity_noalloc) of
             the nodes of a mesh that is uploaded and has its policy set: what
             every step of a vortex computation repeats
  points     bs_eval_points at points that are not nodes
  stage      one stage of a Lagrangian run: bs_mesh_update with moved nodes
             and new vorticity, then bs_eval_velocity on the moved mesh, whose
             boundary is then no longer convex
  gradient   bs_velocity_gradient and bs_stretching_rate of given velocities
  selector   a step of the rule selector's training: labels and features of
             sampled pairs, then the network's forward and backward pass

The meshes are the seeded Kuhn-split boxes (and the ball) of the library's
workloads at several sizes: the swirl in a cube, a Gaussian-core ring, a
random Fourier field, two coaxial rings, Hill's vortex in a ball.  Positions
are jittered and amplitudes drawn from the seed.

The pair sums are formed in binary32 and only their last sum is FP64, so the
velocities are handed on in the type they are computed in (torch.float32);
velocity gradients and stretching rates are FP64 throughout and stay FP64.
"""
import itertools
import json
import math
import os

import numpy as np
import torch

import paper_0712_1695_amd as bs

HERE = os.path.dirname(os.path.abspath(__file__))
# the selector network the tests use (trained from the oracle's labels)
NETWORK = os.path.join(HERE, "..", "tests", "golden", "selector_blob.json")

BOXES = {
    "swirl": ((-1.0, -1.0, -1.0), (1.0, 1.0, 1.0), 0.10),
    "ring": ((-1.5, -1.5, -0.5), (1.5, 1.5, 0.5), 0.15),
    "fourier": ((-1.0, -1.0, -1.0), (1.0, 1.0, 1.0), 0.20),
    "rings": ((-1.5, -1.5, -1.5), (1.5, 1.5, 1.5), 0.20),
    "ball": ((-1.0, -1.0, -1.0), (1.0, 1.0, 1.0), 0.10),
}
CUTS = (2.0, 4.0, 8.0)  # the default cut distances, in mean edge lengths


def listed():
    return [
        # the smallest call in use (the 10^3 box of the selector's training
        # and of most tests), where launches and latency are what counts
        dict(name="swirl_10", kind="eval", box="swirl", cx=10, cy=10, cz=10, policy="fixed"),
        # the same range through the entry point for serving loops and graph
        # capture, on a ragged box
        dict(name="swirl_ragged_noalloc", kind="eval", box="swirl", cx=13, cy=9, cz=11, policy="learned", noalloc=True),
        # the single-ring workload with the default policy
        dict(name="ring_64", kind="eval", box="ring", cx=64, cy=64, cz=22, policy="fixed"),
        # the random field (no empty regions) with the learned rule selector
        dict(name="fourier_48_learned", kind="eval", box="fourier", cx=48, cy=48, cz=48, policy="learned"),
        # the largest: the two-ring workload of the library's benchmark
        dict(name="rings_80_learned", kind="eval", box="rings", cx=80, cy=80, cz=80, policy="learned"),
        # the same workload with the treecode far field at its defaults, as
        # the long Lagrangian runs take it
        dict(name="rings_80_tree", kind="eval", box="rings", cx=80, cy=80, cz=80, policy="fixed", theta=0.3, order=4),
        # the treecode where it equals the all-pairs sum, with the selector
        dict(name="ring_64_tree_tight", kind="eval", box="ring", cx=64, cy=64, cz=22, policy="learned", theta=0.2,
             order=6),
        # the paper's own method, every pair ray traced (convergence studies)
        dict(name="ball_20_pure_rt", kind="eval", box="ball", cx=20, cy=20, cz=20, policy="pure_rt", lines=24),
        # velocities at points in and around the mesh (probes, tracers)
        dict(name="ring_40_points", kind="points", box="ring", cx=40, cy=40, cz=14, policy="fixed", points=20011),
        # a Lagrangian stage on a moved mesh
        dict(name="rings_33_stage", kind="stage", box="rings", cx=33, cy=31, cz=35, policy="fixed"),
        # the vortex-stretching term of a step of the large run
        dict(name="rings_64_stretch", kind="gradient", box="rings", cx=64, cy=64, cz=64),
        # a training step of the rule selector
        dict(name="selector_65536", kind="selector", box="swirl", cx=10, cy=10, cz=10, rows=65536),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _box(rng, box, lo, hi):
    """Cell counts of a box with about lo^3 .. hi^3 cells, roughly cubic cells, ragged."""
    a, b, _ = BOXES[box]
    side = _log_int(rng, lo, hi)
    ext = [b[k] - a[k] for k in range(3)]
    h = (ext[0] * ext[1] * ext[2]) ** (1 / 3) / side
    return dict(box=box, **{"c" + "xyz"[k]: max(3, round(ext[k] / h) + rng.randrange(-1, 2)) for k in range(3)})


def draw(rng):
    kind = rng.choice(("eval", "eval", "eval", "eval", "small", "small", "pure_rt", "points", "stage", "gradient",
                       "selector"))
    if kind == "eval":
        c = dict(kind="eval", **_box(rng, rng.choice(("ring", "fourier", "rings")), 16, 72),
                 policy=rng.choice(("fixed", "learned")))
        if rng.random() < 0.5:
            c.update(theta=rng.choice((0.2, 0.3, 0.5)), order=rng.choice((4, 6)))
        return c
    if kind == "small":
        return dict(kind="eval", **_box(rng, "swirl", 4, 15), policy=rng.choice(("fixed", "learned")),
                    noalloc=rng.random() < 0.5)
    if kind == "pure_rt":
        return dict(kind="eval", **_box(rng, rng.choice(("ball", "fourier")), 6, 22), policy="pure_rt",
                    lines=rng.choice((4, 16, 24)))
    if kind == "points":
        return dict(kind="points", **_box(rng, rng.choice(("ring", "fourier")), 8, 40), policy="fixed",
                    points=_log_int(rng, 10, 40000))
    if kind == "stage":
        c = dict(kind="stage", **_box(rng, rng.choice(("ring", "rings")), 10, 40), policy="fixed")
        if rng.random() < 0.5:
            c.update(theta=0.3, order=4)
        return c
    if kind == "gradient":
        return dict(kind="gradient", **_box(rng, rng.choice(("fourier", "rings")), 6, 72))
    return dict(kind="selector", **_box(rng, "swirl", 8, 16), rows=_log_int(rng, 512, 200000))


# ------------------------------------------------------------------- inputs

def _mesh(case, seed):
    """Node positions, vorticity (FP64) and tetrahedra (int32) on the GPU."""
    dev = torch.device("cuda")
    g = torch.Generator(device=dev).manual_seed(int(seed))
    lo, hi, alpha = BOXES[case["box"]]
    c = (case["cx"], case["cy"], case["cz"])
    lo_t = torch.tensor(lo, dtype=torch.float64, device=dev)
    h = (torch.tensor(hi, dtype=torch.float64, device=dev) - lo_t) / torch.tensor(c, dtype=torch.float64, device=dev)
    k, j, i = torch.meshgrid(*(torch.arange(c[q] + 1, device=dev) for q in (2, 1, 0)), indexing="ij")
    idx = torch.stack([i, j, k], dim=-1).reshape(-1, 3)
    inside = ((idx > 0) & (idx < torch.tensor(c, device=dev))).all(dim=1)
    u = torch.rand(idx.shape, dtype=torch.float64, device=dev, generator=g) * 2 - 1
    x = lo_t + idx * h + torch.where(inside[:, None], u * alpha * h, torch.zeros_like(u))
    x = torch.where(idx == torch.tensor(c, device=dev), torch.tensor(hi, dtype=torch.float64, device=dev).expand_as(x), x)
    # six tets per cell around its main diagonal, positively oriented
    k, j, i = torch.meshgrid(*(torch.arange(c[q], device=dev) for q in (2, 1, 0)), indexing="ij")
    base = (i + (c[0] + 1) * (j + (c[1] + 1) * k)).reshape(-1)
    step = (1, c[0] + 1, (c[0] + 1) * (c[1] + 1))
    tets = []
    for perm in itertools.permutations(range(3)):
        v = [base]
        for ax in perm:
            v.append(v[-1] + step[ax])
        if perm in ((0, 2, 1), (1, 0, 2), (2, 1, 0)):
            v[2], v[3] = v[3], v[2]
        tets.append(torch.stack(v, dim=1))
    tets = torch.stack(tets, dim=1).reshape(-1, 4)
    if case["box"] == "ball":  # the smooth map of the cube onto the ball
        q = x * x
        x = x * torch.stack([torch.sqrt(1 - q[:, a] / 2 - q[:, b] / 2 + q[:, a] * q[:, b] / 3)
                             for a, b in ((1, 2), (2, 0), (0, 1))], dim=1)
    amp = 0.75 + 0.5 * torch.rand(8, dtype=torch.float64, device=dev, generator=g)
    return x.contiguous(), _vorticity(case["box"], x, amp, g).contiguous(), tets.to(torch.int32).contiguous()


def _ring(x, radius, sigma, z0):
    z = x[:, 2] - z0
    rc = torch.hypot(x[:, 0], x[:, 1])
    mag = torch.exp(-((rc - radius) ** 2 + z * z) / sigma ** 2) / (math.pi * sigma ** 2) / rc.clamp_min(1e-300)
    return torch.stack([-x[:, 1] * mag, x[:, 0] * mag, torch.zeros_like(mag)], dim=1)


def _vorticity(box, x, amp, g):
    if box == "swirl":
        e = amp[0] * torch.exp(-(x * x).sum(dim=1) / 0.25)
        return torch.stack([-x[:, 1] * e, x[:, 0] * e, torch.zeros_like(e)], dim=1)
    if box == "ring":
        return amp[0] * _ring(x, 1.0, 0.1, 0.0)
    if box == "rings":
        return amp[0] * _ring(x, 1.0, 0.08, -0.25) + amp[1] * _ring(x, 0.8, 0.08, 0.25)
    if box == "ball":
        return amp[0] * torch.stack([-x[:, 1], x[:, 0], torch.zeros_like(x[:, 0])], dim=1)
    om = torch.zeros_like(x)
    for m in range(8):
        n = torch.randint(-3, 4, (3,), device=x.device, generator=g)
        kap = math.pi * torch.where(n.abs().sum() > 0, n, torch.ones_like(n)).to(torch.float64)
        a = amp[m] * torch.randn(3, dtype=torch.float64, device=x.device, generator=g) / kap.norm()
        ph = 2 * math.pi * torch.rand((), dtype=torch.float64, device=x.device, generator=g)
        om += -torch.sin(x @ kap + ph)[:, None] * torch.linalg.cross(kap, a)[None, :]
    return om / om.norm(dim=1).max()


def _moved(x, seed):
    """The nodes a little later: a smooth displacement that also bends the box's faces."""
    g = torch.Generator(device=x.device).manual_seed(int(seed) + 77)
    ph = 2 * math.pi * torch.rand(3, dtype=torch.float64, device=x.device, generator=g)
    return (x + 0.01 * torch.sin(2.0 * x.roll(1, dims=1) + ph) * torch.cos(1.5 * x.roll(2, dims=1))).contiguous()


def _points(case, seed, device):
    g = torch.Generator(device=device).manual_seed(int(seed) + 13)
    lo, hi, _ = BOXES[case["box"]]
    lo, hi = (torch.tensor(v, dtype=torch.float64, device=device) for v in (lo, hi))
    u = torch.rand((case["points"], 3), dtype=torch.float64, device=device, generator=g)
    return ((lo + hi) / 2 + (u - 0.5) * 1.1 * (hi - lo)).contiguous()  # some outside the mesh


def _lines(case):
    return case.get("lines", 16)


def _set_policy(h, case):
    kw = dict(n_phi=_lines(case), n_theta=_lines(case))
    kw["kind"] = {"fixed": bs.BS_POLICY_FIXED, "learned": bs.BS_POLICY_LEARNED, "pure_rt": bs.BS_POLICY_PURE_RT}[
        case["policy"]]
    if case["policy"] == "learned":
        with open(NETWORK) as f:
            net = json.load(f)
        kw.update(mlp_bf16=np.array(net["blob_bf16_bits"], dtype=np.uint16), conf_min=net["conf_min"])
    if "theta" in case:
        kw.update(far_field="treecode", tree_theta=case["theta"], tree_order=case["order"])
    bs.bs_set_policy(h, **kw)


def prepare(case, seed):
    kind = case["kind"]
    x, w, t = _mesh(case, seed)
    dev = x.device
    s = dict(kind=kind, mesh=bs.bs_mesh_upload(x, w, t))
    if kind == "selector":
        bs.bs_set_policy(s["mesh"], kind=bs.BS_POLICY_FIXED)
        pairs = bs.bs_learn_sample_pairs(s["mesh"], case["rows"], int(seed))
        with open(NETWORK) as f:
            blob = np.array(json.load(f)["blob_bf16_bits"], dtype=np.uint16)
        s.update(pairs=pairs, blob=blob, class_w=(0.67, 0.1, 0.23, 1.0))
        return s
    if kind == "gradient":
        n = x.shape[0]
        # a smooth velocity, as an evaluation would have left it
        s.update(vel=(torch.sin(1.3 * x.roll(1, dims=1)) * torch.cos(0.7 * x) + 0.1 * w / w.abs().max()).contiguous(),
                 grad=torch.empty((n, 3, 3), dtype=torch.float64, device=dev),
                 rate=torch.empty((n, 3), dtype=torch.float64, device=dev))
        return s
    _set_policy(s["mesh"], case)
    if kind == "points":
        p = _points(case, seed, dev)
        s["points"] = p
        n = p.shape[0]
    else:
        n = x.shape[0]
    if kind == "stage":
        s.update(xyz=_moved(x, seed), omega=(1.05 * w).contiguous())
    s.update(noalloc=bool(case.get("noalloc")), out=torch.empty((n, 3), dtype=torch.float64, device=dev),
             vel=torch.empty((n, 3), dtype=torch.float32, device=dev))
    return s


def run(state):
    m, kind = state["mesh"], state["kind"]
    if kind == "selector":
        feats, labels, errs = bs.bs_learn_pairs(m, state["pairs"], 0.01)
        loss, grads = bs.bs_mlp_grad(state["blob"], feats, labels, class_w=state["class_w"])
        return dict(features=feats, labels=labels, errors=errs, loss=loss, grads=grads)
    if kind == "gradient":
        bs.bs_velocity_gradient(m, vel=state["vel"], out=state["grad"])
        bs.bs_stretching_rate(m, vel=state["vel"], out=state["rate"])
        return dict(grad=state["grad"], rate=state["rate"])
    if kind == "points":
        bs.bs_eval_points(m, state["points"], out=state["out"])
    elif state["noalloc"]:
        bs.bs_eval_velocity_noalloc(m, state["out"])
    else:
        if kind == "stage":
            bs.bs_mesh_update(m, xyz=state["xyz"], omega=state["omega"])
        bs.bs_eval_velocity(m, out=state["out"])
    return dict(velocity=state["vel"].copy_(state["out"]))


# --------------------------------------------------------------------- work

def _sizes(case):
    nodes = (case["cx"] + 1) * (case["cy"] + 1) * (case["cz"] + 1)
    return nodes, 6 * case["cx"] * case["cy"] * case["cz"]


def work(case):
    """Bytes and operations (FMA = 2) of the method: 26 per Gauss point; ray
    tracing 9 per pair, 7 per line and 156 per line that hits; the treecode a
    few hundred accepted clusters per node."""
    n, T = _sizes(case)
    mesh = 48.0 * n + 16.0 * T
    if case["kind"] == "gradient":
        return dict(bytes=mesh + 24.0 * n + 96.0 * n, flops=110.0 * T + 30.0 * 4 * T)
    if case["kind"] == "selector":
        r = case["rows"]
        # per pair: four faces of a 24 x 24 rule, 50 each; network 3 x 10752
        return dict(bytes=r * (8.0 + 64 + 1 + 12), flops=r * (4 * 576 * 50.0 + 3 * 10752))
    nt = case.get("points", n)
    L = 2.0 * _lines(case) ** 2
    # a Kuhn cell's mean edge is about 1.3 cell edges
    near = [min(T, 6 * 4 / 3 * math.pi * (1.3 * c) ** 3) for c in CUTS]
    flops = 0.0
    if case["policy"] == "pure_rt":
        hits = L * 1.5 * max(case["cx"], case["cy"], case["cz"])
        flops = nt * (T * (9.0 + 3.5 * L) + 156.0 * hits)
    else:
        flops += nt * 26.0 * (4 * (near[2] - near[1]) + 11 * (near[1] - near[0]))
        flops += nt * (near[0] * (9.0 + 3.5 * L) + 156.0 * 2 * L)
        if case["policy"] == "learned":
            flops += nt * near[0] * 10752.0
        if "theta" in case:
            D = case["order"] + 1
            flops += nt * min(T / 64.0, 40.0 * case["theta"] ** -2) * 12.0 * (D + 1) * (D + 2) * (D + 3) / 6
        else:
            flops += nt * 26.0 * (T - near[2])
    return dict(bytes=mesh + 36.0 * nt + (24.0 * nt if "points" in case else 0.0), flops=flops)


# ------------------------------------------------------------ FP64 reference

def exact(case, seed):
    if case["kind"] == "selector" or case.get("policy") == "learned" or "theta" in case:
        return None  # a BF16 network's decisions; expansions
    n, T = _sizes(case)
    x, w, t = _mesh(case, seed)
    if case["kind"] == "gradient":
        vel = (torch.sin(1.3 * x.roll(1, dims=1)) * torch.cos(0.7 * x) + 0.1 * w / w.abs().max())
        grad = _gradient64(x, t.long(), vel)
        return dict(grad=grad, rate=(grad @ w[:, :, None])[:, :, 0])
    if n * T > 1e10 or (case["policy"] == "pure_rt" and n * T * _lines(case) ** 2 > 1e10):
        return None  # minutes in plain torch
    tgt = None
    if case["kind"] == "points":
        tgt = _points(case, seed, x.device)
    elif case["kind"] == "stage":
        x, w = _moved(x, seed), 1.05 * w
    return dict(velocity=_velocity64(x, w, t.long(), tgt, _lines(case), case["policy"] == "pure_rt"))


def _gradient64(x, t, vel):
    e = x[t[:, 1:]] - x[t[:, :1]]
    d = vel[t[:, 1:]] - vel[t[:, :1]]
    vol = torch.linalg.det(e).abs() / 6
    g = d.transpose(1, 2) @ torch.linalg.inv(e.transpose(1, 2))
    num = torch.zeros((x.shape[0], 9), dtype=torch.float64, device=x.device)
    den = torch.zeros(x.shape[0], dtype=torch.float64, device=x.device)
    for k in range(4):
        num.index_add_(0, t[:, k], (g * vol[:, None, None]).reshape(-1, 9))
        den.index_add_(0, t[:, k], vol)
    return (num / den[:, None]).reshape(-1, 3, 3)


def _rays(lines, device):
    t, q = np.polynomial.legendre.leggauss(lines)
    phi, th = (1 + t) * math.pi / 2, (1 + t) * math.pi / 2
    d = np.stack([np.sin(phi)[:, None] * np.cos(th)[None, :], np.sin(phi)[:, None] * np.sin(th)[None, :],
                  np.repeat(np.cos(phi)[:, None], lines, axis=1)], axis=-1).reshape(-1, 3)
    k = (math.pi / 16 * np.sin(phi)[:, None] * q[:, None] * q[None, :]).reshape(-1)
    return (torch.tensor(np.concatenate([d, -d]), dtype=torch.float64, device=device),
            torch.tensor(np.concatenate([k, k]), dtype=torch.float64, device=device))


def _gauss_rules():
    a, b = (5 + 3 * math.sqrt(5)) / 20, (5 - math.sqrt(5)) / 20
    four = [([a if j == q else b for j in range(4)], 0.25) for q in range(4)]
    c, d = (1 + math.sqrt(5 / 14)) / 4, (1 - math.sqrt(5 / 14)) / 4
    eleven = [([0.25] * 4, -148 / 1875)]
    eleven += [([11 / 14 if j == q else 1 / 14 for j in range(4)], 343 / 7500) for q in range(4)]
    eleven += [([c if j in p else d for j in range(4)], 56 / 375) for p in itertools.combinations(range(4), 2)]
    return four, eleven


def _sum_points(x, p, W, on):
    """sum over the points p (strengths W) of on * W x (x - p) / |x - p|^3."""
    c = x.mean(dim=0)
    xc, pc = x - c, p - c
    d2 = torch.addmm((pc * pc).sum(dim=1)[None, :] + (xc * xc).sum(dim=1)[:, None], xc, pc.t(), alpha=-2)
    s = d2.rsqrt_()
    s = torch.where(on, s * s * s, torch.zeros((), dtype=torch.float64, device=x.device))
    return torch.linalg.cross(s @ W, xc) - s @ torch.linalg.cross(W, pc)


def _velocity64(x, w, t, tgt, lines, all_rt):
    dev, T = x.device, t.shape[0]
    v, om = x[t], w[t]
    e = torch.cat([t[:, p] for p in ([0, 1], [0, 2], [0, 3], [1, 2], [1, 3], [2, 3])])
    e = torch.unique(e.min(dim=1).values * x.shape[0] + e.max(dim=1).values)
    hbar = float((x[e // x.shape[0]] - x[e % x.shape[0]]).norm(dim=1).mean())
    rt2, g11_2, g4_2 = (float(np.float32((c * hbar) ** 2)) for c in CUTS)
    vol = torch.linalg.det(v[:, 1:] - v[:, :1]).abs() / 6
    cen = (((v[:, 0] + v[:, 1]) + v[:, 2]) + v[:, 3]) * 0.25
    c32 = cen.float()
    rules = [[(cen, om.mean(dim=1) * (vol / (4 * math.pi))[:, None])]]
    for rule in _gauss_rules():
        lam = torch.tensor([r[0] for r in rule], dtype=torch.float64, device=dev)
        rules.append([((v * lam[q][None, :, None]).sum(dim=1),
                       (om * lam[q][None, :, None]).sum(dim=1) * (rule[q][1] * vol / (4 * math.pi))[:, None])
                      for q in range(len(rule))])
    reach = (v - cen[:, None, :]).norm(dim=2).max(dim=1).values
    # the barycentric coordinates around the centroid, lam_j = 1/4 + gl_j . y,
    # and the vorticity's gradient G[b, c] = d omega_c / d y_b
    inv = torch.linalg.inv((v[:, 1:] - v[:, :1]).transpose(1, 2))
    gl = torch.cat([-inv.sum(dim=1, keepdim=True), inv], dim=1)
    tet = torch.cat([cen, reach[:, None], om.mean(dim=1), gl.reshape(-1, 12), (gl.transpose(1, 2) @ om).reshape(-1, 9)],
                    dim=1)
    dirs, kap = _rays(lines, dev)
    X = x if tgt is None else tgt
    out = torch.zeros((X.shape[0], 3), dtype=torch.float64, device=dev)
    # targets by coarse cells, so that those of one chunk are close together
    cell = ((X - X.min(dim=0).values) / (4 * hbar)).long()
    order = torch.argsort((cell[:, 2] * 4096 + cell[:, 1]) * 4096 + cell[:, 0], stable=True)
    B = int(max(32, min(1024, 3e8 // max(T, 1))))
    for c0 in range(0, X.shape[0], B):
        ids = order[c0:c0 + B]
        xc, b = X[ids], ids.numel()
        x32 = xc.float()
        d2 = (x32[:, None, 0] - c32[None, :, 0]).square_()
        d2 += (x32[:, None, 1] - c32[None, :, 1]).square_()
        d2 += (x32[:, None, 2] - c32[None, :, 2]).square_()
        rt = d2 < rt2
        if all_rt:
            rt = torch.ones_like(rt)
        elif tgt is None:
            loc = torch.full((x.shape[0],), -1, dtype=torch.int64, device=dev)
            loc[ids] = torch.arange(b, device=dev)
            lt = loc[t]
            at = (lt >= 0).nonzero()
            rt[lt[at[:, 0], at[:, 1]], at[:, 0]] = True
        acc = torch.zeros((b, 3), dtype=torch.float64, device=dev)
        if not all_rt:
            m11 = (d2 < g11_2) & ~rt
            m4 = (d2 < g4_2) & ~(d2 < g11_2) & ~rt
            acc += _sum_points(xc, *rules[0][0], ~(m11 | m4 | rt))
            for on, rule in ((m4, rules[1]), (m11, rules[2])):
                sel = on.any(dim=0).nonzero()[:, 0]
                on = on[:, sel]
                for p, W in rule:
                    acc += _sum_points(xc, p[sel], W[sel], on)
        pairs = rt.nonzero()
        del d2, rt
        P = int(max(1, 3e8 // dirs.shape[0]))
        for p0 in range(0, pairs.shape[0], P):
            _ray_trace(xc, tet, pairs[p0:p0 + P], dirs, kap, acc)
        out[ids] = acc
    return out


def _ray_trace(xc, tet, pairs, dirs, kap, acc):
    """Adds the chords of the rays from targets pairs[:, 0] through tets
    pairs[:, 1]: each ray is clipped by the four face planes and at the
    target, the vorticity along it is linear."""
    i, q = pairs[:, 0], tet[pairs[:, 1]]
    c = q[:, :3] - xc[i]
    # rays that can meet the tet: those within its bounding sphere's cone
    dist = c.norm(dim=1).clamp_min(1e-300)
    ratio = (q[:, 3] * (1 + 1e-9) / dist).clamp_max(1.0)
    cmin = torch.where(ratio < 1, (1 - ratio * ratio).sqrt() - 1e-5, torch.full_like(ratio, -2.0))
    ok = (c / dist[:, None]).float() @ dirs.float().t() >= cmin.float()[:, None]
    pr, l = ok.nonzero(as_tuple=True)
    del ok
    gl, G = q[:, 7:19].reshape(-1, 4, 3), q[:, 19:].reshape(-1, 3, 3)
    lam0 = 0.25 - (gl @ c[:, :, None])[:, :, 0]
    w0 = q[:, 4:7] - (c[:, :, None] * G).sum(dim=1)
    d = dirs[l]
    near = torch.zeros(l.shape[0], dtype=torch.float64, device=d.device)
    far = torch.full_like(near, math.inf)
    for f in range(4):
        sl = (gl[:, f][pr] * d).sum(dim=1)
        rho = -lam0[:, f][pr] / sl
        near = torch.where(sl > 0, torch.maximum(near, rho), near)
        far = torch.where(sl < 0, torch.minimum(far, rho), far)
    hit = far > near
    pr, d, near, far, l = pr[hit], d[hit], near[hit], far[hit], l[hit]
    slope = (d[:, :, None] * G[pr]).sum(dim=1)
    wsum = 2 * w0[pr] + (near + far)[:, None] * slope
    acc.index_add_(0, i[pr], torch.linalg.cross(d, wsum) * (kap[l] * (far - near) / 2)[:, None])
