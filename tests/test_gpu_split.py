"""The 16-bit split contractions (bs_split_dev.h) at the edges of their
dispatch, against the FP64 oracle: tet counts around the 32-tet unit and the
256-tet chunk, coordinates and strengths far from one, strengths over many
decades in one mesh, and an extent beyond the contraction's number range
(more than 128 G4 cuts), which the binary32 contraction takes.

Tolerances as in the parity tests: relative L2 error 1e-6 over all nodes, and
at every node 5e-6 of the larger of its own and the root-mean-square
velocity.  Also rays that leave the mesh and enter it again."""
import numpy as np
import pytest

import oracle
import paper_0712_1695_amd as bs
import workloads as W

pytestmark = pytest.mark.gpu

CUTS = dict(near_cut=0.5, d_g11=0.75, d_g4=1.0)  # G1 pairs on the smallest meshes


def compare(v, ref, label):
    scale = np.sqrt(np.mean(np.sum(ref * ref, axis=1)))
    e = float(np.linalg.norm(v - ref) / np.linalg.norm(ref))
    worst = float((np.linalg.norm(v - ref, axis=1) / np.maximum(np.linalg.norm(ref, axis=1), scale)).max())
    print(f"  {label} rel-L2 {e:.3e}, worst node {worst:.3e}", flush=True)
    assert e <= 1e-6 and worst <= 5e-6, (label, e, worst)


def run(xyz, om, tets, cuts=CUTS, **pol):
    h = bs.bs_mesh_upload(xyz, om, tets)
    bs.bs_set_policy(h, kind=bs.BS_POLICY_FIXED, **cuts, **pol)
    v, st = bs.bs_eval_velocity(h, stats=True)
    bs.bs_mesh_free(h)
    return v, st


@pytest.mark.parametrize("cells", [(1, 1, 1), (5, 1, 1), (2, 3, 1), (6, 7, 1), (43, 1, 1), (8, 7, 6)])
def test_tet_counts_around_units_and_chunks(cells):
    """6, 30, 36, 252, 258 and 2,016 tets."""
    m = W.make_config("C1", scale=cells)
    v, st = run(m.xyz, m.omega, m.tets)
    ref, cnt = oracle.evaluate(m.xyz, m.omega, m.tets, oracle.make_policy("fixed", **CUTS), return_counters=True)
    assert st["pairs_by_rule"] == cnt["pairs_by_rule"]
    compare(v, ref, f"{cells} {st['pairs_by_rule']}")


@pytest.mark.parametrize("length,strength", [(1.0, 1e20), (1.0, 1e-20), (1000.0, 3e-7), (1 / 64, 7e5)])
def test_scales(length, strength):
    m = W.make_config("C1", scale=(8, 7, 6))
    xyz, om = length * m.xyz, strength * m.omega
    ref = oracle.evaluate(xyz, om, m.tets, oracle.make_policy("fixed"))
    compare(run(xyz, om, m.tets, cuts={})[0], ref, f"length {length} strength {strength}")


def test_strengths_over_many_decades():
    m = W.make_config("C1", scale=(8, 7, 6))
    om = m.omega * 10.0 ** np.random.default_rng(3).uniform(-30, 0, size=(m.n_nodes, 1))
    ref = oracle.evaluate(m.xyz, om, m.tets, oracle.make_policy("fixed"))
    compare(run(m.xyz, om, m.tets, cuts={})[0], ref, "strengths over 30 decades")


@pytest.mark.parametrize("far", [10.0, 2000.0])
def test_points_far_outside(far):
    """Points beyond the mesh (nodes of no tet): an extent within 128 G4 cuts
    and one beyond.  512 mesh nodes and 128 points, so that no 64-node block
    mixes the two; the vorticity has a net strength, so the far velocities do
    not cancel."""
    m = W.make_config("C1", scale=(7, 7, 7))
    om = m.omega + np.array([0.3, -0.2, 0.5])
    pts = np.random.default_rng(5).uniform(-1, 1, size=(128, 3)) + far * np.array([1.0, 0.3, 0.2])
    xyz, om = np.concatenate([m.xyz, pts]), np.concatenate([om, np.zeros((128, 3))])
    ref = oracle.evaluate(xyz, om, m.tets, oracle.make_policy("fixed"))
    v, _ = run(xyz, om, m.tets, cuts={})
    compare(v[:512], ref[:512], "mesh")
    compare(v[512:], ref[512:], "far points")


@pytest.mark.parametrize("prec", [0, 1, 2])
@pytest.mark.parametrize("kind", ["pure_rt", "fixed"])
def test_rays_entering_the_mesh_again(kind, prec):
    """A box with a slot cut out and a hole: rays leave the mesh and enter it
    again, some twice, and the nodes inside the cut belong to no tet.
    (Precision 0 sums in plain binary32: ten times the tolerance.)"""
    m = W.make_config("C1", scale=(9, 8, 7))
    c = m.xyz[m.tets].mean(axis=1)
    cut = ((np.abs(c[:, 0]) < 0.35) & (c[:, 1] > -0.3)) | (np.linalg.norm(c - [0.6, 0.4, 0.1], axis=1) < 0.3)
    tets = np.ascontiguousarray(m.tets[~cut])
    h = bs.bs_mesh_upload(m.xyz, m.omega, tets)
    k = bs.BS_POLICY_PURE_RT if kind == "pure_rt" else bs.BS_POLICY_FIXED
    bs.bs_set_policy(h, kind=k, n_phi=8, n_theta=12, precision=prec)
    v, st = bs.bs_eval_velocity(h, stats=True)
    bs.bs_mesh_free(h)
    ref, cnt = oracle.evaluate(m.xyz, m.omega, tets, oracle.make_policy(kind, n_phi=8, n_theta=12),
                               return_counters=True)
    assert st["pairs_by_rule"] == cnt["pairs_by_rule"]
    e = float(np.linalg.norm(v - ref) / np.linalg.norm(ref))
    scale = np.sqrt(np.mean(np.sum(ref * ref, axis=1)))
    worst = float((np.linalg.norm(v - ref, axis=1) / np.maximum(np.linalg.norm(ref, axis=1), scale)).max())
    print(f"  {kind} precision {prec}: {st['rt_walk_nodes']} walked, {st['rt_candidate_nodes']} with candidate rays, "
          f"rel-L2 {e:.3e}, worst node {worst:.3e}", flush=True)
    f = 1 if prec else 10
    assert e <= 1e-6 * f and worst <= 5e-6 * f, (e, worst)


@pytest.mark.parametrize("prec", [0, 1, 2])
def test_points_walk_from_their_tet(prec):
    """Points (fixed rule, convex box): deep inside tets, within 1e-6 of
    faces, edges and nodes, on them, and outside; those clear of every face
    walk from the tet that holds them, the others take candidate rays.  The
    oracle takes the points as nodes of no tet."""
    m = W.make_config("C1", scale=(7, 8, 6))
    rng = np.random.default_rng(2)
    t = m.xyz[m.tets[rng.choice(m.n_tets, 240, replace=False)]]
    lam = rng.dirichlet([2.0] * 4, size=240)
    lam[60:120] = rng.dirichlet([1.0] * 3, size=60) @ np.eye(4)[:3]
    lam[60:90, 3] = 1e-6
    lam[120:150] = [0.3, 0.7, 0.0, 0.0]
    lam[150:160] = [1.0, 0.0, 0.0, 0.0]
    lam /= lam.sum(axis=1, keepdims=True)
    pts = np.einsum("ij,ijk->ik", lam, t)
    pts[220:] += np.array([2.5, 0.1, -0.2])  # outside
    pts[90:120] += 1e-3 * rng.normal(size=(30, 3))
    # (on a shared face, edge or node the chord's start is a tie: not compared)
    keep = np.r_[0:90, 90:120, 160:240]
    h = bs.bs_mesh_upload(m.xyz, m.omega, m.tets)
    bs.bs_set_policy(h, kind=bs.BS_POLICY_FIXED, precision=prec)
    v, st = bs.bs_eval_points(h, pts, stats=True)
    bs.bs_mesh_free(h)
    assert np.isfinite(v).all() and st["rt_walk_nodes"] > 100 and st["rt_candidate_nodes"] >= 20
    xyz, om = np.concatenate([m.xyz, pts]), np.concatenate([m.omega, np.zeros_like(pts)])
    ref, cnt = oracle.evaluate(xyz, om, m.tets, oracle.make_policy("fixed"),
                               targets=np.arange(m.n_nodes, m.n_nodes + len(pts)), return_counters=True)
    assert st["pairs_by_rule"] == cnt["pairs_by_rule"]
    v, ref = v[keep], ref[keep]
    scale = np.sqrt(np.mean(np.sum(ref * ref, axis=1)))
    e = float(np.linalg.norm(v - ref) / np.linalg.norm(ref))
    worst = float((np.linalg.norm(v - ref, axis=1) / np.maximum(np.linalg.norm(ref, axis=1), scale)).max())
    print(f"  points precision {prec}: {st['rt_walk_nodes']} walked, {st['rt_candidate_nodes']} with candidate rays, "
          f"rel-L2 {e:.3e}, worst {worst:.3e}", flush=True)
    f = 1 if prec else 10
    assert e <= 1e-6 * f and worst <= 5e-6 * f, (e, worst)
