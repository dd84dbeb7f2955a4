"""The far field's range: targets far from every tet, weak strengths, and
evaluations beside evaluation points, against the FP64 oracle.

A far pair's term carries a few units in the last place of binary32 (the
distance, the reciprocal square root cubed, the products): 3e-7 of the sum of
the terms' magnitudes S, in L2 over the targets.  S and not the velocity is the
scale because the terms may cancel."""
import numpy as np
import pytest

import oracle
import paper_0712_1695_amd as bs
import workloads as W

pytestmark = pytest.mark.gpu


def fixed(h, **kw):
    bs.bs_set_policy(h, kind=bs.BS_POLICY_FIXED, **kw)


def magnitudes(x, om, tets, pts):
    v = x[tets]
    vol = np.abs(W.signed_volumes6(x, tets)) / 6.0
    w = np.linalg.norm(om[tets].mean(axis=1), axis=1) * vol / (4 * np.pi)
    d2 = ((pts[:, None] - v.mean(axis=1)[None]) ** 2).sum(axis=2)
    return (w[None] / d2).sum(axis=1)


@pytest.mark.parametrize("cells", [(1, 1, 1), (7, 7, 7)])
@pytest.mark.parametrize("cut", [0.51, 0.99])
@pytest.mark.parametrize("far", [4, 20, 30, 34, 60, 100, 125])
def test_targets_far_from_every_tet(cells, cut, far):
    """Points `far` G4 cuts away, the cut just above and just below a power of
    two, with the field as it is (no net strength) and with one added."""
    m = W.make_config("C1", scale=cells)
    if cells == (1, 1, 1):
        m.omega = np.random.default_rng(9).normal(size=m.xyz.shape)
    x = m.xyz * (cut / (8 * oracle.mean_edge(m.xyz, m.tets)))
    rng = np.random.default_rng(far)
    p = far * cut * np.array([1.0, 0.3, 0.2]) / np.linalg.norm([1.0, 0.3, 0.2])
    pts = p + 0.1 * cut * rng.uniform(-1, 1, size=(64, 3))
    for om in (m.omega, m.omega + np.array([0.3, -0.2, 0.5])):
        h = bs.bs_mesh_upload(x, om, m.tets)
        fixed(h)
        v = bs.bs_eval_points(h, pts)
        bs.bs_mesh_free(h)
        ref = oracle.evaluate(np.concatenate([x, pts]), np.concatenate([om, 0 * pts]), m.tets,
                              oracle.make_policy("fixed"), targets=np.arange(len(x), len(x) + 64))
        e = np.linalg.norm(v - ref) / np.linalg.norm(magnitudes(x, om, m.tets, pts))
        print(f"  {m.n_tets} tets, {far} cuts of {cut}: error {e:.2e} of the terms", flush=True)
        assert e <= 3e-7, e


@pytest.mark.parametrize("exponent", [-22, -24, -26, -28, -31, -34])
def test_weak_vorticity(exponent):
    """Velocities are linear in the vorticity down to the end of binary32's
    normal range (relative L2 1e-6, as for vorticity of order one)."""
    m = W.make_config("C1", scale=(8, 7, 6))
    cuts = dict(near_cut=0.5, d_g11=0.75, d_g4=1.0)
    om = m.omega * 10.0 ** exponent
    h = bs.bs_mesh_upload(m.xyz, om, m.tets)
    fixed(h, **cuts)
    v = bs.bs_eval_velocity(h)
    bs.bs_mesh_free(h)
    ref = oracle.evaluate(m.xyz, om, m.tets, oracle.make_policy("fixed", **cuts))
    e = np.linalg.norm((v - ref) * 10.0 ** -exponent) / np.linalg.norm(ref * 10.0 ** -exponent)
    print(f"  vorticity 1e{exponent}: rel-L2 {e:.2e}", flush=True)
    assert e <= 1e-6, e


@pytest.mark.parametrize("far", [3.0, 10.0, 20.0, 40.0, 1000.0])
def test_nodes_after_points(far):
    """Evaluation points stay with the mesh; wherever they lie, the nodes' own
    velocities are the same bits after them as before."""
    m = W.make_config("C1", scale=(8, 7, 6))
    cuts = dict(near_cut=0.5, d_g11=0.75, d_g4=1.0)
    cut = oracle.mean_edge(m.xyz, m.tets)
    h = bs.bs_mesh_upload(m.xyz, m.omega, m.tets)
    fixed(h, **cuts)
    v0 = bs.bs_eval_velocity(h)
    bs.bs_eval_points(h, np.array([[far * cut, 0.1, -0.2], [0.3, 0.2, 0.1]]))
    v1 = bs.bs_eval_velocity(h)
    bs.bs_mesh_free(h)
    assert np.array_equal(v0, v1), np.abs(v0 - v1).max()
