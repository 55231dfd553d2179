"""Primary hits by rasterisation against the traversal.

A launch that counts its box and triangle tests traces its primary rays through
the hierarchy; the same launch without the counts rasterises them where the
rule says so.  Both must find the same triangle for every ray (the first
hit, ties by distance, then by index), so forces, torques and hit counts are
bitwise equal, and so are the gradients of a batch and of its items alone
(one evaluation of these sizes is below the rasteriser's threshold).
The traversal is compared with the oracle elsewhere."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

FIELDS = ("force", "torque", "n_rays", "n_hits", "n_secondary", "n_secondary_hits", "status", "n_clamped")


def _mesh(kind):
    if kind == "sphere":
        return synth.icosphere(subdiv=4)              # one node, 5,120 triangles
    if kind == "cluttered":
        return synth.procedural_sized(7, 4000)        # boxes, zero-area triangles at the dish's apex
    if kind == "many nodes":
        return synth.greebled_spacecraft(seed=3, bus_n=8, n_greebles=20, seg_nx=3, seg_ny=4)   # 65 nodes
    return synth.plate((-1, -1, 0), (2, 0, 0), (0, 2, 0), nu=8, nv=8)   # 128 coplanar triangles


def _suns(kind, items, rng):
    s = rng.normal(size=(items, 3))
    if kind == "plate":
        # along a diagonal of shared edges, edge-on, and windows down to a sliver's width
        for k, z in enumerate((0.0, 1e-12, 1e-7, 1e-3)):
            s[k] = (1.0, 1.0, z)
        s[4] = (0.0, 0.0, 1.0)
        s[5] = (0.0, 0.0, -1.0)
    else:
        s[0], s[1], s[2] = (1, 0, 0), (0, 1, 0), (0, 0, -1)
    return s


@pytest.mark.parametrize("kind,n,items", [
    ("sphere", 256, 16),        # 16,384 patches: the fewest that are rasterised, on 8-pixel tiles
    ("cluttered", 250, 20),     # rows and columns past the grid
    ("many nodes", 321, 12),
    ("plate", 129, 60),
    ("cluttered", 520, 31),     # 135,036 patches: 16-pixel tiles, ragged
    ("many nodes", 1024, 8),
    ("plate", 512, 32),
])
@pytest.mark.parametrize("bounces", [0, 2])
def test_rasterised_hits_are_the_traversals(kind, n, items, bounces):
    import torch
    assert torch.cuda.is_available()
    import paper_2608_07307_amd as srp
    mesh = _mesh(kind)
    sc = srp.Scene(mesh)
    rng = np.random.default_rng(n)
    suns = _suns(kind, items, rng)
    ang = rng.uniform(-1.0, 1.0, size=(items, mesh.n_dof))
    out = [srp.results_to_numpy(srp.eval_batch([(sc, a, srp.params(s, n, bounces, count=c)) for a, s in zip(ang, suns)]))
           for c in (False, True)]
    for f in FIELDS:
        assert np.array_equal(out[0][f], out[1][f]), f
    assert out[1]["n_box_tests"].min() >= 0 and out[0]["n_hits"].sum() > 0


def test_a_batch_mixing_rasterised_and_traced_items():
    import paper_2608_07307_amd as srp
    fine, coarse = _mesh("cluttered"), synth.box_wing()
    entries = []
    rng = np.random.default_rng(1)
    for k in range(40):
        m = fine if k % 3 else coarse
        entries.append((m, rng.uniform(-1, 1, m.n_dof), rng.normal(size=3), (250, 97, 60)[k % 3] + k))
    scenes = {id(m): srp.Scene(m) for m in (fine, coarse)}
    out = [srp.results_to_numpy(srp.eval_batch(
        [(scenes[id(m)], a, srp.params(s, n, 1, count=c)) for m, a, s, n in entries])) for c in (False, True)]
    for f in FIELDS:
        assert np.array_equal(out[0][f], out[1][f]), f


@pytest.mark.parametrize("n,items", [(250, 20), (520, 31)])
def test_gradients_from_rasterised_hits(n, items):
    import paper_2608_07307_amd as srp
    mesh = _mesh("cluttered")
    sc = srp.Scene(mesh)
    rng = np.random.default_rng(n)
    ent = [(sc, rng.uniform(-1, 1, mesh.n_dof), srp.params(s, n, 2, grad_dir=True)) for s in rng.normal(size=(items, 3))]
    out, grad = srp.eval_grad_batch(ent)
    for k in (0, items // 2, items - 1):
        o1, g1 = srp.eval_grad_batch([ent[k]])
        assert srp.results_to_numpy(out)[k].tobytes() == srp.results_to_numpy(o1)[0].tobytes()
        assert np.array_equal(grad[k].cpu().numpy(), g1[0].cpu().numpy())


def test_replayed_plan_with_rasterised_hits():
    """A captured batch replayed with new attitudes, with eager work between the replays."""
    import torch
    import paper_2608_07307_amd as srp
    mesh = _mesh("cluttered")
    sc = srp.Scene(mesh)
    rng = np.random.default_rng(3)

    def entries():
        return [(sc, rng.uniform(-1, 1, mesh.n_dof), srp.params(s, 250, 1)) for s in rng.normal(size=(20, 3))]
    plan = srp.Plan(entries())
    for _ in range(4):
        e = entries()
        plan.update(e)
        got = srp.results_to_numpy(plan.launch())
        torch.cuda.synchronize()
        assert got.tobytes() == srp.results_to_numpy(srp.eval_batch(e)).tobytes()
    plan.close()


@pytest.mark.parametrize("n", [1024, 1100])
def test_recorded_rays_of_a_rasterised_evaluation(n):
    """One evaluation fine enough to be rasterised, with every ray recorded."""
    import paper_2608_07307_amd as srp
    mesh = _mesh("cluttered")
    sc = srp.Scene(mesh)
    sc.set_angles(np.full(mesh.n_dof, 0.4))
    sun = np.array([0.3, -0.5, 0.8])
    r = [srp.eval(sc, sun, n, bounces=2, count=c, record=True) for c in (False, True)]
    assert r[0]["ids"].min() == -1 and r[0]["ids"].max() < len(mesh.tris)
    assert np.array_equal(r[0]["ids"], r[1]["ids"]) and np.array_equal(r[0]["ts"], r[1]["ts"])
    plain = srp.eval(sc, sun, n, bounces=2)
    for f in FIELDS:
        assert np.array_equal(np.asarray(r[0][f]), np.asarray(plain[f])), f
