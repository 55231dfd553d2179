"""Rasterised launches at the edges of their rule and through every call that can
take one, against launches that trace all primary rays (they count their tests)
or against the items alone.  Which of these sizes are rasterised is checked on
the CPU (test_host_calls.py)."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

FIELDS = ("force", "torque", "n_rays", "n_hits", "n_secondary", "n_secondary_hits", "status", "n_clamped")


def _on_booms(subdiv, length):
    """A sphere of 20 x 4^subdiv triangles and six bare booms of `length` times its radius."""
    L, w = length, 0.02
    parts = [synth.icosphere(subdiv=subdiv)] + [synth.plate(o, u, v, nu=4, nv=1) for o, u, v in (
        ((-L, -w, 0), (2 * L, 0, 0), (0, 2 * w, 0)), ((-w, 0, -L), (0, 0, 2 * L), (2 * w, 0, 0)),
        ((0, -L, -w), (0, 2 * L, 0), (0, 0, 2 * w)))]
    m = synth.icosphere(subdiv=0)
    at = np.cumsum([0] + [len(p.verts) for p in parts])
    m.tris = np.concatenate([p.tris + a for p, a in zip(parts, at)]).astype(np.int32)
    m.verts = np.concatenate([p.verts for p in parts])
    m.tri_mat, m.tri_node = np.zeros(len(m.tris), np.int32), np.zeros(len(m.tris), np.int32)
    return m


@pytest.mark.parametrize("kind,n,items", [
    ("even", 400, 53),       # 0.51 triangles per pixel in 132,500 patches: only big launches are rasterised
    ("even", 372, 60),       # 0.592, the last tenth below the limit, ragged
    ("crowded", 1024, 8),    # 6,000 triangles in a tile: its node stack fills and goes depth first
    ("crowded", 1040, 8),
])
def test_dense_images(kind, n, items):
    import paper_2608_07307_amd as srp
    sc = srp.Scene(synth.icosphere(subdiv=6) if kind == "even" else _on_booms(6, 20))
    suns = np.random.default_rng(n).normal(size=(items, 3))
    out = [srp.results_to_numpy(srp.eval_batch([(sc, None, srp.params(s, n, 1, count=c)) for s in suns]))
           for c in (False, True)]
    for f in FIELDS:
        assert np.array_equal(out[0][f], out[1][f]), f
    assert (out[1]["n_box_tests"] > 0).all() and (out[0]["n_box_tests"] == 0).all()


@pytest.mark.parametrize("n,items", [(256, 16), (512, 30)])   # with the hits in the fixed 64 MiB; without room for them
def test_allocation_free_calls(n, items):
    import torch
    import paper_2608_07307_amd as srp
    mesh = synth.procedural_sized(7, 4000)
    sc = srp.Scene(mesh)
    rng = np.random.default_rng(items)
    e = [(sc, rng.uniform(-1, 1, mesh.n_dof), srp.params(s, n, 2)) for s in rng.normal(size=(items, 3))]
    out = torch.empty(items * srp.RESULT_DTYPE.itemsize, dtype=torch.uint8, device="cuda")
    srp.eval_batch_noalloc(e, out, torch.cuda.current_stream())
    assert srp.results_to_numpy(out).tobytes() == srp.results_to_numpy(srp.eval_batch(e)).tobytes()


def test_a_rasterised_batch_split_at_the_workspace_cap():
    import paper_2608_07307_amd as srp
    sc = srp.Scene(synth.icosphere(subdiv=4))
    # 520 bytes per patch for the hits: 28 images of 8192^2 pass 16 GiB
    e = [(sc, None, srp.params(s, 8192, 0)) for s in np.random.default_rng(4).normal(size=(30, 3))]
    out = srp.results_to_numpy(srp.eval_batch(e))
    for k in (0, 14, 15, 29):
        assert srp.results_to_numpy(srp.eval_batch([e[k]]))[0].tobytes() == out[k].tobytes()
    assert (out["n_hits"] > 0).all()
