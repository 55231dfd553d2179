"""Tiles that the rasteriser leaves to the traversal (hit more than 24 times over),
beside tiles that it finishes, against launches that trace every primary ray
(they count their tests): forces, torques, counts, recorded rays and gradients."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

FIELDS = ("force", "torque", "n_rays", "n_hits", "n_secondary", "n_secondary_hits", "status", "n_clamped")


def _fins(layers, width):
    """A sphere of 5,120 triangles, a plate, and a stack of `layers` fins `width` wide beside it."""
    parts = [synth.icosphere(subdiv=4), synth.plate((-3, -3, -1.5), (6, 0, 0), (0, 6, 0), nu=16, nv=16)]
    parts += [synth.plate((1.5, 1, -0.4 + 0.8 * k / layers), (width, 0, 0), (0, width, 0), nu=2, nv=2) for k in range(layers)]
    m = synth.icosphere(subdiv=0)
    at = np.cumsum([0] + [len(p.verts) for p in parts])
    m.tris = np.concatenate([p.tris + a for p, a in zip(parts, at)]).astype(np.int32)
    m.verts = np.concatenate([p.verts for p in parts])
    m.tri_mat, m.tri_node = np.zeros(len(m.tris), np.int32), np.zeros(len(m.tris), np.int32)
    return m


@pytest.mark.parametrize("layers,n,items,bounces", [
    (120, 250, 20, 2),    # 8-pixel tiles, ragged
    (120, 520, 31, 1),    # 16-pixel tiles, ragged
    (40, 512, 32, 0),     # fins just above the limit
    (400, 1024, 1, 2),    # one evaluation
])
def test_left_tiles_are_the_traversals(layers, n, items, bounces):
    import paper_2608_07307_amd as srp
    sc = srp.Scene(_fins(layers, 1.0))
    rng = np.random.default_rng(layers)
    suns = rng.normal(size=(items, 3))
    suns[0] = (0.05, -0.03, 1.0)    # along the stack: every layer behind every other
    out = [srp.results_to_numpy(srp.eval_batch([(sc, None, srp.params(s, n, bounces, count=c)) for s in suns]))
           for c in (False, True)]
    for f in FIELDS:
        assert np.array_equal(out[0][f], out[1][f]), f
    assert (out[1]["n_tri_tests"] > 0).all() and (out[0]["n_hits"] > 0).all()


def test_left_tiles_recorded_and_differentiated():
    import paper_2608_07307_amd as srp
    sc = srp.Scene(_fins(120, 1.0))
    sun = np.array([0.05, -0.03, 1.0])
    r = [srp.eval(sc, sun, 1030, bounces=2, count=c, record=True) for c in (False, True)]
    assert np.array_equal(r[0]["ids"], r[1]["ids"]) and np.array_equal(r[0]["ts"], r[1]["ts"])
    # rasterised, with left tiles, in the batch; traced alone (too few patches)
    ent = [(sc, None, srp.params(s, 250, 2, grad_dir=True)) for s in np.random.default_rng(1).normal(size=(20, 3)) * 0.1 + sun]
    out, grad = srp.eval_grad_batch(ent)
    for k in (0, 10, 19):
        o1, g1 = srp.eval_grad_batch([ent[k]])
        assert srp.results_to_numpy(out)[k].tobytes() == srp.results_to_numpy(o1)[0].tobytes()
        assert np.array_equal(grad[k].cpu().numpy(), g1[0].cpu().numpy())
