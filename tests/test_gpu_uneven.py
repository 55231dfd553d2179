"""Batches of evaluations of very different sizes: every item's result and
gradient is bitwise that of the item alone, whatever stands beside it (the
rasteriser's tiles and the adjoint's blocks are numbered through the batch, and
gradient groups of 8 to 64 patches share one launch)."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

NODES65 = dict(seed=3, bus_n=8, n_greebles=20, seg_nx=3, seg_ny=4)


def _group(n, slots):
    """Patches per gradient group: the smallest power of two from 8 to 64 whose
    partials of `slots` doubles fit 8 MiB."""
    patches, g = 4 * (-(-n // 16)) ** 2, 8
    while g < 64 and -(-patches // g) * slots * 8 > 8 << 20:
        g *= 2
    return g


def _alone(srp, entries, out, grad, which):
    res = srp.results_to_numpy(out)
    for k in which:
        if grad is None:
            o1 = srp.eval_batch([entries[k]])
        else:
            o1, g1 = srp.eval_grad_batch([entries[k]])
            w = g1.shape[1]
            assert np.array_equal(grad[k, :w].cpu().numpy(), g1[0].cpu().numpy()), k
        assert res[k].tobytes() == srp.results_to_numpy(o1)[0].tobytes(), k


@pytest.mark.parametrize("grad", [False, True])
@pytest.mark.parametrize("first", [True, False])
def test_one_fine_image_among_coarse_ones(grad, first):
    import paper_2608_07307_amd as srp
    fine, coarse = srp.Scene(synth.procedural_sized(7, 4000)), srp.Scene(synth.box_wing())
    rng = np.random.default_rng(2)
    entries = [(coarse, None, srp.params(s, int(n), 1)) for s, n in zip(rng.normal(size=(300, 3)), rng.integers(1, 80, 300))]
    for n, at in ((1100, 0 if first else 250), (300, 100), (64, 299)):
        entries.insert(at, (fine, None, srp.params(rng.normal(size=3), n, 2)))
    out, g = srp.eval_grad_batch(entries) if grad else (srp.eval_batch(entries), None)
    _alone(srp, entries, out, g, [0, 1, 99, 100, 101, 102, 249, 250, 251, 252, 300, 301, 302])


@pytest.mark.parametrize("n,group", [(700, 8), (1000, 16), (1500, 32), (2000, 64)])
def test_material_gradients_at_every_group_size(n, group):
    """In rho_d of a scene without specular reflection the force is affine, so
    dF/drho_d is exactly (F(rho_d + h) - F(rho_d)) / h; the last group is ragged
    at n = 1000, 1500 and 2000."""
    import paper_2608_07307_amd as srp
    mesh = synth.greebled_spacecraft(**NODES65)
    sc = srp.Scene(mesh)
    M = len(mesh.mats)
    assert _group(n, 9 * len(mesh.parent) + 6 * M) == group
    assert group == 8 or 4 * (-(-n // 16)) ** 2 % group != 0
    rng = np.random.default_rng(n)
    mats = np.zeros((M, 2))
    mats[:, 1] = 0.25
    sc.set_materials(mats)
    ang, p = rng.uniform(-1, 1, mesh.n_dof), srp.params(rng.normal(size=3), n, 0)
    out, grad = srp.eval_grad_batch([(sc, ang, p)])
    g = grad[0].cpu().numpy()[3 * M:6 * M].reshape(M, 3)
    F0 = srp.results_to_numpy(out)[0]["force"]
    for m in range(M):
        moved = mats.copy()
        moved[m, 1] = 0.75
        sc.set_materials(moved)
        F1 = srp.results_to_numpy(srp.eval_batch([(sc, ang, p)]))[0]["force"]
        # FP32 terms of at most a few times the largest force per hit: the rounding
        # of both evaluations and of the gradient's terms stays below 2^-20 of the force
        assert np.abs((F1 - F0) / 0.5 - g[m]).max() <= 2.0 ** -20 * 4 * np.abs(F0).max(), m


def test_one_batch_of_every_group_size():
    import paper_2608_07307_amd as srp
    mesh = synth.greebled_spacecraft(**NODES65)
    big, small = srp.Scene(mesh), srp.Scene(synth.box_wing())
    rng = np.random.default_rng(9)
    sizes = [(small, 33), (big, 2000), (big, 100), (big, 1000), (small, 500), (big, 1500), (small, 16)]
    slots = 9 * len(mesh.parent) + 6 * len(mesh.mats) + 9
    assert {_group(n, slots) for s, n in sizes if s is big} == {8, 16, 32, 64}
    entries = [(s, rng.uniform(-1, 1, s.n_dof), srp.params(rng.normal(size=3), n, 1, grad_dir=True)) for s, n in sizes]
    out, grad = srp.eval_grad_batch(entries)
    _alone(srp, entries, out, grad, range(len(entries)))
