"""The adjoint's gradient groups: whatever the number of patches (fewer than a
group, a ragged last group, groups of 8 and of 64 patches) and of bounces, the
gradients of one evaluation through the adjoint equal the difference of two
evaluations where the force is affine: in rho_d of a scene without specular
reflection, dF/drho_d is exactly (F(rho_d + h) - F(rho_d)) / h."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nodes", [(1, 9), (16, 9), (17, 9), (100, 9), (250, 9), (700, 65)])
@pytest.mark.parametrize("bounces", [0, 4])
def test_material_gradients_of_a_matt_body(n, nodes, bounces):
    import paper_2608_07307_amd as srp
    mesh = synth.procedural_sized(3, 3000) if nodes == 9 else \
        synth.greebled_spacecraft(seed=3, bus_n=8, n_greebles=20, seg_nx=3, seg_ny=4)
    assert len(mesh.parent) == nodes
    sc = srp.Scene(mesh)
    rng = np.random.default_rng(n)
    sun, ang = rng.normal(size=3), rng.uniform(-1, 1, mesh.n_dof)
    M = len(mesh.mats)
    mats = np.zeros((M, 2))
    mats[:, 1] = 0.25
    sc.set_materials(mats)
    p = srp.params(sun, n, bounces)
    out, grad = srp.eval_grad_batch([(sc, ang, p)])
    g = grad[0].cpu().numpy()[3 * M:6 * M].reshape(M, 3)
    F0 = srp.results_to_numpy(out)[0]["force"]
    scale = np.abs(F0).max()
    for m in range(M):
        moved = mats.copy()
        moved[m, 1] = 0.75
        sc.set_materials(moved)
        F1 = srp.results_to_numpy(srp.eval_batch([(sc, ang, p)]))[0]["force"]
        # FP32 terms of at most a few times the largest force per hit: the rounding
        # of both evaluations and of the gradient's terms stays below 2^-20 of the force
        assert np.abs((F1 - F0) / 0.5 - g[m]).max() <= 2.0 ** -20 * 4 * max(scale, 1e-30), m


@pytest.mark.parametrize("bounces", [2, 3, 4])
def test_material_gradients_of_long_chains(bounces):
    """With fixed specular fractions the paths do not depend on rho_d and the
    force is affine in it, so the same difference is exact over chains of as
    many hits as there are words read ahead (three) and more."""
    import paper_2608_07307_amd as srp
    mesh = synth.procedural_sized(3, 3000)
    sc = srp.Scene(mesh)
    rng = np.random.default_rng(5)
    M = len(mesh.mats)
    mats = np.zeros((M, 2))
    mats[:, 0], mats[:, 1] = 0.5, 0.125
    items = [(sc, rng.uniform(-1, 1, mesh.n_dof), srp.params(rng.normal(size=3), 300, bounces)) for _ in range(6)]
    sc.set_materials(mats)
    if bounces > 2:   # some chains are longer than those of one bounce less
        fewer = [(s, a, srp.params(p.sun_dir, 300, bounces - 1)) for s, a, p in items]
        count = [srp.results_to_numpy(srp.eval_batch(x))["n_secondary_hits"].sum() for x in (fewer, items)]
        assert count[1] > count[0]
    out, grad = srp.eval_grad_batch(items)
    g = grad.cpu().numpy()[:, 3 * M:6 * M].reshape(len(items), M, 3)
    F0 = srp.results_to_numpy(out)["force"]
    scale = max(np.abs(F0).max(), np.abs(g).max())
    for m in range(M):
        moved = mats.copy()
        moved[m, 1] = 0.375
        sc.set_materials(moved)
        F1 = srp.results_to_numpy(srp.eval_batch(items))["force"]
        # FP32 rounding of the terms of up to five hits, in both forces (over the step of
        # a fourth) and in the recovered weights: below 2^-20 of the largest value each
        assert np.abs((F1 - F0) / 0.25 - g[:, m]).max() <= 2.0 ** -20 * 16 * scale, m
