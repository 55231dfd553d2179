"""Adjoint chains held a part at a time: a captured gradient batch beyond the
workspace cap traces and sweeps its patches in windows of 1 GiB of chains, cut
inside evaluations, and gives bitwise the gradients of the eager call, which is
split at the cap and holds whole chains."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def test_captured_gradients_in_chain_windows():
    import torch
    import paper_2608_07307_amd as srp
    mesh = synth.procedural_sized(7, 4000)
    sc, small = srp.Scene(mesh), srp.Scene(synth.box_wing())
    rng = np.random.default_rng(6)

    def entries():
        e = [(sc, rng.uniform(-1, 1, mesh.n_dof) if k % 50 == 0 else None, srp.params(rng.normal(size=3), 2048, 4))
             for k in range(150)]
        e.insert(70, (small, None, srp.params(rng.normal(size=3), 100, 4)))
        return e
    # whole chains and hits of these pass the 16 GiB cap; the chains alone are 12 windows
    assert 150 * 65536 * (256 * 5 + 520) > 16 << 30 and 150 * 65536 * 256 * 5 > 11 << 30
    plan = srp.Plan(entries(), grad=True)
    for _ in range(2):
        e = entries()
        plan.update(e)
        out = srp.results_to_numpy(plan.launch())
        torch.cuda.synchronize()
        got = plan.grad.cpu().numpy().copy()
        out2, grad2 = srp.eval_grad_batch(e)
        assert out.tobytes() == srp.results_to_numpy(out2).tobytes()
        assert np.array_equal(got, grad2.cpu().numpy())
        assert np.abs(got).max() > 0 and (out["status"] == 0).all() and out["n_secondary_hits"].sum() > 0
    plan.close()
