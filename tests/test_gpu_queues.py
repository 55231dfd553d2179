"""The trace kernel's work queues hand out every chunk once: a patch that none
or two waves traced would change the item's sums and counts, so batches whose
chunk totals lie around multiples of the 64 queues, and at the shortest and
longest runs that one request takes, are compared bitwise with single
evaluations (which the oracle checks elsewhere)."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,items,ppc,bpc", [
    (16, 1, 1, 1),      # 4 chunks: most queues empty
    (16, 15, 1, 4),     # 60
    (16, 16, 1, 4),     # 64: one per queue
    (16, 17, 1, 2),     # 68
    (33, 7, 1, 1),      # 252
    (33, 7, 5, 4),      # a last chunk shorter than the others in every item
    (16, 2049, 1, 4),   # 8,196
    (100, 90, 1, 1),    # 17,640 chunks on the smallest grid: long runs
    (100, 91, 2, 4),    # 8,918
])
def test_every_chunk_is_traced_once(n, items, ppc, bpc):
    import torch
    assert torch.cuda.is_available()
    import paper_2608_07307_amd as srp
    mesh = synth.box_wing()
    sc = srp.Scene(mesh)
    rng = np.random.default_rng(n * 1000 + items)
    sun = rng.normal(size=(items, 3))
    ang = rng.uniform(-1.0, 1.0, size=(items, mesh.n_dof))
    batch = srp.Batch([(sc, a, srp.params(s, n, 1)) for a, s in zip(ang, sun)])
    try:
        srp.set_schedule(ppc, bpc)
        out = srp.results_to_numpy(srp.eval_batch(batch))
    finally:
        srp.set_schedule(0, 0)
    for k in list(range(items)) if items < 20 else [0, 1, items // 2, items - 1]:
        sc.set_angles(ang[k])
        one = srp.eval(sc, sun[k], n, bounces=1)
        for f in ("force", "torque", "n_hits", "n_secondary", "n_secondary_hits", "status"):
            assert np.array_equal(np.asarray(out[k][f]), np.asarray(one[f])), (k, f)
