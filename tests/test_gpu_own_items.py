"""Launches whose waves have an item each trace every patch once: chunk totals
around the launch sizes at which they begin (256 blocks) and end (one item more
than waves), at one and two blocks per compute unit and ragged chunks, bitwise
against single evaluations."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,items,ppc,bpc", [
    (16, 255, 1, 1),    # 1,020 chunks, 255 blocks: queues
    (16, 256, 1, 1),    # 1,024, 256: own items, every wave has one
    (16, 257, 1, 1),    # 1,028 on 256 blocks: queues
    (16, 257, 1, 2),    # 257 blocks: own items
    (33, 30, 1, 2),     # 1,080 chunks on 270 blocks
    (16, 511, 1, 2),    # 2,044 on 511
    (16, 512, 1, 2),    # 2,048 on 512
    (16, 513, 1, 2),    # 2,052 on 512: queues
    (33, 150, 5, 2),    # 1,200 chunks, the last of every item shorter
    (16, 1024, 1, 4),   # 4,096 on 1,024
])
def test_every_wave_traces_its_own_item(n, items, ppc, bpc):
    import paper_2608_07307_amd as srp
    mesh = synth.box_wing()
    sc = srp.Scene(mesh)
    rng = np.random.default_rng(n * 1000 + items)
    sun, ang = rng.normal(size=(items, 3)), rng.uniform(-1.0, 1.0, size=(items, mesh.n_dof))
    entries = [(sc, a, srp.params(s, n, 1)) for a, s in zip(ang, sun)]
    try:
        srp.set_schedule(ppc, bpc)
        out = srp.results_to_numpy(srp.eval_batch(entries))
        plan = srp.Plan(entries)
        replays = [srp.results_to_numpy(plan.launch()) for _ in range(10)]   # (ordered by cost from the ninth on)
        plan.close()
    finally:
        srp.set_schedule(0, 0)
    assert all(r.tobytes() == out.tobytes() for r in replays)
    for k in [0, 1, items // 2, items - 1]:
        sc.set_angles(ang[k])
        one = srp.eval(sc, sun[k], n, bounces=1)
        for f in ("force", "torque", "n_hits", "n_secondary", "n_secondary_hits", "status"):
            assert np.array_equal(np.asarray(out[k][f]), np.asarray(one[f])), (k, f)
