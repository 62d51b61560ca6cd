"""The persistent batched schedule while small pairs finish early: their
remaining tasks are skipped, so that a workgroup claims task after task with
nothing between the claims, next to the first sweeps of large pairs.  Every
wave has to take the task its workgroup claimed, whatever holds it up: the
results of all repetitions are the same bits."""

import hashlib

import numpy as np
import pytest


torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_skipped_tasks_beside_large_pairs():
    import paper_1909_00101_amd as hz
    rng = np.random.default_rng(2)
    pairs = []
    for n, count in ((16, 160), (30, 160), (200, 48), (247, 48)):
        for _ in range(count):
            f = rng.standard_normal((n + n // 2, n))
            g = rng.standard_normal((2 * n, n))
            pairs.append((torch.from_numpy(np.asfortranarray(f)).cuda(),
                          torch.from_numpy(np.asfortranarray(g)).cuda()))
    digests = set()
    for rep in range(30):
        st, outs = hz.gsvd_batched(pairs)
        assert st == 0, (rep, sorted({o["status"] for o in outs}))
        z = torch.cat([o["Z"].t().reshape(-1) for o in outs]).cpu().numpy()
        digests.add(hashlib.sha256(z.tobytes()).hexdigest())
    assert len(digests) == 1
