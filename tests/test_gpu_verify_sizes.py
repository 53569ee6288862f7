"""Verification of explicit rows at the edges of its block sizes (one wavefront
per 2048 entries, two threads per 64-entry chunk), bit for bit against the
oracle: rejections whose residual is ordinary, zero everywhere (the draw falls
back to p), confined to the last entry, and drawn with the largest uniform."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,W", [(4, 1), (60, 3), (64, 65), (68, 5), (2044, 4), (2048, 4),
                                 (2052, 4), (4096, 3), (4100, 3), (8192, 3), (8196, 3), (16384, 2)])
def test_verify_probs_at_block_edges(V, W):
    import paper_2608_18183_amd as P
    rng = np.random.default_rng(V)
    B = 10
    p = (rng.random((B, W, V)) ** 4).astype(np.float32)
    p[3, :, : V // 2] = 0
    p /= p.sum(-1, keepdims=True, dtype=np.float32)
    q = (rng.random((B, W, V)) ** 4).astype(np.float32)
    q /= q.sum(-1, keepdims=True, dtype=np.float32)
    drafts = rng.integers(0, V, (B, W)).astype(np.int32)
    ua = rng.random((B, W)).astype(np.float32)
    ur = rng.random(B).astype(np.float32)
    top = np.float32(1.0 - 2.0 ** -24)
    q[1] = p[1]                                   # residual zero: drawn from p
    z = drafts[1, 0]
    q[1, 0, z] = np.nextafter(p[1, 0, z], np.float32(2.0))
    ua[1, 0] = top
    q[2] = np.maximum(q[2], p[2])                 # residual in the last entry only
    q[2, :, V - 1] = 0
    drafts[2] = 0
    q[2, :, 0] = 1
    ua[2] = top
    ur[4:6] = top                                 # the target meets the total
    ur[6] = 0
    ua[4:7] = top
    rc, rt = oracle.verify_probs(p, q, drafts, ua, ur)
    dev = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (p, q, drafts, ua, ur)]
    gc, gt = P.hbsjd_verify_probs(*dev)
    assert np.array_equal(gc.cpu().numpy(), rc)
    assert np.array_equal(gt.cpu().numpy(), rt)
    assert rc[2] == 1 and rt[2, 0] == V - 1 and rt[1, rc[1] - 1] >= 0
