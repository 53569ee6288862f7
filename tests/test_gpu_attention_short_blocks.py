"""Attention of blocks of up to 16 query rows, whose K and V go straight to LDS:
greedy rollouts (cached AR, one row a round, and windows of 2, 8 and 16 rows)
over caches of one to nine key tiles, so that a wavefront takes none, one and
several, with prefixes that start at the tiles' edges. Each committed token
must be the argmax of a teacher-forced forward of the finished sequence on
another attention kernel.

Tolerance: two fp16 evaluations differ by about 1e-3 of a logit's standard
deviation each (their error against 64 bits), so a committed token's logit may
lie below the largest by the difference of four such errors, 2e-3 of it on
average; ten times that bounds all of the few thousand positions. A wrong key
or value moves logits by their standard deviation."""
import numpy as np
import pytest

import paper_2608_18183_amd as hb
import synth
from tests import gpu_util as gu

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,mode", [(1, "ar"), (1, "greedy"), (7, "greedy"), (15, "greedy")])
def test_committed_tokens_are_the_argmax_of_a_forward(monkeypatch, W, mode):
    shape = synth.ModelShape(2, 128, 2, 320, 256, 5, 24)
    blob = synth.make_weights(shape, 7, std=0.1)
    rng = np.random.default_rng(W)
    T = shape.T
    plen = np.array([0, 63, 64, 255, 256, 257, 511, T - 1], np.int32)
    B = len(plen)
    toks = torch.from_numpy(rng.integers(0, 256, (B, T)).astype(np.int32)).cuda()
    labels = rng.integers(0, 5, B).astype(np.int32)
    out = gu.make_ctx(shape, "bf16", blob).hbsjd_rollout(
        toks, plen, labels, np.ones(B, np.float32), W, seed=3,
        verify_mode=hb.VERIFY_AR_GREEDY if mode == "ar" else hb.VERIFY_GREEDY)["tokens"]
    monkeypatch.setenv("HBSJD_ATTN_KERNEL", "seq")
    logits = gu.make_ctx(shape, "bf16", blob).hbsjd_forward(out, [T - 1] * B, labels)
    lg = logits.cpu().numpy().reshape(B, T, -1)
    new = np.arange(T)[None, :] >= plen[:, None]
    chosen = np.take_along_axis(lg, out.cpu().numpy()[:, :, None], 2)[:, :, 0]
    below = (lg.max(2) - chosen)[new] / lg.std()
    assert lg.std() > 0.1 and below.max() <= 0.02, (lg.std(), below.max())
