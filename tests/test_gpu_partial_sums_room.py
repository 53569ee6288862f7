"""The partial sums of the O and W2 products over a rollout whose rounds cut K
and whose prefill does not: 3310 prefill rows take one K part, the 1740 rows of a
round take two, so the round's sums (3480 rows) are the larger. The tokens must
equal those of a context whose buffers a larger call has grown first. (A round
that writes past an undersized buffer need not show here, as it reads the same
addresses back: the sizes themselves are checked in test_partial_sum_rows.py.)"""
import numpy as np
import pytest

import synth
from tests import gpu_util as gu

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_rollout_whose_rounds_split_k_and_whose_prefill_does_not():
    shape = synth.ModelShape(1, 768, 12, 2048, 256, 5, 16)
    blob = synth.make_weights(shape, 2, std=0.03)
    rng = np.random.default_rng(0)
    B, W = 29, 29
    plen = np.full(B, 51, np.int32)            # 58 sequences of 52 rows
    plen[-1] = 256 - 2 * W                     # and a longer one, the rounds stay few
    toks = torch.from_numpy(rng.integers(0, 256, (B, 256)).astype(np.int32)).cuda()
    labels = rng.integers(0, 5, B).astype(np.int32)
    tau = np.ones(B, np.float32)

    def run(ctx):
        return ctx.hbsjd_rollout(toks, plen, labels, tau, W, top_k=50, cfg_scale=2.0,
                                 seed=4)["tokens"].cpu().numpy()

    plain = gu.make_ctx(shape, "bf16", blob)
    grown = gu.make_ctx(shape, "bf16", blob)
    grown.hbsjd_forward(toks.repeat(2, 1)[:48], [200] * 48, [0] * 48)
    assert np.array_equal(run(plain), run(grown))
