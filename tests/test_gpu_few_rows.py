"""The few-rows products (one wavefront per tile of 16 rows by 16 or 32 columns)
against the 64 x 64 kernel: every output element sums its K products in the
same order in both, so forward logits must agree bit for bit. The shapes put
one K step, fewer than the steps in flight, exactly all of them and several
rounds of them through it (64 / 192 / 768 / 1280 and 3456 deep), with K parts
and without, and rows at the edges of a 16-row tile."""
import numpy as np
import pytest

import synth
from tests import gpu_util as gu

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,f,rows", [(64, 64, 1), (64, 192, 15), (192, 320, 16), (192, 576, 17),
                                      (768, 2048, 18), (768, 2048, 33), (768, 2048, 100),
                                      (1024, 2816, 49), (1280, 3456, 16), (1280, 3456, 131)])
def test_few_rows_equal_the_64x64_kernel(monkeypatch, d, f, rows):
    shape = synth.ModelShape(2, d, d // 64, f, 192, 10, 12, has_lm_bias=True)
    blob = synth.make_weights(shape, 3, std=0.05, bias_std=1.0)
    rng = np.random.default_rng(rows)
    # sequences of uneven lengths with `rows` rows in all
    lens = []
    while sum(lens) + len(lens) < rows:
        lens.append(min(int(rng.integers(0, 60)), rows - sum(lens) - len(lens) - 1))
    toks = rng.integers(0, shape.vocab, size=(len(lens), shape.T)).astype(np.int32)
    labels = rng.integers(0, shape.n_classes + 1, size=len(lens)).astype(np.int32)
    outs = []
    for force in ["small", ""]:
        if force:
            monkeypatch.setenv("HBSJD_GEMM_TILE", force)
        else:
            monkeypatch.delenv("HBSJD_GEMM_TILE", raising=False)
        ctx = gu.make_ctx(shape, "bf16", blob)
        outs.append(ctx.hbsjd_forward(torch.from_numpy(toks).cuda(), lens, labels).cpu().numpy())
        del ctx
    assert outs[0].shape[0] == rows and np.isfinite(outs[0]).all() and outs[0].std() > 0.1
    assert np.array_equal(outs[0].view(np.uint32), outs[1].view(np.uint32))
