"""The fp32 path's small-launch products (16 x 16 tiles, K in passes of 128) and
its attention at their edges, against the oracle: widths that leave part of a
tile, an odd MLP width (which takes the general kernel), one pass and several
with a remainder, a launch on each side of the rule, head dims of 4 to 64 and
positions on both sides of a 64-key page. Both sides add in fp32 in the same
order up to the exponentials, so the fp32 forward's bar of 1e-4 holds."""
import numpy as np
import pytest

import oracle
import synth
from tests import gpu_util as gu

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,heads,f,V,grid,lens", [
    (16, 4, 30, 20, 4, [0, 16]), (20, 5, 33, 36, 4, [15]), (64, 1, 176, 256, 9, [63, 64, 81]),
    (132, 3, 260, 100, 9, [0, 31, 65]), (192, 3, 516, 1024, 12, [143, 1, 127, 128]),
    (64, 2, 64, 4096, 12, [144, 140, 100])])
def test_forward_f32_small_launches_match_oracle(d, heads, f, V, grid, lens):
    shape = synth.ModelShape(2, d, heads, f, V, 7, grid, has_lm_bias=True)
    blob = synth.make_weights(shape, 4, std=0.08, bias_std=0.5)
    rng = np.random.default_rng(d)
    toks = rng.integers(0, V, size=(len(lens), shape.T)).astype(np.int32)
    labels = rng.integers(0, shape.n_classes + 1, size=len(lens)).astype(np.int32)
    ctx = gu.make_ctx(shape, "f32", blob)
    got = ctx.hbsjd_forward(torch.from_numpy(toks).cuda(), lens, labels).cpu().numpy()
    ref = np.concatenate(oracle.Model(shape, blob).forward_batch(
        labels, [toks[i, :n] for i, n in enumerate(lens)]))
    assert got.shape == ref.shape and ref.std() > 0.1
    assert np.abs(got - ref).max() < 1e-4
