"""A context's forwards between calls of other shapes: the page table and the
packed metadata follow each call's own sequences (the logits equal, bit for
bit, those of a context that made no other call), and a token outside the
vocabulary is refused without disturbing the calls after it."""
import numpy as np
import pytest

import synth
from tests import gpu_util as gu

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_forwards_between_other_calls(dtype):
    import paper_2608_18183_amd as P
    shape = synth.ModelShape(2, 64, 1, 128, 64, 5, 9)
    blob = synth.make_weights(shape, 1, std=0.1)
    rng = np.random.default_rng(2)

    def inputs(n):
        toks = torch.from_numpy(rng.integers(0, 64, (n, shape.T)).astype(np.int32)).cuda()
        return toks, rng.integers(0, shape.T + 1, n).tolist(), rng.integers(0, 6, n).tolist()

    calls = [inputs(n) for n in (2, 7, 1, 7, 40, 2)]
    want = []
    for c in calls:
        ctx = gu.make_ctx(shape, dtype, blob)
        want.append(ctx.hbsjd_forward(*c).clone())
        del ctx
    ctx = gu.make_ctx(shape, dtype, blob)
    for c, w in zip(calls, want):
        assert torch.equal(ctx.hbsjd_forward(*c), w)
        ctx.hbsjd_rollout(c[0], [60] * len(c[1]), [0] * len(c[1]), [1.0] * len(c[1]), 6,
                          cfg_scale=1.5 if len(c[1]) > 4 else 0.0, seed=9)
        assert torch.equal(ctx.hbsjd_forward(*c), w)
        bad = c[0].clone()
        bad[0, 0] = 64
        with pytest.raises(P.HbsjdError) as e:
            ctx.hbsjd_forward(bad, [shape.T] * len(c[1]), c[2])
        assert e.value.code == "EINVAL"
        assert torch.equal(ctx.hbsjd_forward(*c), w)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_new_weights_do_not_meet_the_old_ones_values(dtype):
    """Weights that diverged leave NaN keys and values in the KV pool. After a
    load of good ones, no later sequence may see them: its last key tile reaches
    past its end, and a probability of zero times NaN is NaN."""
    shape = synth.ModelShape(2, 64, 1, 128, 64, 5, 9)
    blob = synth.make_weights(shape, 1, std=0.1)
    rng = np.random.default_rng(3)
    toks = torch.from_numpy(rng.integers(0, 64, (3, shape.T)).astype(np.int32)).cuda()
    args = ([5, 40, 70], [0, 1, 2])
    want = gu.make_ctx(shape, dtype, blob).hbsjd_forward(toks, *args).clone()
    ctx = gu.make_ctx(shape, dtype, np.full_like(blob, np.nan))
    assert torch.isnan(ctx.hbsjd_forward(toks, [shape.T] * 3, [0, 1, 2])).all()
    ctx.hbsjd_load_weights(blob)
    assert torch.equal(ctx.hbsjd_forward(toks, *args), want)
    ro = dict(seed=9)
    a = ctx.hbsjd_rollout(toks, [60] * 3, [0] * 3, [1.0] * 3, 6, **ro)["tokens"]
    b = gu.make_ctx(shape, dtype, blob).hbsjd_rollout(toks, [60] * 3, [0] * 3, [1.0] * 3, 6, **ro)["tokens"]
    assert torch.equal(a, b)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("how", ["forward", "score", "calibrate"])
def test_a_sequence_that_overflows_leaves_nothing_to_later_calls(dtype, how):
    """Token 1 (and class 0, which calibration uses) has no finite embedding, so
    every row from it on is NaN; a later call without it must not meet those
    rows' values."""
    shape = synth.ModelShape(2, 64, 1, 128, 64, 5, 9)
    V, d, T = shape.vocab, shape.d_model, shape.T
    blob = synth.make_weights(shape, 1, std=0.1)
    blob[d: 2 * d] = np.inf
    blob[V * d: (V + 1) * d] = np.inf
    rng = np.random.default_rng(3)
    good = torch.from_numpy(rng.integers(2, 64, (3, T)).astype(np.int32)).cuda()
    bad = good.clone()
    bad[:, 20:] = 1
    args = ([5, 40, 70], [1, 2, 3])
    want = gu.make_ctx(shape, dtype, blob).hbsjd_forward(good, *args).clone()
    assert torch.isfinite(want).all()
    ctx = gu.make_ctx(shape, dtype, blob)
    if how == "forward":
        assert not torch.isfinite(ctx.hbsjd_forward(bad, [T] * 3, [1, 2, 3])).all()
    elif how == "score":
        other = gu.make_ctx(shape, dtype, blob)
        ctx.hbsjd_score_bikl(other, bad, [10] * 3, [1, 2, 3])
        assert torch.equal(other.hbsjd_forward(good, *args), want)
    else:
        ctx.hbsjd_calibrate_gamma(3, 4)
    assert torch.equal(ctx.hbsjd_forward(good, *args), want)
    assert torch.equal(ctx.hbsjd_forward(good, *args), want)
