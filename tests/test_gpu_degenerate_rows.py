"""Rollouts whose logits define no distribution: every entry -inf, or NaN. No token
index out of range may come of them: a greedy rollout of -inf rows takes the
first entry, as the oracle's argmax does, and everything else ends in the
device check's error."""
import numpy as np
import pytest

import oracle
import synth
from tests import gpu_util as gu

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SHAPES = {"f32": synth.ModelShape(2, 64, 4, 176, 256, 10, 8, True),
          "bf16": synth.ModelShape(1, 128, 2, 192, 256, 10, 8, True)}


def _rollout(dtype, bias, mode, window=4):
    shape = SHAPES[dtype]
    blob = synth.make_weights(shape, 0)
    blob[-shape.vocab:] = bias
    B, T = 3, shape.T
    rng = np.random.default_rng(1)
    toks = torch.from_numpy(rng.integers(0, shape.vocab, (B, T)).astype(np.int32)).cuda()
    plen = np.array([0, 7, T - 3], np.int32)
    ctx = gu.make_ctx(shape, dtype, blob)
    out = ctx.hbsjd_rollout(toks, plen, np.zeros(B, np.int32), np.ones(B, np.float32), window,
                            seed=3, verify_mode=mode)
    return toks.cpu().numpy(), plen, out["tokens"].cpu().numpy()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("mode", ["VERIFY_GREEDY", "VERIFY_AR_GREEDY"])
def test_greedy_rollout_of_minus_infinity_takes_the_first_entry(dtype, mode):
    import paper_2608_18183_amd as P
    assert oracle.argmax(np.full(8, -np.inf, np.float32)) == 0
    toks, plen, got = _rollout(dtype, -np.inf, getattr(P, mode))
    for b, k in enumerate(plen):
        assert np.array_equal(got[b, :k], toks[b, :k])
        assert np.all(got[b, k:] == 0)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("bias,mode", [(-np.inf, "VERIFY_PROB"), (-np.inf, "VERIFY_AR"),
                                       (np.nan, "VERIFY_PROB"), (np.nan, "VERIFY_AR"),
                                       (np.nan, "VERIFY_GREEDY"), (np.nan, "VERIFY_AR_GREEDY")])
def test_rollout_without_a_distribution_ends_in_an_error(dtype, bias, mode):
    import paper_2608_18183_amd as P
    with pytest.raises(P.HbsjdError) as e:
        _rollout(dtype, bias, getattr(P, mode))
    assert e.value.code == "EINTERNAL"


def test_transform_of_a_row_of_minus_infinity():
    import paper_2608_18183_amd as P
    x = np.full((2, 260), -np.inf, np.float32)
    x[1, 5] = 1.0
    for top_k in (0, 3):
        p, am, z = P.hbsjd_transform_rows(torch.from_numpy(x).cuda(), torch.ones(2, device="cuda"),
                                          torch.ones(2, dtype=torch.int32, device="cuda"),
                                          top_k=top_k)
        assert am.tolist() == [0, 5] and z.tolist() == [-1, 5]
        assert p[1, 5] == 1.0 and p[1].sum() == 1.0
