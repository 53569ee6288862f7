"""The distribution transform at the edges of its block sizes (one wavefront per
2048 entries, two threads per 64-entry chunk), against the oracle: the kept
set, the argmax and the draw are decisions and compared exactly (the draw with
the oracle's inverse CDF on the GPU's own row), p to the last-bit difference of
the two exponentials (2e-6 relative, as the full-vocabulary tests derive it).
Rows hold masked entries (-inf), ties at the top-k threshold, ranges that have no
finite width, and ranges on both sides of the one where the quotients come from
the reciprocal."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V", [4, 60, 64, 68, 2044, 2048, 2052, 4096, 4100, 8192, 8196, 16380])
def test_transform_rows_at_block_edges(V):
    import paper_2608_18183_amd as P
    rng = np.random.default_rng(V)
    n = 12
    for cfg in (0.0, 2.0):
        x = rng.normal(0, 1, (n, 2 if cfg else 1, V)).astype(np.float32)
        x[1::4] *= 12                                   # quotients below 2^-80
        x[2, :, rng.permutation(V)[: V // 2]] = 0.5     # ties
        tau = np.where(np.arange(n) % 3 == 0, 1.0, np.where(np.arange(n) % 3 == 1, 0.3, 1.5))
        tau = tau.astype(np.float32)
        pos = rng.integers(1, 600, n).astype(np.int32)
        for top_k in (1, max(1, V // 8), V - 1, 0):
            if top_k == 0 and not cfg:                  # masked entries
                x[3, :, rng.permutation(V)[: V // 4]] = -np.inf
            dev = [torch.from_numpy(np.ascontiguousarray(a)).cuda()
                   for a in (x if cfg else x[:, 0], tau, pos)]
            p, am, z = (t.cpu().numpy() for t in P.hbsjd_transform_rows(
                dev[0], dev[1], dev[2], top_k=top_k, cfg_scale=cfg, seed=77))
            for r in range(n):
                g = oracle.cfg_combine(x[r, 0], x[r, 1], cfg) if cfg else x[r, 0]
                want = oracle.transform(g, float(tau[r]), top_k)
                y = g / tau[r]
                kept = y >= np.sort(y)[::-1][top_k - 1] if 0 < top_k < V else np.ones(V, bool)
                assert not np.any((p[r] > 0) & ~kept)
                np.testing.assert_allclose(p[r], want, rtol=2e-6, atol=np.float32(2.0 ** -126))
                assert am[r] == oracle.argmax(g)
                assert z[r] == oracle.inv_cdf(p[r], oracle.uniforms(77, r, int(pos[r]))[0])


def _wide_row(kind, V, rng):
    """A row whose logits span no finite width, or one too small to divide by."""
    x = rng.normal(0, 1, V).astype(np.float32)
    some = rng.permutation(V)
    if kind == "quarter masked":
        x[some[: V // 4]] = -np.inf
    elif kind == "all but three masked":
        x[some[3:]] = -np.inf
    elif kind == "masked with ties":
        x[some[: V // 2]] = -np.inf
        x[some[V // 2: V // 2 + V // 4]] = 0.25
    elif kind == "lowest finite value":      # / 0.3 overflows
        x[some[: V // 4]] = np.finfo(np.float32).min
    elif kind == "overflowing difference":
        x = (x * np.float32(6e37)).astype(np.float32)
        x[some[:2]] = (3.2e38, -3.2e38)
    elif kind == "subnormal":
        x = (rng.integers(0, V, V) * 2.0 ** -149).astype(np.float32)
    elif kind == "signed zeros":
        x = np.where(rng.integers(0, 2, V) == 1, np.float32(-0.0), np.float32(0.0))
        x[some[: V // 4]] = -np.inf
        x[some[V // 4: V // 4 + V // 8]] = 2.0 ** -130
    return x


@pytest.mark.parametrize("V", [64, 260, 2052, 16384])
def test_transform_rows_top_k_over_ranges_without_finite_width(V):
    """The kept set is the oracle's whatever the row's range: masked entries,
    differences that overflow and ranges too small to divide by."""
    import paper_2608_18183_amd as P
    rng = np.random.default_rng(V)
    kinds = ["quarter masked", "all but three masked", "masked with ties", "lowest finite value",
             "overflowing difference", "subnormal", "signed zeros"]
    for cfg in (0.0, 2.0):
        x = np.stack([_wide_row(k, V, rng) for k in kinds])
        tau = np.array([0.3 if k == "lowest finite value" else 1.0 for k in kinds], np.float32)
        pos = rng.integers(1, 600, len(kinds)).astype(np.int32)
        # the guided rows are u + 2 (c - u): u = 0 keeps masked entries masked,
        # u = c / 2 elsewhere makes 1.5 c, and u = c leaves the row that would
        # overflow as it is
        u = np.where(np.abs(x) > 1e38, np.float32(0), x / np.float32(2)).astype(np.float32)
        u[kinds.index("overflowing difference")] = x[kinds.index("overflowing difference")]
        dev = [torch.from_numpy(np.ascontiguousarray(a)).cuda()
               for a in (np.stack([x, u], 1) if cfg else x, tau, pos)]
        for top_k in (1, V // 16, V // 8, V // 2, V - 1):
            p, am, z = (t.cpu().numpy() for t in P.hbsjd_transform_rows(
                dev[0], dev[1], dev[2], top_k=top_k, cfg_scale=cfg, seed=78))
            for r, kind in enumerate(kinds):
                g = oracle.cfg_combine(x[r], u[r], cfg) if cfg else x[r]
                want = oracle.transform(g, float(tau[r]), top_k)
                with np.errstate(over="ignore"):
                    y = g / tau[r]
                kept = y >= np.sort(y)[::-1][top_k - 1]
                assert not np.any((p[r] > 0) & ~kept), (kind, cfg, top_k)
                np.testing.assert_allclose(p[r], want, rtol=2e-6, atol=np.float32(2.0 ** -126),
                                           err_msg=f"{kind} {cfg} {top_k}")
                assert am[r] == oracle.argmax(g)
                assert z[r] == oracle.inv_cdf(p[r], oracle.uniforms(78, r, int(pos[r]))[0])


def test_transform_rows_from_several_threads_and_after_an_error():
    """Calls at once from several host threads on streams of their own report
    their own NaN rows and nobody else's, and a later call is clean."""
    import threading

    import paper_2608_18183_amd as P
    rng = np.random.default_rng(5)
    x = rng.normal(0, 1, (64, 1024)).astype(np.float32)
    tau = torch.ones(64, device="cuda")
    pos = torch.arange(64, dtype=torch.int32, device="cuda")
    good = torch.from_numpy(x).cuda()
    x[63, 1023] = np.nan
    bad = torch.from_numpy(x).cuda()
    want = P.hbsjd_transform_rows(good, tau, pos, top_k=100, seed=3)
    torch.cuda.synchronize()
    wrong = []

    def work(k):
        stream = torch.cuda.Stream()
        for _ in range(20):
            if k % 2:
                try:
                    P.hbsjd_transform_rows(bad, tau, pos, top_k=100, seed=3, stream=stream)
                    wrong.append("a NaN went unseen")
                except P.HbsjdError as e:
                    if e.code != "EINVAL":
                        wrong.append(e.code)
            else:
                got = P.hbsjd_transform_rows(good, tau, pos, top_k=100, seed=3, stream=stream)
                if not all(torch.equal(g, w) for g, w in zip(got, want)):
                    wrong.append("rows differ")

    threads = [threading.Thread(target=work, args=(k,)) for k in range(6)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong
    got = P.hbsjd_transform_rows(good, tau, pos, top_k=100, seed=3)
    assert all(torch.equal(g, w) for g, w in zip(got, want))
