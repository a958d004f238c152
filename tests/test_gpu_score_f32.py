"""fp32 score path at the edges of its variants: query counts around the
32-query blocks and the 128-query tile (one block splits the columns over four
waves, two over two), corpora around its 64-row tiles, slices of one tile (ranked),
of a few tiles, and of many (seeded), lists of up to 16 keys (in LDS) and more."""
import numpy as np
import pytest
import torch

import synth
from gpu_harness import check_dedup, check_unique_topk, device, note, run_merge, to_dev

pytestmark = pytest.mark.gpu


def _rows(n, d, stream):
    return synth.gaussian_rows(77, stream, n, d, "f32")[0]


# 70,001 rows of 64-row tiles are 1,094 tiles: more than four in each of the 256
# slices of one query tile, so the seed pass runs; 2,501 rows are 40 one-tile
# slices; 300 queries over 20,011 rows make slices of a few tiles, unseeded.
@pytest.mark.parametrize("nu,n,d,k", [
    (1, 1, 4, 1), (1, 63, 28, 16), (31, 64, 32, 17), (32, 65, 36, 10), (33, 2_501, 100, 16),
    (64, 2_501, 96, 17), (65, 2_501, 64, 10), (128, 2_501, 68, 40), (129, 2_501, 64, 10),
    (300, 20_011, 32, 10), (20, 70_001, 36, 10), (40, 70_001, 36, 17), (120, 70_001, 36, 1),
    (130, 70_001, 36, 100),
])
def test_f32_variant_edges(nu, n, d, k):
    note(f"fp32 n_u={nu} N={n} d={d} k={k}")
    keys = np.random.default_rng(nu).permutation(nu).astype(np.int64)
    q, c = _rows(nu, d, 201), _rows(n, d, 202)
    m = run_merge(keys, q, c, k)
    check_unique_topk(m, check_dedup(m, keys), q, c, k)


@pytest.mark.parametrize("n", [2_501, 70_001])
def test_f32_scores_do_not_depend_on_the_batch(n):
    # the sum of a score has one order whatever the batch: the first b queries
    # alone (through each variant) give the rows they have in the batch of 130
    import paper_2607_22578_amd as hs
    d, k, nu = 100, 12, 130
    q, c = _rows(nu, d, 203), _rows(n, d, 204)
    c[n // 2] = c[7]                     # equal rows: bit-identical scores, lower row first
    q[3] = c[7]
    dev = device()
    m = hs.MergedRetrieval(nu, d, n, k, hs.HS_F32, hs.HS_F32, device=dev)
    qd, cd = to_dev(q), to_dev(c)
    m.q_unique[:nu].copy_(qd)

    def score(b):
        hs.hs_score_topk(m.plan, m.q_unique, b, None, cd, None, m.topk_score, m.topk_index, m.ws)
        torch.cuda.synchronize()
        return m.topk_score[:b].cpu().numpy().copy(), m.topk_index[:b].cpu().numpy().copy()

    all_s, all_i = score(nu)
    assert list(all_i[3][:2]) == [7, n // 2]
    assert all_s[3][0].view(np.uint32) == all_s[3][1].view(np.uint32)
    for b in (1, 32, 33, 64, 65, 128, 129):
        s, i = score(b)
        np.testing.assert_array_equal(i, all_i[:b])
        np.testing.assert_array_equal(s.view(np.uint32), all_s[:b].view(np.uint32))


@pytest.mark.parametrize("n,k", [(40, 10), (2_501, 20)])
def test_f32_infinite_and_nan_rows(n, k):
    # a NaN score is never ranked; infinities are, in their places
    d, nu = 32, 3
    keys = np.arange(nu, dtype=np.int64)
    q, c = np.abs(_rows(nu, d, 205)) + 0.1, _rows(n, d, 206)
    c[5] = np.nan
    c[9] = np.inf
    c[11] = -np.inf
    c[13, 0], c[13, 1] = np.inf, -np.inf  # NaN sum
    m = run_merge(keys, q, c, k)
    s, i = m.topk_score[:nu].cpu().numpy(), m.topk_index[:nu].cpu().numpy()
    finite = np.setdiff1d(np.arange(n), [5, 9, 11, 13])
    for u in range(nu):
        assert i[u][0] == 9 and np.isposinf(s[u][0])
        exact = c[finite].astype(np.float64) @ q[u].astype(np.float64)
        order = finite[np.argsort(-exact, kind="stable")][:k - 1]
        np.testing.assert_array_equal(i[u][1:], order)


def _score_ms(requests, nu, n, d, k, runs=5):
    """Shortest of a few hs_score_topk calls on nu distinct queries, in ms."""
    import paper_2607_22578_amd as hs
    m = hs.MergedRetrieval(requests, d, n, k, hs.HS_F32, hs.HS_F32, device=device())
    g = torch.Generator(device=device())
    g.manual_seed(n)
    q, c = (torch.randn(r, d, device=device(), generator=g) for r in (nu, n))
    m.q_unique[:nu].copy_(q)
    best = float("inf")
    for _ in range(runs):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        hs.hs_score_topk(m.plan, m.q_unique, nu, None, c, None, m.topk_score, m.topk_index, m.ws)
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b))
    return best, m.topk_index[:nu].cpu().numpy()


@pytest.mark.parametrize("requests,nu,k", [(8_192, 100, 40), (8_192, 300, 40), (32_768, 400, 10),
                                           (200_000, 500, 10)])
def test_f32_many_requests_few_distinct_run_like_the_distinct_alone(requests, nu, k):
    # the slices follow from the distinct queries, not from the plan's requests (which
    # left 8 to 64 of the workgroups with work and took 3 to 30 times as long)
    note(f"fp32 R={requests} n_u={nu} k={k}")
    alone, want = _score_ms(nu, nu, 100_000, 128, k)
    many, got = _score_ms(requests, nu, 100_000, 128, k)
    np.testing.assert_array_equal(got, want)
    assert many < 1.5 * alone + 0.03, f"{many * 1e3:.0f} us, alone {alone * 1e3:.0f} us"


# plans whose lists leave room for a few slices only, for the thresholds but no tiled
# queries, for neither (fewer than four keys per list: the maxima would not fit), and
# for a slice per query, in the 64 MiB of the allocation-free entry point; the same
# plans with a workspace of their own, scored in two orders of the calls
@pytest.mark.parametrize("requests,nu,n,d,k", [
    (8_192, 90, 20_011, 64, 40), (100_000, 140, 20_011, 1_024, 10), (2_100_000, 70, 9_001, 32, 3),
    (8_000, 300, 9_001, 36, 1_000), (200_000, 1_500, 9_001, 32, 33),
])
def test_f32_plans_with_little_room(requests, nu, n, d, k):
    import paper_2607_22578_amd as hs
    note(f"fp32 R={requests} n_u={nu} N={n} d={d} k={k}")
    q, c = _rows(nu, d, 207), _rows(n, d, 208)
    dev = device()
    plan = hs.hs_merge_plan(requests, d, n, k, hs.HS_F32, hs.HS_F32)
    ws = torch.full((plan.workspace_bytes,), 0xA5, dtype=torch.uint8, device=dev)
    qd, cd = to_dev(q), to_dev(c)
    nu_dev = torch.tensor([nu], dtype=torch.int64, device=dev)

    class Out:
        pass

    ref = {"n_unique": nu, "first_index": np.arange(nu, dtype=np.int32)}
    for noalloc, count in ((True, nu), (False, nu), (False, -1), (True, -1)):
        m = Out()
        m.topk_score = torch.full((nu, k), 7.0, device=dev)
        m.topk_index = torch.full((nu, k), -7, dtype=torch.int32, device=dev)
        args = (plan, qd, count, nu_dev, cd, None, m.topk_score, m.topk_index)
        if noalloc:
            hs.hs_score_topk_noalloc(*args)
        else:
            hs.hs_score_topk(*args, ws)
        torch.cuda.synchronize()
        check_unique_topk(m, ref, q, c, k, sel=np.unique(np.linspace(0, nu - 1, 24).astype(int)))
