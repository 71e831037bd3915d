"""Which way the lattice search went (sketch_timings: pairs) on both sides of
the rule between the walk and the pair index, and that the index's buckets
that no record holds are among those that the searches met."""
import numpy as np
import pytest

import oracle
from paper_1803_11449_amd import ddhf
from test_gpu_pair_index import walks_from
from test_gpu_parity import make_sketch, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k,alpha,r", [(13, 7, 5), (14, 6, 5), (14, 9, 4), (15, 6, 5), (16, 8, 4),
                                       (16, 6, 8), (17, 5, 5), (18, 7, 4), (19, 7, 4)])
@pytest.mark.parametrize("share,by_pairs", [(0.01, True), (0.9, True), (1.1, False)])
def test_the_way_taken(k, alpha, r, share, by_pairs):
    p = oracle.Params(64, k, r, alpha)
    h = max(1, min(int(share * walks_from(k)), 2**k - 1))
    rng = np.random.default_rng(k)
    words = np.zeros((r, 1 << k, p.g // 32), np.uint32)
    for row in range(r):
        n = h if row < 2 else min(2**k - 1, 400)
        words[row, 1 + rng.choice(2**k - 1, size=n, replace=False)] = 0xFFFFFFFF
    words = words.reshape(-1)
    with make_sketch(p) as sk:
        sk.set_option(ddhf.SKETCH_OPT_CANDIDATES, 2)
        sk.set_option(ddhf.SKETCH_OPT_TIMING, 1)
        sk.upload(words)
        got = sk.candidates(40.0)
        t = ddhf.sketch_timings(sk.handle)
    say(f"k={k} {h} hot row-1 LEs: {t['pairs']} pairs")
    assert t["search"] == 2 and t["lattice_points"] == h << (32 - k)
    assert t["pairs"] == (h * h if by_pairs and 14 <= k <= 18 else 0)
    assert np.array_equal(got, oracle.candidates(p, words, 40.0, "brute"))


@pytest.mark.parametrize("k,alpha", [(15, 6), (16, 6), (17, 5), (18, 5)])
def test_buckets_that_no_record_holds(k, alpha):
    """All of the pairs go through buckets whose parts exceed a record's, where
    the hash family has enough of them."""
    held = 6 if k == 15 else 4
    span = 4 if k == 15 else 1
    n = 2 ** (32 - k)
    for seed in range(64):
        p = oracle.Params(64, k, 5, alpha, seed=(seed * 0x9E3779B97F4A7C15 + 12345) % 2**64)
        a0, b0 = (int(x) for x in oracle.hash_coeffs(p.seed)[:2])
        z = np.arange(n, dtype=np.uint64)
        cnt = np.bincount((((z * np.uint64(a0)) << np.uint64(k)) >> np.uint64(32 + k))
                          .astype(np.int64), minlength=n)
        wrap = np.concatenate([cnt, cnt[:span]])
        over = sum(wrap[i:i + n] for i in range(span + 1)) > held
        # hot row-1 LEs of one hot row-0 LE whose pair starts in such a bucket
        c0 = 5
        low = np.arange(2**k, dtype=np.uint64)
        at = np.uint64((c0 << (64 - k)) - b0 & (2**64 - 1)) - np.uint64(a0) * low
        hit = over[(at >> np.uint64(32 + k)).astype(np.int64)]
        if hit.sum() >= 800:
            break
    assert hit.sum() >= 800, "no hash family of 64 has such buckets"
    some = np.random.default_rng(k).choice(low[hit], size=min(800, int(hit.sum())), replace=False)
    cells = c0 ^ some.astype(np.int64)
    words = np.zeros((p.r, 1 << k, p.g // 32), np.uint32)
    words[0, c0] = 0xFFFFFFFF
    words[1, cells] = 0xFFFFFFFF
    words[2:, 1:] = 0xFFFFFFFF
    words = words.reshape(-1)
    with make_sketch(p) as sk:
        sk.set_option(ddhf.SKETCH_OPT_CANDIDATES, 2)
        sk.set_option(ddhf.SKETCH_OPT_TIMING, 1)
        sk.upload(words)
        got = sk.candidates(40.0)
        t = ddhf.sketch_timings(sk.handle)
    want = oracle.candidates(p, words, 40.0, "brute")
    say(f"k={k} seed {seed}: {hit.sum()} such pairs, {t['pairs']} gone through, {len(want)} found")
    assert len(want) > 10 and t["pairs"] == len(cells) and np.array_equal(got, want)
