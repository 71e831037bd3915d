"""The lattice search's two ways through the hot row-0 cells, the walk and the
pair index, around the rule between them and at the ends of the range of k
that has an index, against every address the oracle finds."""
import numpy as np
import pytest

import oracle
from paper_1803_11449_amd import ddhf
from test_gpu_parity import assert_spl_equal, make_sketch, say

pytestmark = pytest.mark.gpu


def walks_from(k):
    """|HE(1)| from which the walk's addresses are fewer than the pairs' work."""
    return 2 ** (32 - k) / (15 if k >= 16 else 20 if k == 15 else 98)


@pytest.mark.parametrize("k,alpha,r", [(13, 7, 5), (14, 6, 5), (14, 9, 4), (15, 6, 5), (16, 8, 4),
                                       (16, 6, 8), (17, 5, 5), (18, 7, 4), (19, 7, 4)])
@pytest.mark.parametrize("share", [0.0, 0.01, 0.9, 1.1])
def test_candidates_around_the_rule(k, alpha, r, share):
    """share: row 1's hot cells over the number at which the rule turns; the
    rows past it as hot as leaves about 2000 candidates."""
    p = oracle.Params(64, k, r, alpha)
    f = min(share * walks_from(k) / 2 ** k, 1.0)
    rest = min(1.0, (2000 / (2 ** 32 * f * f)) ** (1 / (r - 2))) if f else 0.0
    rng = np.random.default_rng(11 * k + int(10 * share))
    hot = rng.random((r, 1 << k)) < np.array([f, f] + [rest] * (r - 2))[:, None]
    words = np.zeros((r, 1 << k, p.g // 32), np.uint32)
    words[hot] = 0xFFFFFFFF
    words[:, 0] = 0                      # no row without a zero bit
    words = words.reshape(-1)
    theta = 40.0
    say(f"pair index k={k} alpha={alpha} r={r}, {f:.4f}, {rest:.4f} of the cells hot")
    with make_sketch(p) as sk:
        sk.set_option(ddhf.SKETCH_OPT_CANDIDATES, 2)
        sk.upload(words)
        assert np.array_equal(sk.candidates(theta), oracle.candidates(p, words, theta, "brute"))
        ip, sz, c, _ = oracle.restore(p, words, theta, mode="brute")
        for fn in (sk.restore, sk.restore_noalloc):
            assert_spl_equal(fn(theta)[0], ip, sz, c)
        sk.set_option(ddhf.SKETCH_OPT_CANDIDATES, 0)
        assert_spl_equal(sk.restore(theta)[0], ip, sz, c)


@pytest.mark.parametrize("k,alpha,r", [(14, 6, 5), (15, 6, 5), (16, 6, 5), (17, 5, 5), (18, 5, 5)])
@pytest.mark.parametrize("seed", [0, 1, 2, 3, 4, 5])
def test_uneven_buckets(k, alpha, r, seed):
    """Other hashes: buckets with more parts than a record holds, and fewer."""
    p = oracle.Params(64, k, r, alpha, seed=(seed * 0x9E3779B97F4A7C15 + 12345) % 2 ** 64)
    h = int(min(0.4 * walks_from(k), 1500))
    rng = np.random.default_rng(seed)
    words = np.zeros((r, 1 << k, p.g // 32), np.uint32)
    rest = (500 / (2 ** 32 * (h / 2 ** k) ** 2)) ** (1 / (r - 2))
    for row in range(r):
        n = h if row < 2 else int(min(1.0, rest) * 2 ** k)
        words[row, rng.choice(2 ** k, size=n, replace=False)] = 0xFFFFFFFF
    words = words.reshape(-1)
    a0 = int(oracle.hash_coeffs(p.seed)[0])
    z = np.arange(2 ** (32 - k), dtype=np.uint64)
    parts = np.bincount((((z * np.uint64(a0)) << np.uint64(k)) >> np.uint64(32 + k)).astype(np.int64))
    say(f"uneven buckets k={k} seed {seed}: up to {parts.max()} parts in a bucket")
    with make_sketch(p) as sk:
        sk.set_option(ddhf.SKETCH_OPT_CANDIDATES, 2)
        sk.upload(words)
        assert np.array_equal(sk.candidates(40.0), oracle.candidates(p, words, 40.0, "brute"))
