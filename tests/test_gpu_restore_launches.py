"""The restore's shorter launch chains against the oracle: the scans of small
and large sketches (from kept and from counted zeros), the join as one walk,
the one-launch sort at its limit, and restores launched by what the sketch's
last restore found when the next one needs something else (the other search,
the long sort). Integers are compared bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from paper_1803_11449_amd import ddhf
from test_gpu_parity import assert_spl_equal, crafted_hot_sketch, make_sketch, rand_pairs, say, to_dev

pytestmark = pytest.mark.gpu


def hosts_sketch(p, m, seed):
    """A sketch in which m random hosts have every bit of their LEs set."""
    rng = np.random.default_rng(seed)
    hosts = rng.choice(2**32, size=m, replace=False).astype(np.uint32)
    pairs = np.stack([hosts, np.zeros(m, np.uint32)], 1)
    words = oracle.build_sketch(p, pairs).reshape(-1, p.g // 32) if m else \
        np.zeros((p.words() // (p.g // 32), p.g // 32), np.uint32)
    words[words.any(axis=1)] = 0xFFFFFFFF
    return words.reshape(-1)


def zeros_per_row(p, words):
    ones = np.unpackbits(words.view(np.uint8)).reshape(p.r, -1).sum(1)
    return [int(p.g * 2**p.k - o) for o in ones]


def test_lists_around_the_one_launch_sort():
    """Each sketch is restored twice at one threshold: the first restore goes
    by the sketch before it (another list length), the second by itself."""
    p = oracle.Params(128, 18, 5, 5)
    with make_sketch(p) as sk:
        for m in (0, 1, 2, 3, 64, 65, 1536, 2047, 2048, 2049, 5, 2100, 1, 9000):
            words = hosts_sketch(p, m, m + 7)
            ip, sz, c, _ = oracle.restore(p, words, 100.0, mode="brute")
            say(f"one-launch sort: {m} hosts, {len(ip)} records")
            sk.upload(words)
            for _ in range(2):
                recs, info = sk.restore(100.0)
                assert info["n_reported"] == len(ip)
                assert_spl_equal(recs, ip, sz, c)
                again, _ = sk.restore_noalloc(100.0)
                assert np.array_equal(again, recs)


def test_expected_search_turns_out_the_other():
    """Sketches that call for the join and for the lattice search in turn, at
    one threshold: eager, without allocation, batched, and in a plan."""
    p = oracle.Params()
    theta = 700.0
    words = [crafted_hot_sketch(p, f, 3 + i) for i, f in enumerate((0.002, 0.06, 0.003, 0.05))]
    refs = [oracle.restore(p, w, theta, mode="brute") for w in words]
    with make_sketch(p) as sk, make_sketch(p) as other:
        other.upload(words[0])
        searches = set()
        sk.set_option(ddhf.SKETCH_OPT_TIMING, 1)
        for rep in range(2):
            for w, (ip, sz, c, _) in zip(words, refs):
                sk.upload(w)
                recs, _ = sk.restore(theta)
                assert_spl_equal(recs, ip, sz, c)
                searches.add(ddhf.sketch_timings(sk.handle)["search"])
        assert searches == {1, 2}
        sk.set_option(ddhf.SKETCH_OPT_TIMING, 0)
        for fn in (sk.restore_noalloc, lambda th: ddhf.restore_batch([(sk, th), (other, th)])[0]):
            for w, (ip, sz, c, _) in zip(words, refs):
                say(f"expected search, {len(ip)} records")
                sk.upload(w)
                assert_spl_equal(fn(theta)[0], ip, sz, c)
                assert np.array_equal(sk.candidates(theta), oracle.candidates(p, w, theta, "brute"))
        # a plan without a reset restores the sketch as it is
        empty = torch.zeros((0, 2), dtype=torch.int32, device="cuda:0")
        with ddhf.Plan([(sk, empty, theta), (other, empty, theta)], reset=False) as plan:
            for rep in range(3):
                for w, (ip, sz, c, _) in zip(words, refs):
                    sk.upload(w)
                    plan.run()
                    res = plan.results()
                    assert_spl_equal(res[0][0], ip, sz, c)
                    assert_spl_equal(res[1][0], *refs[0][:3])
                    torch.cuda.synchronize()


@pytest.mark.parametrize("blocks", [0, 1])
@pytest.mark.parametrize("frac", [0.0005, 0.004, 0.02])
@pytest.mark.parametrize("p", [oracle.Params(128, 14, 5, 6), oracle.Params(128, 14, 4, 9),
                               oracle.Params(256, 12, 6, 5), oracle.Params(512, 14, 7, 4),
                               oracle.Params(128, 10, 8, 4), oracle.Params(128, 16, 3, 16)],
                         ids=lambda p: f"g{p.g}k{p.k}r{p.r}a{p.alpha}")
def test_join_walk(p, frac, blocks):
    """The walk's candidates equal the brute force, and its partial addresses
    per stage the staged join's (which the call without allocation keeps)."""
    say(f"join walk g={p.g} k={p.k} r={p.r} frac={frac} blocks={blocks}")
    words = crafted_hot_sketch(p, frac, p.k + p.r)
    hosts = hosts_sketch(p, 30, 5)                      # at least 30 candidates
    words |= hosts
    theta = 0.9 * p.g
    with make_sketch(p) as sk:
        sk.set_option(ddhf.SKETCH_OPT_CANDIDATES, 1)
        sk.set_option(ddhf.SKETCH_OPT_JOIN_BLOCKS, blocks)
        sk.upload(words)
        cand = sk.candidates(theta)
        recs, info = sk.restore(theta)
        sk.set_option(ddhf.SKETCH_OPT_JOIN_BLOCKS, 0)       # room for the staged partials
        staged, sinfo = sk.restore_noalloc(theta)
    assert len(cand) >= 30
    assert np.array_equal(cand, oracle.candidates(p, words, theta, "brute"))
    assert np.array_equal(recs, staged)
    assert info["n_partials"] == sinfo["n_partials"] and (p.r == 3) == (info["n_partials"][2] == 0)


def test_join_walk_reads_large_tables_where_they_are():
    """Hot lists of rows 2.. too long for the walk's LDS tables."""
    p = oracle.Params(128, 14, 4, 9)
    say("join walk, global tables")
    words = crafted_hot_sketch(p, 0.45, 5).reshape(p.r, 1 << p.k, -1)
    sparse = crafted_hot_sketch(p, 0.002, 6).reshape(p.r, 1 << p.k, -1)
    words[:2] = sparse[:2]
    words = words.reshape(-1)
    with make_sketch(p) as sk:
        sk.set_option(ddhf.SKETCH_OPT_CANDIDATES, 1)
        sk.upload(words)
        cand = sk.candidates(100.0)
        _, info = sk.restore(100.0)
    assert min(info["he_count"][2:4]) > 4096
    assert np.array_equal(cand, oracle.candidates(p, words, 100.0, "brute"))


@pytest.mark.parametrize("p", [oracle.Params(128, 5, 8, 5), oracle.Params(8192, 8, 6, 7),
                               oracle.Params(1024, 11, 5, 8), oracle.Params(256, 16, 5, 6),
                               oracle.Params(128, 17, 5, 5), oracle.Params(128, 19, 5, 5),
                               oracle.Params(64, 17, 5, 5)],
                         ids=lambda p: f"g{p.g}k{p.k}r{p.r}a{p.alpha}")
def test_scans(p):
    """ZR(i), |HE(i)| and the list from the zero counts that an update kept
    and, after a direct update, from counting them in the sketch."""
    say(f"scan g={p.g} k={p.k} r={p.r} alpha={p.alpha}")
    rng = np.random.default_rng(p.k)
    n = min(400_000, int(0.3 * p.g * 2**p.k))
    pairs = rand_pairs(rng, n, max(1, n // 300))
    theta = 0.37 * p.g + 0.123
    with make_sketch(p) as sk:
        sk.reset()
        sk.update(to_dev(pairs))
        for step in range(2):
            ref = oracle.build_sketch(p, pairs)
            ones = np.unpackbits(ref.view(np.uint8)).reshape(p.r, 1 << p.k, p.g).sum(2)
            hot = p.g - ones < p.g * np.exp(-theta / p.g)
            recs, info = sk.restore(theta)
            assert info["zr"][:p.r] == zeros_per_row(p, ref)
            assert info["he_count"][:p.r] == hot.sum(1).tolist()
            ip, sz, c, _ = oracle.restore(p, ref, theta, mode="brute")
            assert_spl_equal(recs, ip, sz, c)
            more = rand_pairs(rng, 2_000, 50)
            sk.set_option(ddhf.SKETCH_OPT_UPDATE_PATH, 1)
            sk.update(to_dev(more))
            pairs = np.concatenate([pairs, more])


@pytest.mark.parametrize("k,alpha,path,blocks,frac,m",
                         [(14, 6, 2, 0, 0.17, 0)] +
                         [(k, a, 1, 1, 0.0, m) for k, a in ((14, 6), (18, 5))
                          for m in (512, 513, 700)])
def test_candidates_past_the_block_buffer(k, alpha, path, blocks, frac, m):
    """A search block keeps its first 512 candidates until it ends; the rest
    go out one by one. k = 14 joins in one walk, k = 18 in stages; the crafted
    sketch's lattice search finds more than 512 per block."""
    p = oracle.Params(128, k, 5, alpha)
    words = crafted_hot_sketch(p, frac, 11) if frac else hosts_sketch(p, m, 17)
    say(f"candidates: k={p.k} path={path} frac={frac} hosts={m}")
    with make_sketch(p) as sk:
        sk.set_option(ddhf.SKETCH_OPT_CANDIDATES, path)
        sk.set_option(ddhf.SKETCH_OPT_JOIN_BLOCKS, blocks)
        sk.upload(words)
        cand = sk.candidates(100.0)
        recs, _ = sk.restore(100.0)
    want = oracle.candidates(p, words, 100.0, "brute")
    assert len(want) >= (500_000 if frac else m)
    assert np.array_equal(cand, want) and np.array_equal(recs["ip"], want)
