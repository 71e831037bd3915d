"""Which kernels an update takes, by the sketch's size and options and the
window's: launches counted by name, the sketch compared with the oracle."""
import numpy as np
import pytest

import oracle
from paper_1803_11449_amd import ddhf
from test_gpu_parity import make_sketch, rand_pairs, say, to_dev
from test_gpu_restore_passes import kernels

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,fresh", [(100_000, True), (131_072, True), (131_073, False),
                                     (600_000, False)])
@pytest.mark.parametrize("p", [oracle.Params(1024, 5, 8, 5), oracle.Params(32, 5, 8, 5),
                               oracle.Params(1024, 9, 6, 6), oracle.Params(1024, 14, 5, 6)],
                         ids=lambda p: f"g{p.g}k{p.k}r{p.r}a{p.alpha}")
def test_a_raised_minimum(p, n, fresh):
    """SKETCH_OPT_BINNED_MIN_PAIRS above the window: a reset sketch is built
    from all its pairs only while they are few, whatever its tiles."""
    pairs = rand_pairs(np.random.default_rng(n), n, 4000)
    dev = to_dev(pairs)
    with make_sketch(p) as sk:
        sk.set_option(ddhf.SKETCH_OPT_BINNED_MIN_PAIRS, 1 << 40)
        sk.update(dev)
        sk.reset()
        _, k = kernels(lambda: sk.update(dev))
        say(f"minimum raised, {n} pairs, {p.words()} words: {dict(k)}")
        assert (k["k_update_fresh"], k["k_update"]) == ((1, 0) if fresh else (0, 1))
        assert np.array_equal(sk.download(), oracle.build_sketch(p, pairs))


@pytest.mark.parametrize("p,n,linear", [
    # 4, 12 and 32 tiles of a sketch of few
    (oracle.Params(1024, 5, 8, 5), 650_000, True), (oracle.Params(1024, 5, 8, 5), 660_000, False),
    (oracle.Params(1024, 7, 7, 5), 4_000_000, True), (oracle.Params(1024, 7, 7, 5), 4_050_000, False),
    (oracle.Params(1024, 9, 5, 8), 12_000_000, True),
    # large estimators
    (oracle.Params(2048, 13, 5, 7), 1_600_000, True),
    (oracle.Params(4096, 13, 5, 7), 1_600_000, True),
    (oracle.Params(8192, 12, 5, 7), 1_572_864, True),
    (oracle.Params(8192, 12, 5, 7), 1_572_865, False)],
    ids=lambda x: f"g{x.g}k{x.k}r{x.r}" if isinstance(x, oracle.Params) else str(x))
def test_heavy_tiles(p, n, linear):
    """A window that would leave few workgroups with long tiles goes through the
    passes that cut them; half the pairs are one source's."""
    rng = np.random.default_rng(n)
    pairs = rand_pairs(rng, n, 4000)
    pairs[rng.random(n) < 0.5, 0] = 77
    dev = to_dev(pairs)
    want = oracle.build_sketch(p, pairs)
    with make_sketch(p) as sk:
        for fresh in (True, False):
            _, k = kernels(lambda: sk.update(dev))
            say(f"{p} {n} pairs, fresh {fresh}: {dict(k)}")
            assert bool(k["k_lin_apply"]) == linear and bool(k["k_bin_apply"]) != linear
            assert np.array_equal(sk.download(), want)
        if n < 1_000_000:               # the same rounds as one update of a large window
            sk.set_option(ddhf.SKETCH_OPT_BINNED_ROUND, 100_000)
            sk.reset()
            _, k = kernels(lambda: sk.update(dev))
            assert k["k_lin_apply"] == 7 and np.array_equal(sk.download(), want)


@pytest.mark.parametrize("share", [0.0, 0.03, 0.1, 0.6])
@pytest.mark.parametrize("p", [oracle.Params(1024, 14, 5, 6), oracle.Params(2048, 13, 4, 10)],
                         ids=lambda p: f"g{p.g}k{p.k}r{p.r}")
def test_shares_of_one_source(p, share):
    """A scatter's filter that goes on past its block's second batch, or does
    not: more than three batches to each block, pairs that come again, the
    shares of one source around the line."""
    rng = np.random.default_rng(int(share * 100))
    n = 5_100_007
    pairs = rand_pairs(rng, n, 300_000)
    pairs[rng.random(n) < share, 0] = 99
    pairs[n // 2:n // 2 + n // 4] = pairs[:n // 4]
    dev = to_dev(pairs)
    want = oracle.build_sketch(p, pairs)
    with make_sketch(p) as sk:
        for fresh in (True, False):
            _, k = kernels(lambda: sk.update(dev))
            say(f"{p} share {share}, fresh {fresh}: {dict(k)}")
            assert k["k_lin_scatter"] and np.array_equal(sk.download(), want)


@pytest.mark.parametrize("p,n", [(oracle.Params(1024, 12, 5, 7), 1_500_000),
                                 (oracle.Params(16384, 9, 5, 8), 1_500_000),
                                 (oracle.Params(65536, 8, 5, 8), 1_600_000),
                                 (oracle.Params(65536, 9, 5, 8), 1_600_000),
                                 (oracle.Params(1024, 18, 5, 5), 1_600_000)],
                         ids=lambda x: f"g{x.g}k{x.k}" if isinstance(x, oracle.Params) else str(x))
@pytest.mark.parametrize("seed", [oracle.Params().seed, 5, 3])
def test_source_zero(p, n, seed):
    """The scatter's filter tells source 0 and the next sources, one of which
    stands for no owner in 0's slot, from a slot without an owner."""
    p = oracle.Params(p.g, p.k, p.r, p.alpha, seed)
    rng = np.random.default_rng(n + seed % 1000)
    pairs = rand_pairs(rng, n, 4000)
    u = rng.random(n)
    pairs[u < 0.3, 0] = 0
    near = (u > 0.3) & (u < 0.6)
    pairs[near, 0] = rng.integers(1, 64, int(near.sum()))
    pairs[-(n // 3):] = pairs[:n // 3]
    dev = to_dev(pairs)
    want = oracle.build_sketch(p, pairs)
    with make_sketch(p) as sk:
        sk.set_option(ddhf.SKETCH_OPT_SCATTER_PPT, 4)
        sk.set_option(ddhf.SKETCH_OPT_BINNED_BLOCKS, 40)
        for _ in range(2):
            _, k = kernels(lambda: sk.update(dev))
            say(f"{p} {n} pairs: {dict(k)}")
            assert k["k_lin_scatter"] or k["k_bin_scatter"]
            assert np.array_equal(sk.download(), want)


@pytest.mark.parametrize("k,alpha,n,reset,written", [
    (14, 6, 24_575, "k_update_fresh", "k_update"), (14, 6, 24_576, "linear", "linear"),
    (16, 6, 24_576, "linear", "k_update"), (16, 6, 40_959, "linear", "k_update"),
    (16, 6, 40_960, "linear", "linear")])
def test_small_updates(k, alpha, n, reset, written):
    """Few further pairs are set one by one rather than by rewriting a written
    sketch, more of them the larger it is."""
    p = oracle.Params(1024, k, 5, alpha)
    pairs = rand_pairs(np.random.default_rng(n), 2 * n, 4000)
    with make_sketch(p) as sk:
        sk.reset()
        for dev, name in ((to_dev(pairs[:n]), reset), (to_dev(pairs[n:]), written)):
            _, kern = kernels(lambda: sk.update(dev))
            say(f"k={k}, {n} pairs: {dict(kern)}")
            assert set(kern) == ({"k_lin_scatter", "k_lin_apply"} if name == "linear" else {name})
        assert np.array_equal(sk.download(), oracle.build_sketch(p, pairs))
