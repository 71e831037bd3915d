"""The update's kernels for small sketches and small windows (whole tiles
built from every pair, and batches written in order with a directory of
runs), against the oracle bit for bit: the window sizes at which the path or
the batch changes, tiles of every cut, LEs larger than a tile, a repeat-heavy
source, updates on top of a written sketch, pairs off a 16-byte boundary,
and several jobs in one launch. The zero counts that these updates keep are
checked through ZR(i) and the reported list."""
import numpy as np
import pytest
import torch

import oracle
from paper_1803_11449_amd import ddhf
from test_gpu_parity import (assert_not_boundary, assert_spl_equal, make_sketch,
                             rand_pairs, say, to_dev)

pytestmark = pytest.mark.gpu

REPEAT = 0x0A0B0C0D


def skewed(rng, n, share=0.3):
    """n pairs, a share of them from one source (more than its LE has bits)."""
    pairs = rand_pairs(rng, n, max(1, n // 25))
    pairs[rng.random(n) < share, 0] = REPEAT
    return pairs


def zeros_per_row(p, words):
    ones = np.unpackbits(words.view(np.uint8)).reshape(p.r, -1).sum(1)
    return [int(p.g * 2**p.k - o) for o in ones]


def check(p, sk, ref, theta=None):
    torch.cuda.synchronize()
    assert np.array_equal(sk.download(), ref)
    theta = theta or 0.7 * p.g
    recs, info = sk.restore(theta)
    assert info["zr"][:p.r] == zeros_per_row(p, ref)
    ip, sz, c, _ = oracle.restore(p, ref, theta)
    assert_not_boundary(info)
    assert_spl_equal(recs, ip, sz, c)


@pytest.mark.parametrize("n", [1, 63, 1024, 4097, 24_575, 24_576, 262_143, 524_287, 524_288,
                               1_048_575, 1_048_576, 1_572_864, 3_000_001])
def test_window_sizes_around_the_path_changes(n):
    say(f"small window n={n}")
    p = oracle.Params()
    rng = np.random.default_rng(n)
    pairs = skewed(rng, n)
    ref = oracle.build_sketch(p, pairs)
    with make_sketch(p) as sk:
        sk.update(to_dev(skewed(rng, 30_000)))      # stale contents
        sk.reset()
        sk.update(to_dev(pairs))
        check(p, sk, ref)
        # on top of a written sketch, 8 bytes past a 16-byte boundary
        more = skewed(rng, n)
        sk.update(to_dev(np.concatenate([more[:1], more]))[1:])
        check(p, sk, oracle.build_sketch(p, np.concatenate([pairs, more])))


# 160 KiB tiles cut 0 to 4 times (k = 16 at r = 5, g = 1024 is the largest
# sketch of this path), LEs across the edge of a cut tile, LEs without kept zero
# counts, every r
SHAPES = [(1024, 16, 5, 6), (1024, 15, 5, 6), (512, 14, 6, 5), (256, 12, 7, 4), (128, 10, 8, 4),
          (32, 14, 5, 6), (65536, 8, 5, 8), (16384, 11, 4, 11), (65536, 5, 8, 5), (4096, 12, 5, 7), (512, 16, 3, 16)]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "g%dk%dr%da%d" % s)
@pytest.mark.parametrize("n", [5_000, 60_001, 1_100_003])
def test_sketch_shapes(shape, n):
    p = oracle.Params(*shape)
    say(f"small window shape={shape} n={n}")
    n = min(n, int(0.6 * p.g * 2**p.k))
    rng = np.random.default_rng(n + p.k)
    pairs = skewed(rng, n)
    ref = oracle.build_sketch(p, pairs)
    with make_sketch(p) as sk:
        sk.reset()
        sk.update(to_dev(pairs))
        torch.cuda.synchronize()
        assert np.array_equal(sk.download(), ref)
        assert sk.restore(3.0 * p.g)[1]["zr"][:p.r] == zeros_per_row(p, ref)


# the region kernels at every r (sketches over the linear path's 40 MiB)
@pytest.mark.parametrize("shape", [(1024, 17, 4, 8), (1024, 17, 6, 4), (2048, 16, 8, 3)],
                         ids=lambda s: "g%dk%dr%da%d" % s)
def test_region_update_of_every_r(shape):
    p = oracle.Params(*shape)
    say(f"regions shape={shape}")
    rng = np.random.default_rng(p.r)
    pairs = skewed(rng, 1_500_001)
    with make_sketch(p, 2) as sk:
        sk.reset()
        sk.update(to_dev(pairs))
        torch.cuda.synchronize()
        assert np.array_equal(sk.download(), oracle.build_sketch(p, pairs))


@pytest.mark.parametrize("large", [False, True], ids=["linear", "joins-regions"])
def test_batches_of_small_and_large_jobs(large):
    """Linear, fresh and direct jobs in one call, twice (the second time on
    written sketches); with a sketch of the region path in the call the
    linear jobs take that path too."""
    say(f"batch large={large}")
    rng = np.random.default_rng(5 + large)
    specs = [(oracle.Params(), 700_000), (oracle.Params(1024, 16, 5, 6), 2_000_001),
             (oracle.Params(256, 12, 5, 7), 90_000), (oracle.Params(), 5_000),
             (oracle.Params(), 30_001)]
    if large:
        specs.append((oracle.Params(1024, 18, 5, 5), 1_000_000))
    sks = [make_sketch(p) for p, _ in specs]
    try:
        for sk in sks:
            sk.update(to_dev(rand_pairs(rng, 50_000, 2_000)))
            sk.reset()
        data = [np.zeros((0, 2), np.uint32) for _ in specs]
        for rep in range(2):
            new = [skewed(rng, n) for _, n in specs]
            data = [np.concatenate([d, x]) for d, x in zip(data, new)]
            ddhf.update_batch([(sk, to_dev(x)) for sk, x in zip(sks, new)])
            for sk, (p, _), d in zip(sks, specs, data):
                check(p, sk, oracle.build_sketch(p, d), 0.8 * p.g)
    finally:
        for sk in sks:
            sk.close()
