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
