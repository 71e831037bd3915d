"""Work on one sketch from the null stream and from others in turn, with the
null stream's ordering events recorded at once (a sketch's first uses, and
after a change of streams) and late (a sketch that stayed on the null stream).
Every sketch and list is compared bit for bit with the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_1803_11449_amd import ddhf
from test_gpu_parity import assert_spl_equal, make_sketch, rand_pairs, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("before", [0, 3, 4, 5, 40])
@pytest.mark.parametrize("n", [700, 60_000])
def test_null_stream_then_another(before, n):
    """before: updates on the null stream alone, before the streams change."""
    p = oracle.Params(128, 14, 5, 6)
    side = torch.cuda.Stream()
    pairs = rand_pairs(np.random.default_rng(3), n * (before + 4), 400)
    dev = to_dev(pairs)
    torch.cuda.synchronize()
    part = [dev[i * n:(i + 1) * n] for i in range(before + 4)]
    with make_sketch(p) as sk, make_sketch(p) as other, make_sketch(p) as late:
        for x in part[:before]:
            sk.update(x)
            late.update(x)
        for i in range(before, before + 4):
            sk.update(part[i], stream=None if i % 2 else side)
        words = oracle.build_sketch(p, pairs)
        other.update(dev, stream=side)
        say(f"{before} updates of {n} pairs on the null stream, 4 in turn")
        ip, sz, c, _ = oracle.restore(p, words, 6.0, mode="brute")
        for stream in (side, None, side):
            recs, _ = sk.restore(6.0, stream=stream)
            assert_spl_equal(recs, ip, sz, c)
        recs, _ = other.restore(6.0)
        assert_spl_equal(recs, ip, sz, c)
        # the host asks for a lane that was left late
        assert np.array_equal(late.download(), oracle.build_sketch(p, pairs[:before * n]))
        late.merge(sk, stream=side)
        recs, _ = ddhf.restore_batch([(late, 6.0), (other, 6.0)])[0]
        assert_spl_equal(recs, ip, sz, c)
        other.reset(stream=side)
        other.update(part[0])
        assert np.array_equal(other.download(), oracle.build_sketch(p, pairs[:n]))


def test_destroyed_after_work_that_was_left_late():
    p = oracle.Params(128, 14, 5, 6)
    pairs = rand_pairs(np.random.default_rng(5), 50_000, 3000)
    dev = to_dev(pairs)
    for _ in range(3):
        sk = make_sketch(p)
        for _ in range(8):
            sk.update(dev)
        sk.close()
    with make_sketch(p) as sk:
        sk.update(dev)
        assert np.array_equal(sk.download(), oracle.build_sketch(p, pairs))
