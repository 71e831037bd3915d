"""An update that finds no room for its codes fails with NOMEM, and with that
alone: its own sketches' state and the calls after it are what they were."""
import numpy as np
import pytest
import torch

import oracle
from paper_1803_11449_amd import ddhf
from test_gpu_parity import assert_spl_equal, make_sketch, say
from test_gpu_restore_launches import hosts_sketch

pytestmark = pytest.mark.gpu

LEFT = 128 << 20                     # bytes left free; the codes take 860 MiB a job


def refused(fn):
    """fn() on a device whose memory is taken, which it must refuse."""
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    free = torch.cuda.mem_get_info()[0]
    hog = torch.empty(free - LEFT, dtype=torch.uint8, device="cuda:0")
    say(f"{free >> 20} MiB free, all but {LEFT >> 20} taken")
    with pytest.raises(ddhf.SketchError) as e:
        fn()
    assert e.value.code == -2
    del hog
    torch.cuda.empty_cache()


def test_the_next_call_does_not_report_it():
    p = oracle.Params(1024, 16, 5, 6)
    words = hosts_sketch(p, 50, 6)
    want = oracle.restore(p, words, 700.0, mode="brute")[:3]
    pairs = torch.zeros((64 << 20, 2), dtype=torch.int32, device="cuda:0")
    with make_sketch(p) as sk, make_sketch(p) as other:
        other.upload(words)
        sk.set_option(ddhf.SKETCH_OPT_TRIM_POOLS, 0)
        refused(lambda: sk.update(pairs))
        assert_spl_equal(other.restore(700.0)[0], *want)


@pytest.mark.parametrize("reset", [False, True])
def test_the_sketch_is_what_it_was(reset):
    """Also what a reset made of it, and zero counts that were stale before."""
    p = oracle.Params(1024, 16, 5, 6)
    words = hosts_sketch(p, 50, 6)
    want = oracle.restore(p, words, 700.0, mode="brute")[:3]
    pairs = torch.zeros((64 << 20, 2), dtype=torch.int32, device="cuda:0")
    with make_sketch(p) as sk, make_sketch(p) as other:
        for s in (sk, other):
            s.reset()
            s.update(pairs[:50_000])                # zero counts of other words
            s.upload(words)
            if reset:
                s.reset()
        sk.set_option(ddhf.SKETCH_OPT_TRIM_POOLS, 0)
        refused(lambda: ddhf.update_batch([(other, pairs), (sk, pairs)]))
        for s in (sk, other):
            recs, info = s.restore(700.0)
            if reset:
                assert len(recs) == 0 and not any(info["he_count"])
            else:
                assert_spl_equal(recs, *want)
            assert np.array_equal(s.download(), words * 0 if reset else words)
        sk.reset()
        sk.update(pairs[:100])
        assert np.array_equal(sk.download(),
                              oracle.build_sketch(p, np.zeros((100, 2), np.uint32)))
