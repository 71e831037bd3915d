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
