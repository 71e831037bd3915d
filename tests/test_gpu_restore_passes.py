"""How many times a call runs the restore: kernels counted by the profiler. A
restore launched by what the last one found, and wrong, runs again; that must
not happen to a caller whose windows do not change."""
import time
from collections import Counter

import pytest
import torch
from torch.profiler import ProfilerActivity, profile

import oracle
from paper_1803_11449_amd import ddhf
from test_gpu_parity import assert_spl_equal, make_sketch, say
from test_gpu_restore_launches import hosts_sketch

pytestmark = pytest.mark.gpu


def kernels(fn):
    """(fn's result, launches by kernel name) of one call."""
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        # the profiler drops kernels near its ends (its two clocks differ)
        time.sleep(0.05)
        out = fn()
        torch.cuda.synchronize()
        time.sleep(0.05)
    n = Counter()
    for e in prof.key_averages():
        if "ddhf::" in e.key:
            n[e.key.split("ddhf::")[1].split("(")[0].split("<")[0]] += e.count
    return out, n


@pytest.mark.parametrize("m", [1000, 3000])
def test_candidates_between_restores(m):
    """The candidate list has no records, which says nothing of the next
    restore's."""
    p = oracle.Params(128, 18, 5, 5)
    words = hosts_sketch(p, m, m)
    want = oracle.restore(p, words, 100.0, mode="brute")[:3]
    with make_sketch(p) as sk:
        sk.upload(words)
        for i in range(4):
            sk.candidates(100.0)
            (recs, _), n = kernels(lambda: sk.restore(100.0))
            say(f"{m} records after the candidates, time {i}: {dict(n)}")
            assert_spl_equal(recs, *want)
            assert n["k_estimate"] == 1


def test_a_join_that_outgrows_the_fixed_array():
    """A join of one block, whose partial addresses do not fit the no-alloc
    restore's array: the join and the lattice search, two passes a call, and
    one for a restore that has the buffers."""
    p = oracle.Params(128, 18, 5, 5)
    words = hosts_sketch(p, 300, 1)
    want = oracle.restore(p, words, 100.0, mode="brute")[:3]
    with make_sketch(p) as sk:
        sk.set_option(ddhf.SKETCH_OPT_JOIN_BLOCKS, 1)
        sk.upload(words)
        for _ in range(2):
            sk.restore(100.0)                # the pools grow
        for i in range(4):
            (recs, _), n = kernels(lambda: sk.restore_noalloc(100.0))
            say(f"no-alloc join, time {i}: {dict(n)}")
            assert_spl_equal(recs, *want)
            assert n["k_compact"] == 2 and n["k_join"]
        (recs, info), n = kernels(lambda: sk.restore(100.0))
        assert_spl_equal(recs, *want)
        assert n["k_compact"] == 1 and info["n_partials"][2] > 2560
