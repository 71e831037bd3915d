"""How many times a call runs the restore: kernels counted by the profiler. A
restore launched by what the last one found, and wrong, runs again; that must
not happen to a caller whose windows do not change."""
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
        out = fn()
        torch.cuda.synchronize()
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
