"""How many times a call runs the restore: kernels counted by the profiler. A
restore launched by what the last one found, and wrong, runs again; that must
not happen to a caller whose windows do not change."""
import time
from collections import Counter

import numpy as np
import pytest
import torch
from torch.profiler import ProfilerActivity, profile

import oracle
from paper_1803_11449_amd import ddhf
from test_gpu_parity import assert_spl_equal, crafted_hot_sketch, make_sketch, say
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


def kinds_in_turn(what):
    """(parameters, theta, windows whose restores need other kernels)."""
    if what == "search":
        p, theta = oracle.Params(), 700.0
        windows = [crafted_hot_sketch(p, f, 3) for f in (0.002, 0.06)]
    else:
        p, theta = oracle.Params(128, 18, 5, 5), 100.0
        windows = [hosts_sketch(p, m, m) for m in (1000, 2500)]
    return p, theta, [(w, oracle.restore(p, w, theta, mode="brute")[:3]) for w in windows]


@pytest.mark.parametrize("fn", ["restore", "restore_noalloc", "batch"])
@pytest.mark.parametrize("what", ["search", "list"])
@pytest.mark.parametrize("each", [1, 3])
def test_windows_of_two_kinds_in_turn(what, fn, each):
    """`each` windows of a kind at a time: one restore is run again, not every
    one that follows a window of the other kind."""
    p, theta, windows = kinds_in_turn(what)
    passes = 0
    with make_sketch(p) as sk:
        sk._cap = 1 << 13
        restore = {"batch": lambda: ddhf.restore_batch([(sk, theta)])[0]}.get(
            fn, lambda: getattr(sk, fn)(theta))
        for i in range(6 * each):
            words, want = windows[i // each % 2]
            sk.upload(words)
            (recs, _), n = kernels(restore)
            assert_spl_equal(recs, *want)
            passes += n["k_estimate"]
        say(f"{what}, {fn}, {each} of a kind: {passes} passes for {6 * each} windows")
        assert passes <= 6 * each + 1
        # windows of one kind: only what they need, once that has been so for a while
        for i in range(10):
            (recs, _), n = kernels(restore)
            assert_spl_equal(recs, *want)
            assert n["k_estimate"] == 1
        searches = [x for x in ("k_lattice", "k_pairs", "k_join", "k_join_walk") if n[x]]
        assert len(searches) == 1 and (n["k_sort_publish"] == 1) == (len(want[0]) <= 1536)


@pytest.mark.parametrize("g,k,r,alpha,walk", [(128, 20, 4, 10, True), (32, 21, 4, 11, False),
                                              (32, 22, 4, 12, False)])
def test_long_joins_go_by_stage(g, k, r, alpha, walk):
    """Without the lattice search (k > 20) a join may be of long lists."""
    p = oracle.Params(g, k, r, alpha)
    words = crafted_hot_sketch(p, 0.0004, 3)
    with make_sketch(p) as sk:
        sk.set_option(ddhf.SKETCH_OPT_CANDIDATES, 1)
        sk.upload(words)
        got, n = kernels(lambda: sk.candidates(0.8 * g))
    say(f"k={k} r={r}: {dict(n)}, {len(got)} candidates")
    assert (n["k_join_walk"], n["k_join"]) == ((1, 0) if walk else (0, r - 2))
    assert np.array_equal(got, oracle.candidates(p, words, 0.8 * g, "brute"))
