"""Restores that the caller collects later (a begun batch, a plan's run) while
their sketches are reset and updated for the next window meanwhile: every list
is the begun window's, compared with the oracle, and the next window is not
disturbed."""
import numpy as np
import pytest
import torch

import oracle
from paper_1803_11449_amd import ddhf
from test_gpu_parity import assert_spl_equal, crafted_hot_sketch, make_sketch, rand_pairs, say, to_dev
from test_gpu_restore_launches import hosts_sketch

pytestmark = pytest.mark.gpu

EMPTY = np.zeros((0, 2), np.uint32)


def crafted(what):
    """(parameters, theta, a window of one kind, a window of the other): hot
    lists for the join and for the lattice search, or lists that the one-launch
    sort takes and that it does not."""
    if what.startswith("search"):
        p, theta = oracle.Params(), 700.0
        kinds = [crafted_hot_sketch(p, f, 3) for f in (0.002, 0.06)]
    else:
        p, theta = oracle.Params(128, 18, 5, 5), 100.0
        kinds = [hosts_sketch(p, m, m) for m in (1000, 2500)]
    return (p, theta, *(kinds if what.endswith("up") else kinds[::-1]))


def next_window(sk, p, meanwhile, words, stream=None):
    """What the caller does before it collects; the sketch it then expects."""
    pairs = rand_pairs(np.random.default_rng(9), 3000 if meanwhile == "small" else 200_000, 900)
    if meanwhile != "more":
        sk.reset(stream)
        words = np.zeros_like(words)
    if meanwhile == "reset":
        return words
    sk.update(to_dev(pairs), stream)
    return words | oracle.build_sketch(p, pairs)


@pytest.mark.parametrize("meanwhile", ["reset", "small", "large", "more"])
@pytest.mark.parametrize("what", ["search up", "search down", "list up", "list down"])
def test_begun_restore_of_another_kind(what, meanwhile):
    p, theta, before, words = crafted(what)
    ip, sz, c, _ = oracle.restore(p, words, theta, mode="brute")
    say(f"begun restore: {what}, {meanwhile}, {len(ip)} records")
    with make_sketch(p) as sk, make_sketch(p) as other:
        other.upload(before)
        sk.upload(before)
        for _ in range(3):
            sk.restore(theta)
        sk.upload(words)
        pend = ddhf.restore_batch_begin([(sk, theta), (other, theta)])
        after = next_window(sk, p, meanwhile, words)
        (recs, _), (rest, _) = pend.end()
        assert_spl_equal(recs, ip, sz, c)
        assert_spl_equal(rest, *oracle.restore(p, before, theta, mode="brute")[:3])
        assert np.array_equal(sk.download(), after)
        ip, sz, c, _ = oracle.restore(p, after, theta, mode="brute")
        assert_spl_equal(sk.restore(theta)[0], ip, sz, c)


@pytest.mark.parametrize("meanwhile", ["reset", "small", "large", "more"])
@pytest.mark.parametrize("what", ["search up", "search down", "list up", "list down"])
def test_plan_run_of_another_kind(what, meanwhile):
    """A plan that restores the sketch as it is, after runs on windows of one
    kind; the sketch moves on before the results are asked for."""
    p, theta, before, words = crafted(what)
    ip, sz, c, _ = oracle.restore(p, words, theta, mode="brute")
    say(f"plan run: {what}, {meanwhile}, {len(ip)} records")
    with make_sketch(p) as sk, ddhf.Plan([(sk, to_dev(EMPTY), theta)], reset=False) as plan:
        sk.upload(before)
        for _ in range(3):
            plan.run()
            plan.results()
        sk.upload(words)
        plan.run()
        after = next_window(sk, p, meanwhile, words)
        assert_spl_equal(plan.results()[0][0], ip, sz, c)
        assert np.array_equal(sk.download(), after)


def overflowing(p, m):
    """A window of m super points: past the 6144 records a handle's sorted list
    starts with, so that a first restore is run again."""
    words = hosts_sketch(p, m, m)
    return (words, *oracle.restore(p, words, 100.0, mode="brute")[:3])


@pytest.mark.parametrize("planned", [False, True])
@pytest.mark.parametrize("meanwhile", ["reset", "small", "large", "more"])
def test_a_list_that_outgrows_the_buffers(meanwhile, planned):
    """Run again on the words that the restore read, or refused when they have
    been written again; never another window's list."""
    p = oracle.Params(128, 18, 5, 5)
    words, ip, sz, c = overflowing(p, 7000)
    assert len(ip) > 6144
    with make_sketch(p) as sk:
        sk._cap = 1 << 13                   # the caller's own buffer is large enough
        plan = ddhf.Plan([(sk, to_dev(EMPTY), 100.0)], reset=False) if planned else None

        def start():
            return plan.run() if planned else ddhf.restore_batch_begin([(sk, 100.0)])

        def collect(pend):
            return (plan.results() if planned else pend.end())[0][0]

        for again in range(2):              # the first time the buffers grow
            sk.upload(words)
            pend = start()
            after = next_window(sk, p, meanwhile, words)
            say(f"{len(ip)} records, planned {planned}, {meanwhile}, time {again}")
            if meanwhile == "reset" or again:
                assert_spl_equal(collect(pend), ip, sz, c)
            else:
                with pytest.raises(ddhf.SketchError) as e:
                    collect(pend)
                assert e.value.code == ddhf.SKETCH_E_CAPACITY
            assert np.array_equal(sk.download(), after)
        if plan:
            plan.close()


def test_a_lost_job_of_a_batch_leaves_the_others():
    p = oracle.Params(128, 18, 5, 5)
    words, *_ = overflowing(p, 7000)
    small = hosts_sketch(p, 40, 3)
    with make_sketch(p) as sk, make_sketch(p) as other:
        sk._cap = 1 << 13
        sk.upload(words)
        other.upload(small)
        pend = ddhf.restore_batch_begin([(sk, 100.0), (other, 100.0)])
        next_window(sk, p, "large", words)
        (recs, info), (rest, _) = pend.end(raise_errors=False)
        assert recs is None and info["status"] == ddhf.SKETCH_E_CAPACITY
        assert_spl_equal(rest, *oracle.restore(p, small, 100.0, mode="brute")[:3])


@pytest.mark.parametrize("meanwhile", ["reset", "small", "large", "more"])
def test_a_list_longer_than_the_callers_buffer(meanwhile):
    """The facade starts with room for 4096 records and asks again for what the
    same restore found."""
    p = oracle.Params(128, 18, 5, 5)
    words, ip, sz, c = overflowing(p, 5000)
    say(f"{len(ip)} records into 4096, {meanwhile}")
    with make_sketch(p) as sk:
        sk.upload(words)
        pend = ddhf.restore_batch_begin([(sk, 100.0)])
        after = next_window(sk, p, meanwhile, words)
        (recs, info), = pend.end()
        assert_spl_equal(recs, ip, sz, c)
        assert info["n_reported"] == len(ip)
        assert np.array_equal(sk.download(), after)
        for _ in range(2):
            sk._cap, sk._outbuf = 16, None
            sk.upload(words)
            recs, _ = ddhf.restore_batch([(sk, 100.0)])[0]
            assert_spl_equal(recs, ip, sz, c)


def test_an_ended_restore_is_ended_again_only_for_more_room():
    p = oracle.Params(128, 18, 5, 5)
    words = hosts_sketch(p, 60, 4)
    ip, sz, c, _ = oracle.restore(p, words, 100.0, mode="brute")
    with make_sketch(p) as sk:
        sk.upload(words)

        def end(cap):
            jobs = ddhf._RestoreJobs([(sk.handle, 100.0, cap)])
            return ddhf.sketch_restore_batch_end(jobs)[0]

        ddhf.sketch_restore_batch_begin([(sk.handle, 100.0, 8)])
        for cap in (8, 1, 0):
            _, _, st, need = end(cap)
            assert st == ddhf.SKETCH_E_CAPACITY and need == len(ip)
        recs, _, st, _ = end(len(ip))
        assert st == ddhf.SKETCH_OK
        assert_spl_equal(recs, ip, sz, c)
        with pytest.raises(ddhf.SketchError):       # its list has been given out
            end(100)
        ddhf.sketch_restore_batch_begin([(sk.handle, 100.0, 8)])
        assert end(8)[2] == ddhf.SKETCH_E_CAPACITY
        sk.restore(100.0)
        with pytest.raises(ddhf.SketchError):       # another restore has come since
            end(100)
