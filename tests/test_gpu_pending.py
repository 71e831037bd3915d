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
from test_gpu_restore_passes import kernels

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


def left_out(k):
    """Whether a restore's launches (by name) leave a search or the long sort out."""
    return not (k["k_lattice"] and (k["k_join"] or k["k_join_walk"]) and k["k_rank_place"])


@pytest.mark.parametrize("planned", [False, True])
def test_every_kernel_only_where_the_sketch_is_written_meanwhile(planned):
    """Collected before the next window, a restore goes by the last one; the
    first write in between has it enqueued again, and from then on it
    launches every kernel at once."""
    p, theta, before, words = crafted("search up")
    want = [oracle.restore(p, w, theta, mode="brute")[:3] for w in (before, words)]
    with make_sketch(p) as sk:
        plan = ddhf.Plan([(sk, to_dev(EMPTY), theta)], reset=False) if planned else None
        start = plan.run if planned else lambda: ddhf.restore_batch_begin([(sk, theta)])
        collect = (lambda _: plan.results()[0][0]) if planned else lambda x: x.end()[0][0]
        sk.upload(before)
        for i in range(4):
            pend, k = kernels(start)
            say(f"planned {planned}, time {i}: {dict(k)}")
            assert_spl_equal(collect(pend), *want[0])
        assert left_out(k)
        for i in range(4):
            sk.upload((before, words)[i % 2])
            pend, k = kernels(start)
            after, more = kernels(lambda: next_window(sk, p, "large", words))
            say(f"planned {planned}, written {i}: {dict(k)}, then {dict(more)}")
            assert left_out(k) == (i == 0) and (more["k_estimate"] == 1) == (i == 0)
            assert_spl_equal(collect(pend), *want[i % 2])
            assert np.array_equal(sk.download(), after)
        if plan:
            plan.close()


def test_two_plans_of_one_sketch():
    """A plan that resets the sketch runs before another's results are asked
    for; either one's are its own run's, also when the other has gone."""
    p, theta, before, words = crafted("search down")
    want = [oracle.restore(p, w, theta, mode="brute")[:3] for w in (before, words)]
    pairs = rand_pairs(np.random.default_rng(2), 200_000, 900)
    built = oracle.build_sketch(p, pairs)
    theirs = oracle.restore(p, built, theta, mode="brute")[:3]
    with make_sketch(p) as sk:
        one = ddhf.Plan([(sk, to_dev(EMPTY), theta)], reset=False)
        two = ddhf.Plan([(sk, to_dev(pairs), theta)])
        sk.upload(before)
        for _ in range(3):
            one.run()
            assert_spl_equal(one.results()[0][0], *want[0])
        for i in range(3):
            sk.upload((words, before)[i % 2])
            one.run()
            for _ in range(3):
                two.run()
            say(f"two plans, time {i}")
            assert_spl_equal(one.results()[0][0], *want[1 - i % 2])
            assert_spl_equal(two.results()[0][0], *theirs)
            assert np.array_equal(sk.download(), built)
        sk.upload(words)
        two.run()
        two.results()
        two.run()
        one.run()
        one.close()
        assert_spl_equal(two.results()[0][0], *theirs)
        two.run()
        two.close()
        sk.reset()
        sk.update(to_dev(pairs))
        assert_spl_equal(sk.restore(theta)[0], *theirs)


def test_written_on_another_stream():
    """Begun on one stream, written on two others: the restore that is enqueued
    again waits for the first and goes before the write."""
    p, theta, before, words = crafted("search up")
    want = [oracle.restore(p, w, theta, mode="brute")[:3] for w in (before, words)]
    streams = [torch.cuda.Stream() for _ in range(3)]
    with make_sketch(p) as sk, make_sketch(p) as other:
        for i in range(6):
            kind = i % 2
            for s in (sk, other):
                s.upload((before, words)[kind], stream=streams[0])
            pend = ddhf.restore_batch_begin([(sk, theta), (other, theta)], stream=streams[1])
            after = next_window(sk, p, "large", words, streams[2])
            next_window(other, p, "small", words)
            (recs, _), (rest, _) = pend.end()
            assert_spl_equal(recs, *want[kind])
            assert_spl_equal(rest, *want[kind])
            assert np.array_equal(sk.download(stream=streams[i % 3]), after)
