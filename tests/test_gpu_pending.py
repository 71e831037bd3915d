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
