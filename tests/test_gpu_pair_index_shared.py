"""Handles of one hash family share one pair index: what a handle costs, and
lists of handles whose neighbours come and go."""
import numpy as np
import pytest
import torch

import oracle
from paper_1803_11449_amd import ddhf, serving
from test_gpu_parity import assert_spl_equal, make_sketch, say
from test_gpu_restore_launches import hosts_sketch

pytestmark = pytest.mark.gpu


def test_a_handle_costs_what_the_server_counts():
    """64 links of k = 14, each within a seventh of resident_bytes (allocations
    are rounded up), and one index for all."""
    n, params = 64, (1024, 14, 5, 6)
    with ddhf.Sketch(*params, device=0):             # the device's shared buffers
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        links = [ddhf.Sketch(*params, device=0) for _ in range(n)]
        torch.cuda.synchronize()
        took = free - torch.cuda.mem_get_info()[0]
        for sk in links:
            sk.close()
    say(f"{took / n / 2**20:.2f} MiB a handle")
    assert took <= n * serving.resident_bytes(*params) * 8 // 7


@pytest.mark.parametrize("k,alpha", [(14, 6), (15, 6), (18, 5)])
def test_lists_as_neighbours_come_and_go(k, alpha):
    """Two hash families, each with a handle that outlives the one that built
    the index, and one that finds none left."""
    theta, made = 40.0, []
    for seed in (7, 8):
        p = oracle.Params(64, k, 5, alpha, seed=seed)
        words = hosts_sketch(p, 300, seed)
        made.append((p, words, oracle.restore(p, words, theta, mode="brute")[:3]))

    def check(sk, words, want):
        sk.set_option(ddhf.SKETCH_OPT_CANDIDATES, 2)
        sk.upload(words)
        assert_spl_equal(sk.restore(theta)[0], *want)

    for _ in range(2):
        first = [make_sketch(p) for p, _, _ in made]
        second = [make_sketch(p) for p, _, _ in made]
        for sk in first:
            sk.close()
        for sk, (_, words, want) in zip(second, made):
            check(sk, words, want)
        second[0].close()
        with make_sketch(made[0][0]) as again:
            check(again, *made[0][1:])
            check(second[1], *made[1][1:])
        second[1].close()
