"""GPU parity of the coefficient form where a size or a launch reaches a limit:
look-ups far past a block of edges, launches of more work items than one
dimension of a grid takes, outputs cut into parts, and batches cut into rounds."""
import numpy as np
import pytest

import oracle
from paper_2010_08423_amd import inputs
from parity_util import host_threads, say

pytestmark = pytest.mark.gpu

R = None


def setup_module(module):
    global R
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2010_08423_amd as lib

    R = lib
    R.library()


def hub_graph(arrivals, leave, feeders=2000):
    """`arrivals` edges into vertex 0, in order of time from 1 on, `feeders` per
    time; edges from vertex 0 to 40 others at each of the times `leave` (as
    shares of the last arrival's time), and one edge on from each of those."""
    i = np.arange(arrivals)
    last = int(i[-1] // feeders + 1)
    times = np.maximum(1, (np.asarray(leave) * last).astype(np.int64))
    out = 1 + feeders + np.arange(40)
    src = [1 + i % feeders, np.zeros(40 * len(times)), np.tile(out, len(times))]
    dst = [np.zeros(arrivals), np.tile(out, len(times)), np.tile(out, len(times)) + 40]
    t = [1 + i // feeders, np.repeat(times, 40), np.repeat(times, 40) + 1]
    g = inputs.TemporalGraph(1 + feeders + 80, *(np.concatenate(x).astype(np.uint32) for x in (src, dst, t)),
                             name=f"hub{arrivals}")
    return g, last


# The search for the next marked window end goes on past 64 blocks of 1024
# edges in steps of 1024 blocks: one step from some 10^5 arrivals on, with one
# edge per thread and, from 600000 edges on, four; a second step from 1.12*10^6.
@pytest.mark.parametrize("arrivals", [100_000, 400_000, 700_000, 1_300_000])
def test_next_window_end_far_past_a_block(arrivals):
    for leave in ((1.0,), (0.3, 0.97)):
        g, last = hub_graph(arrivals, leave)
        gd = R.Graph.from_inputs(g)
        for k in (3, 4):
            for delta in (2, last // 2, last):
                say("[coef] hub", arrivals, "leave", leave, "k", k, "delta", delta)
                want = oracle.sieve(g.n, g.src, g.dst, g.t, k, delta, 9, threads=host_threads())
                assert R.run(gd, k, delta, 9).fingerprint == want
                assert R.run(gd, k, delta, 9, tuning=R.Tuning(edges_per_tile=16)).fingerprint == want
