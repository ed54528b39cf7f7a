"""Where the transformation changes its way of working: keys on both sides of the key map's end.

The oracle gives order, level and status bit for bit; outputs follow the parity rule."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from tests.test_gpu_parity import _assert_outputs, _assert_transform_exact, _gpu
from workloads import synth

pytestmark = pytest.mark.gpu


def _map_end(N):
    """Keys below this are in the map: 32 times the smallest power of two >= max(64, 2 N)."""
    h = 64
    while h < 2 * N:
        h *= 2
    return 32 * h


def _rekey(pop, g, new):
    """Hidden keys of genome g replaced (in their order) by the sorted keys new."""
    hidden = np.sort(pop.nodes[g, pop.nodes[g, :, 0] >= pop.I + pop.O, 0])
    for k, v in zip(hidden[::-1], new[::-1][:len(hidden)]):  # from above: no key meets a new one
        pop.nodes[g, pop.nodes[g, :, 0] == k, 0] = v
        for col in (0, 1):
            pop.conns[g, pop.conns[g, :, col] == k, col] = v


@pytest.mark.parametrize("N", [7, 32, 33, 64, 65, 128, 129, 200, 257, 513])
def test_keys_at_the_end_of_the_key_map(N):
    print("case", N, flush=True)
    rng = np.random.default_rng(N)
    P, I, O, end = 24, 3, 2, _map_end(N)
    pop = synth.make_population(rng, P, N, 4 * N, I, O, N - 5, synth._k_density(4 * N),
                                synth.CONTROL_ACTS, synth.ALL_AGGS)
    h = N - 5
    for g in range(P):
        kind = g % 6
        if kind == 1:    # the map's last keys
            _rekey(pop, g, np.arange(end - h, end))
        elif kind == 2:  # one key past it
            _rekey(pop, g, np.arange(end - h + 1, end + 1))
        elif kind == 3:  # the largest keys
            _rekey(pop, g, np.arange((1 << 24) - h, 1 << 24))
    for g in range(P // 2, P):
        rows = np.nonzero(~np.isnan(pop.nodes[g, :, 0]))[0]
        on = np.nonzero(pop.conns[g, :, 2] == 1.0)[0]
        if g % 6 == 0 and len(rows) > 1:    # a repeated key
            pop.nodes[g, rows[-1], 0] = pop.nodes[g, rows[-2], 0]
        elif g % 6 == 4 and len(on):        # sources that no node holds, in the map and past it
            pop.conns[g, on[0], 0] = end - 1
            pop.conns[g, on[-1], 0] = end
        elif g % 6 == 5 and len(on) > 1:    # an edge twice, and a missing output
            pop.conns[g, on[1], :2] = pop.conns[g, on[0], :2]
            pop.nodes[g, pop.nodes[g, :, 0] == I, 0] = np.nan
    x = rng.standard_normal((P, 40, I), dtype=np.float32)
    order, level, status, y = _gpu(pop.nodes, pop.conns, I, O, x)
    _assert_transform_exact(pop.nodes, pop.conns, I, O, order, level, status)
    assert (status[:P // 2] == 0).all()
    y64, beta = oracle.forward(pop.nodes, pop.conns, x, I, O)
    _assert_outputs(y, y64, beta, "keys N=%d" % N)
