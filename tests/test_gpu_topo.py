"""Where the transformation changes its way of working: keys on both sides of the key map's end,
and the graphs of groups of more than one wave.

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


def _connect(pop, g, pairs, rng):
    """Genome g's connections replaced by the pairs, in random rows."""
    pop.conns[g] = np.nan
    rows = rng.choice(pop.conns.shape[1], len(pairs), replace=False)
    pop.conns[g, rows, :2] = pairs
    pop.conns[g, rows, 2] = 1.0
    pop.conns[g, rows, 3] = rng.standard_normal(len(pairs)) * 0.5


# connection rows in registers only and beyond them, lists of every length modulo
# eight, in-degrees and depths up to the number of rows
@pytest.mark.parametrize("N,C", [(65, 256), (65, 700), (128, 513), (129, 2000), (300, 1200),
                                 (512, 4000), (1000, 2100)])
def test_graphs_of_larger_groups(N, C):
    print("case", N, C, flush=True)
    rng = np.random.default_rng(N + C)
    P, I, O = 28, 3, 2
    pop = synth.make_population(rng, P, N, C, I, O, N - 5, synth._k_density(C),
                                synth.CONTROL_ACTS, synth.ALL_AGGS)
    for g in range(P):
        keys = pop.nodes[g, :, 0]
        hidden = rng.permutation(keys[keys >= I + O])
        kind = g % 7
        chain = [[a, b] for a, b in zip(np.r_[0, hidden], np.r_[hidden, I])]
        on = np.nonzero(pop.conns[g, :, 2] == 1.0)[0]
        if kind == 1:                     # one long chain
            _connect(pop, g, chain, rng)
        elif kind == 2:                   # the widest fan-in, and a second output fed by g nodes
            _connect(pop, g, [[k % I, h] for k, h in enumerate(hidden)] +
                     [[h, I] for h in hidden[:C - 2 * len(hidden)]] +
                     [[h, I + 1] for h in hidden[:g % 8][:max(0, C - 2 * len(hidden))]], rng)
        elif kind == 3 and len(on) > 1:   # an edge twice: first and last row in use
            pop.conns[g, on[-1], :2] = pop.conns[g, on[0], :2]
        elif kind == 4 and len(hidden):   # a cycle through every hidden node
            _connect(pop, g, chain + [[hidden[-1], hidden[0]]], rng)
        elif kind == 5 and len(on):       # a self-loop at an output, nothing else wrong
            pop.conns[g, on[-1], :2] = I
        elif kind == 6 and len(hidden) > 2:   # a chain whose first node also reads its third
            _connect(pop, g, chain + [[hidden[2], hidden[0]]], rng)
    x = rng.standard_normal((P, 33, I), dtype=np.float32)
    order, level, status, y = _gpu(pop.nodes, pop.conns, I, O, x)
    _assert_transform_exact(pop.nodes, pop.conns, I, O, order, level, status)
    assert (status[0::7] == 0).all() and (status[1::7] == 0).all() and (status[2::7] == 0).all()
    y64, beta = oracle.forward(pop.nodes, pop.conns, x, I, O)
    _assert_outputs(y, y64, beta, "graphs N=%d C=%d" % (N, C))


@pytest.mark.parametrize("N,C", [(7, 20), (62, 248), (64, 900), (65, 260), (200, 3000)])
def test_rejected_genomes_with_keys_past_the_map(N, C):
    """The key table's path: repeated keys, keys that no node holds, repeated edges and missing
    outputs in genomes that all have keys past the map, beside sound ones."""
    print("case", N, C, flush=True)
    rng = np.random.default_rng(N + C)
    P, I, O, end = 20, 3, 2, _map_end(N)
    pop = synth.make_population(rng, P, N, C, I, O, N - 5, synth._k_density(C),
                                synth.CONTROL_ACTS, synth.ALL_AGGS)
    for g in range(P):
        h = N - 5
        _rekey(pop, g, np.sort(rng.choice((1 << 24) - end - h, h, replace=False)) + end + np.arange(h))
        hidden = np.nonzero(pop.nodes[g, :, 0] >= I + O)[0]
        on = np.nonzero(pop.conns[g, :, 2] == 1.0)[0]
        if g % 5 == 1 and len(hidden) > 1:
            pop.nodes[g, hidden[0], 0] = pop.nodes[g, hidden[-1], 0]
        elif g % 5 == 2 and len(on):
            pop.conns[g, on[-1], 0] = (1 << 24) - 1
        elif g % 5 == 3 and len(on) > 1:
            pop.conns[g, on[0], :2] = pop.conns[g, on[-1], :2]
        elif g % 5 == 4:
            pop.nodes[g, pop.nodes[g, :, 0] == I, 0] = np.nan
    x = rng.standard_normal((P, 9, I), dtype=np.float32)
    order, level, status, y = _gpu(pop.nodes, pop.conns, I, O, x)
    _assert_transform_exact(pop.nodes, pop.conns, I, O, order, level, status)
    assert (status[0::5] == 0).all()
    y64, beta = oracle.forward(pop.nodes, pop.conns, x, I, O)
    _assert_outputs(y, y64, beta, "rejected N=%d" % N)
