"""GPU: one launch for every class where the level mapping's rows, and not the
staged inputs and outputs, set the LDS of a wave, at row counts that are no
multiple of 16 bytes: the same bits as LDS rows, and the oracle's values."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import paper_2404_01817_amd as neat
from tests.parity import assert_parity
from workloads import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("N,I,O", [(511, 4, 1), (601, 8, 2), (1023, 4, 4), (1024, 2, 1)])
def test_every_wave_of_a_workgroup(N, I, O):
    P, B = 1200, 20
    print("case", N, I, O, flush=True)
    rng = np.random.default_rng(N)
    # a few hidden nodes only: register classes, whose inputs are staged 16 bytes at a time,
    # beside one genome past them
    base = synth.make_population(rng, 16, N, 4 * N, I, O, 60, synth._k_density(2 * N),
                                 synth.CONTROL_ACTS, synth.ALL_AGGS)
    deep = synth.make_population(rng, 1, N, 4 * N, I, O, N - I - O, lambda r, na: 4 * N,
                                 synth.CONTROL_ACTS, synth.ALL_AGGS)
    base.nodes[3], base.conns[3] = deep.nodes[0], deep.conns[0]
    who = rng.integers(0, 16, P)
    who[:16] = np.arange(16)
    x = rng.standard_normal((P, B, I), dtype=np.float32)
    tn, tc = torch.from_numpy(base.nodes[who]).cuda(), torch.from_numpy(base.conns[who]).cuda()
    tx = torch.from_numpy(x).cuda()
    _, _, _, prog = neat.topo_sort(tn, tc, I, O, want_order=False)
    d = neat.dims_of(tn, tc, I, O)
    y, want = (neat.forward(d, prog, tx, B, variant=v) for v in (neat.FWD_AUTO, neat.FWD_LDS))
    nan = y.isnan()
    assert torch.equal(nan, want.isnan())
    assert torch.equal(y[~nan].view(torch.int32), want[~nan].view(torch.int32))
    y64, beta = oracle.forward(base.nodes, base.conns, x[:16], I, O)
    assert_parity(y[:16].cpu().numpy(), y64, beta, "any class N%d" % N)
