"""GPU: grid queries of networks with so many outputs that a wave's LDS holds
them and not the table of a tile's query offsets: the same bits as the queries
given as inputs, and the oracle's values."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import paper_2404_01817_amd as neat
from tests.parity import assert_parity
from workloads import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# outputs at the limit of two samples per lane (313), of one (631), and one below each, whose
# table does fit; substrates smaller and larger than a tile
@pytest.mark.parametrize("O,Q", [(313, 300), (312, 300), (631, 64), (630, 50)])
@pytest.mark.parametrize("side,first", [(3, 20), (5, 17), (16, 777), (256, 2 ** 32 - 300)])
def test_grid_queries_at_the_lds_limit(O, Q, side, first):
    Q = min(Q, side ** 4 - first)
    print("case", O, Q, side, first, flush=True)
    rng = np.random.default_rng(O + side)
    N = O + 25
    pop = synth.make_population(rng, 6, N, 3 * N, 5, O, 20, synth._k_density(3 * N),
                                synth.CPPN_ACTS, (synth.AGG_SUM,))
    tn, tc = torch.from_numpy(pop.nodes).cuda(), torch.from_numpy(pop.conns).cuda()
    _, _, _, prog = neat.topo_sort(tn, tc, 5, O, want_order=False)
    d = neat.dims_of(tn, tc, 5, O)
    y = neat.forward_grid(d, prog, side, first, Q)
    x = synth.grid_queries(first, Q, side)
    want = neat.forward(d, prog, torch.from_numpy(x).cuda(), Q, shared_inputs=True,
                        variant=neat.FWD_LVL)
    assert torch.equal(y.view(torch.int32), want.view(torch.int32))
    y64, beta = oracle.forward(pop.nodes, pop.conns, x, 5, O, shared_inputs=True)
    assert_parity(y.cpu().numpy(), y64, beta, "grid O%d side%d" % (O, side))
