"""GPU parity of the HyperNEAT substrate layer (neat_substrate_forward,
through the C ABI) against the CPU oracle (``oracle/substrate.py``).

Outputs must satisfy the parity rule of ``oracle.within_tolerance`` with the
substrate oracle's fp32 bound; the weights the call writes must equal the
CPPN grid calculation bit for bit."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from tests.parity import assert_parity
from oracle import substrate
from workloads import synth
from tests.helpers import genome, stack

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _neat():
    import paper_2404_01817_amd as neat
    return neat


def _run(nodes, conns, side, X, theta):
    neat = _neat()
    dev = torch.device("cuda:0")
    tn = torch.from_numpy(np.ascontiguousarray(nodes)).to(dev)
    tc = torch.from_numpy(np.ascontiguousarray(conns)).to(dev)
    _, _, st, prog = neat.topo_sort(tn, tc, 5, 1, want_order=False)
    d = neat.dims_of(tn, tc, 5, 1)
    tx = torch.from_numpy(np.ascontiguousarray(X)).to(dev)
    y, w = neat.substrate_forward(d, prog, side, tx, theta)
    S = side * side
    g = neat.forward_grid(d, prog, side, 0, S * S)
    torch.cuda.synchronize()
    return y.cpu().numpy(), w.cpu().numpy(), g.cpu().numpy().reshape(w.shape)


def _pop(seed, P, bad=True):
    pop = synth.cppn(seed=seed, P=P)
    n, c = pop.nodes.copy(), pop.conns.copy()
    if bad:
        n[1, 5, 3] = 11.0          # the output node's activation code out of range
    return n, c


@pytest.mark.parametrize("side,B", [(8, 70), (8, 1), (16, 64), (16, 130), (24, 33), (32, 65)])
def test_substrate_parity(side, B):
    print("case side", side, "B", B, flush=True)
    n, c = _pop(side + B, 5)
    X = synth.substrate_inputs(seed=B, B=B, side=side)
    y, w, g = _run(n, c, side, X, substrate.THRESHOLD)
    assert np.array_equal(w.view(np.uint32), g.view(np.uint32))
    Y64, bound = substrate.forward(n, c, side, X)
    stats = assert_parity(y, Y64, bound, "")
    assert np.all(np.isnan(y[1]))


@pytest.mark.parametrize("theta", [0.0, 0.5, 1e30])
def test_substrate_thresholds(theta):
    n, c = _pop(3, 4, bad=False)
    X = synth.substrate_inputs(seed=5, B=40, side=8)
    y, _, _ = _run(n, c, 8, X, theta)
    Y64, bound = substrate.forward(n, c, 8, X, theta=theta)
    stats = assert_parity(y, Y64, bound, "")
    if theta == 1e30:
        assert np.all(y == 0.0)


def test_substrate_constant_cppn_exact_structure():
    """A CPPN without edges paints w = act(bias) everywhere: every output of
    an input plane is the same value, tanh(w sum x)."""
    nodes = {k: (k, 0.0, 1.0, 0, 0) for k in range(6)}
    nodes[5] = (5, 0.75, 1.0, 0, 0)
    n, c = stack([genome(6, 4, nodes, {})])
    X = synth.substrate_inputs(seed=9, B=20, side=16)
    y, w, _ = _run(n, c, 16, X, 0.2)
    assert np.all(w == np.float32(0.75))
    ref = np.tanh(0.75 * X.astype(np.float64).sum(axis=1))
    assert np.allclose(y[0], ref[:, None], atol=1e-5)
    assert np.all(y[0] == y[0, :, :1])


def test_substrate_argument_errors():
    neat = _neat()
    dev = torch.device("cuda:0")
    n, c = _pop(1, 2, bad=False)
    tn, tc = torch.from_numpy(n).to(dev), torch.from_numpy(c).to(dev)
    _, _, _, prog = neat.topo_sort(tn, tc, 5, 1, want_order=False)
    d = neat.dims_of(tn, tc, 5, 1)
    for side in (4, 12, 40):
        x = torch.zeros((3, side * side), device=dev)
        with pytest.raises(neat.NeatError):
            neat.substrate_forward(d, prog, side, x)
    with pytest.raises(neat.NeatError):
        neat.substrate_forward(d, prog, 8, torch.zeros((3, 64), device=dev), threshold=-1.0)
    y, _ = neat.substrate_forward(d, prog, 8, torch.zeros((0, 64), device=dev))
    assert y.shape == (2, 0, 64)
    torch.cuda.synchronize()


def test_substrate_full_size_sampled():
    """The benchmark's substrate workload (P=1000 CPPNs, side 16, B=256
    shared input planes) in its launch configuration; the oracle checks
    every output of a sample of genomes."""
    neat = _neat()
    pop = synth.cppn()
    X = synth.substrate_inputs()
    dev = torch.device("cuda:0")
    tn = torch.from_numpy(pop.nodes).to(dev)
    tc = torch.from_numpy(pop.conns).to(dev)
    _, _, st, prog = neat.topo_sort(tn, tc, 5, 1, want_order=False)
    d = neat.dims_of(tn, tc, 5, 1)
    y, _ = neat.substrate_forward(d, prog, 16, torch.from_numpy(X).to(dev))
    torch.cuda.synchronize()
    y = y.cpu().numpy()
    sample = np.concatenate([np.random.default_rng(0).choice(pop.P, 8, replace=False),
                             [0, pop.P - 1]])
    Y64, bound = substrate.forward(pop.nodes[sample], pop.conns[sample], 16, X)
    stats = assert_parity(y[sample], Y64, bound, "")


@pytest.mark.parametrize("side,B", [(8, 63), (8, 65), (16, 64), (16, 127), (24, 129), (8, 257)])
def test_layer_row_tiles(side, B):
    """Input planes on both sides of a workgroup's 64 and 128 rows, against
    the contraction in 64 bits of the weights that the call returns."""
    import paper_2404_01817_amd as neat
    print("case side=%d B=%d" % (side, B), flush=True)
    pop = synth.cppn(seed=side + B, P=5)
    tn, tc = torch.from_numpy(pop.nodes).cuda(), torch.from_numpy(pop.conns).cuda()
    _, _, _, prog = neat.topo_sort(tn, tc, pop.I, pop.O, want_order=False)
    S = side * side
    x = torch.from_numpy(np.random.default_rng(B).uniform(-1, 1, (B, S)).astype(np.float32)).cuda()
    y, w = neat.substrate_forward(neat.dims_of(tn, tc, pop.I, pop.O), prog, side, x, 0.2)
    w64 = torch.where(w.abs() < 0.2, torch.zeros_like(w), w).double().view(-1, S, S)
    for g in range(pop.P):
        z = x.double() @ w64[g]
        # a sum of S products in fp32, then tanh (slope at most 1)
        u = 2.0 ** -24
        bound = S * u / (1 - S * u) * (x.double().abs() @ w64[g].abs()) + 1e-6
        assert ((y[g].double() - torch.tanh(z)).abs() <= bound).all()


# the largest launches take two blocks of rows per wave where the planes fill them
@pytest.mark.parametrize("B", [192, 200, 256])
def test_layer_rows_of_large_launches(B):
    import paper_2404_01817_amd as neat
    print("case side=32 P=25 B=%d" % B, flush=True)
    pop = synth.cppn(seed=B, P=25)
    tn, tc = torch.from_numpy(pop.nodes).cuda(), torch.from_numpy(pop.conns).cuda()
    _, _, _, prog = neat.topo_sort(tn, tc, pop.I, pop.O, want_order=False)
    S = 1024
    x = torch.from_numpy(np.random.default_rng(B).uniform(-1, 1, (B, S)).astype(np.float32)).cuda()
    y, w = neat.substrate_forward(neat.dims_of(tn, tc, pop.I, pop.O), prog, 32, x, 0.2)
    w = w.view(-1, S, S)
    for g in (0, 12, 24):
        w64 = torch.where(w[g].abs() < 0.2, torch.zeros_like(w[g]), w[g]).double()
        u = 2.0 ** -24  # as above
        bound = S * u / (1 - S * u) * (x.double().abs() @ w64.abs()) + 1e-6
        assert ((y[g].double() - torch.tanh(x.double() @ w64)).abs() <= bound).all()
