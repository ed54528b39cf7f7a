"""GPU: the batched path (neat_forward_batch) against single-population
calls and the oracle; graph replays."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from tests.parity import assert_parity
from workloads import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _neat():
    import paper_2404_01817_amd as neat
    return neat


def _same_bits(a, b):
    nan = np.isnan(a)
    return np.array_equal(nan, np.isnan(b)) and np.array_equal(a[~nan].view(np.uint32),
                                                                 b[~nan].view(np.uint32))


class _Pop:
    """Device buffers of one population of a batch."""

    def __init__(self, pop, grid=None):
        neat = _neat()
        dev = torch.device("cuda:0")
        self.pop = pop
        self.nodes = torch.from_numpy(pop.nodes).to(dev)
        self.conns = torch.from_numpy(pop.conns).to(dev)
        self.d = neat.dims_of(self.nodes, self.conns, pop.I, pop.O)
        self.prog = torch.empty((neat.program_bytes(self.d) // 4,), dtype=torch.int32, device=dev)
        self.status = torch.empty((pop.P,), dtype=torch.int32, device=dev)
        self.grid = grid
        if grid is None:
            self.x = torch.from_numpy(pop.inputs).to(dev)
            self.B = pop.B
        else:
            self.x = None
            self.B = grid[2]
        self.y = torch.full((pop.P, self.B, pop.O), 7.0, dtype=torch.float32, device=dev)

    def item(self, with_transform=True):
        neat = _neat()
        kw = dict(nodes=self.nodes, conns=self.conns, status=self.status) if with_transform else {}
        if self.grid is None:
            return neat.batch_item(self.d, self.prog, self.y, inputs=self.x, B=self.B, **kw)
        side, first, Q = self.grid
        return neat.batch_item(self.d, self.prog, self.y, B=Q, grid_side=side, grid_first=first,
                               **kw)

    def single(self):
        """Outputs of the single-population calls."""
        neat = _neat()
        _, _, _, prog = neat.topo_sort(self.nodes, self.conns, self.pop.I, self.pop.O,
                                       want_order=False)
        if self.grid is None:
            y = neat.forward(self.d, prog, self.x, self.B)
        else:
            y = neat.forward_grid(self.d, prog, *self.grid)
        torch.cuda.synchronize()
        return y.cpu().numpy()


def _uneven(seed, n, N_range=(10, 300)):
    return synth.uneven(seed=seed, n_pops=n, P_range=(3, 60), N_range=N_range, B_range=(1, 300))


def test_batch_matches_single_calls_and_oracle():
    """A batch of uneven populations (every slot class, TENSOR and GRID
    items) gives the same bits as one call per population, and the
    oracle's values within the parity rule."""
    neat = _neat()
    pops = [_Pop(p) for p in _uneven(21, 7)]
    cppn = synth.cppn(seed=4, P=12)
    pops.append(_Pop(cppn, grid=(16, 1000, 700)))
    plan = neat.BatchPlan()
    plan.run([p.item() for p in pops])
    torch.cuda.synchronize()
    # transformations: at most one launch per workgroup size (16) and one
    # class listing; calculations: at most one launch per kernel kind and
    # input mode
    assert 2 <= plan.launches <= 16 + 1 + 18
    for k, p in enumerate(pops):
        y = p.y.cpu().numpy()
        assert _same_bits(y, p.single()), k
        if p.grid is None:
            y64, beta = oracle.forward(p.pop.nodes, p.pop.conns, p.pop.inputs, p.pop.I, p.pop.O)
        else:
            q = synth.grid_queries(p.grid[1], p.grid[2])
            y64, beta = oracle.forward(p.pop.nodes, p.pop.conns, q, p.pop.I, p.pop.O,
                                       shared_inputs=True)
        stats = assert_parity(y, y64, beta, "item %d" % k)
        st = p.status.cpu().numpy().astype(np.uint32)
        assert np.array_equal(st, oracle.transform(p.pop.nodes, p.pop.conns, p.pop.I,
                                                   p.pop.O)[2])
    plan.free()


def test_batch_graph_replays():
    """Replays of the recorded graph, with eager work and new input contents
    between them, each equal the eager single-population results; changing
    the items rebuilds the plan."""
    neat = _neat()
    pops = [_Pop(p) for p in _uneven(22, 5, N_range=(10, 150))]
    plan = neat.BatchPlan()
    items = [p.item() for p in pops]
    rng = np.random.default_rng(3)
    for rep in range(4):
        for p in pops:
            p.x.copy_(torch.from_numpy(rng.standard_normal(tuple(p.x.shape)).astype(np.float32)))
            p.y.fill_(7.0)
        plan.run(items)
        torch.cuda.synchronize()
        # eager work between replays
        junk = torch.randn(1 << 20, device="cuda:0").sum().item()
        assert np.isfinite(junk)
        for k, p in enumerate(pops):
            assert _same_bits(p.y.cpu().numpy(), p.single()), (rep, k)
    n0 = plan.launches
    # forward only (programs already built), a different item list
    items2 = [p.item(with_transform=False) for p in pops[:3]]
    plan.run(items2)
    torch.cuda.synchronize()
    assert plan.launches < n0
    for p in pops[:3]:
        assert _same_bits(p.y.cpu().numpy(), p.single())
    plan.free()


def test_batch_argument_errors():
    neat = _neat()
    pops = [_Pop(p) for p in _uneven(23, 2, N_range=(10, 40))]
    items = [p.item() for p in pops]
    items[1].input_genome_stride = 1  # smaller than B * I
    plan = neat.BatchPlan()
    with pytest.raises(neat.NeatError, match="item 1"):
        plan.run(items)
    assert plan.launches == 0


def test_batch_with_the_largest_genomes():
    """A batch mixing small populations with N_max = 600 (LDS rows, tiles of
    64) and N_max = 1024 (LDS rows, half-wave tiles) populations, 230
    outputs live to the end: the same bits as single calls, and the
    oracle's values."""
    neat = _neat()
    rng = np.random.default_rng(77)
    big = []
    for N, C in ((600, 2400), (1024, 2048)):
        P, I, O, B = 3, 6, 230, 37
        nodes = np.full((P, N, 5), np.nan, np.float32)
        conns = np.full((P, C, 4), np.nan, np.float32)
        for p in range(P):
            synth.make_genome(rng, N, C, I, O, int(rng.integers(200, N - I - O)),
                              lambda na: int(rng.integers(C // 2, min(C, na) + 1)),
                              synth.CONTROL_ACTS, synth.ALL_AGGS, nodes_out=nodes[p],
                              conns_out=conns[p])
        pop = synth.Population(nodes, conns, I, O)
        pop.inputs = rng.standard_normal((P, B, I)).astype(np.float32)
        big.append(pop)
    pops = [_Pop(p) for p in _uneven(31, 3)] + [_Pop(p) for p in big]
    plan = neat.BatchPlan()
    plan.run([p.item() for p in pops])
    torch.cuda.synchronize()
    for k, p in enumerate(pops):
        y = p.y.cpu().numpy()
        assert _same_bits(y, p.single()), k
        y64, beta = oracle.forward(p.pop.nodes, p.pop.conns, p.pop.inputs, p.pop.I, p.pop.O)
        stats = assert_parity(y, y64, beta, "item %d" % k)
    plan.free()


def test_items_of_the_two_samples_kernel_share_the_wave_target():
    """Four control-shaped items (N_max = 50, B of 640 to 1000, so every
    genome runs the two-samples-per-lane kernel) large enough that the launch
    gives each wave two tiles of 128 samples (sum of P x ceil(tiles / 2)
    reaches the 32768-wave target, P x ceil(tiles / 3) does not), with
    ragged last tiles: the same bits as one call per item (one tile per wave
    there), and sampled genomes within the oracle's parity rule."""
    neat = _neat()
    base = synth.control(seed=9, P=9000, with_inputs=False)
    rng = np.random.default_rng(19)
    sizes, Bs = (3000, 2500, 2000, 1500), (1000, 777, 1000, 640)
    pops, g0 = [], 0
    for P, B in zip(sizes, Bs):
        part = synth.Population(base.nodes[g0:g0 + P], base.conns[g0:g0 + P], base.I, base.O)
        part.inputs = rng.standard_normal((P, B, base.I)).astype(np.float32)
        pops.append(_Pop(part))
        g0 += P
    tiles = [(B + 127) // 128 for B in Bs]
    assert sum(P * -(-t // 2) for P, t in zip(sizes, tiles)) >= 32768
    assert sum(P * -(-t // 3) for P, t in zip(sizes, tiles)) < 32768
    plan = neat.BatchPlan()
    plan.run([p.item() for p in pops])
    torch.cuda.synchronize()
    for k, p in enumerate(pops):
        y = p.y.cpu().numpy()
        assert _same_bits(y, p.single()), k
        pick = np.sort(rng.choice(p.pop.P, 48, replace=False))
        y64, beta = oracle.forward(p.pop.nodes[pick], p.pop.conns[pick], p.pop.inputs[pick],
                                   p.pop.I, p.pop.O)
        assert_parity(y[pick], y64, beta, "item %d" % k)
    plan.free()


# populations on both sides of the rules for several at once: the level mapping
# past 222 rows up to 16 inputs, one launch for every class past 300 rows (126
# when the launches follow one another), and the launches per class
@pytest.mark.parametrize("no_alloc", [False, True], ids=["graph", "in order"])
def test_mappings_of_shared_populations(no_alloc):
    import paper_2404_01817_amd as neat
    rng = np.random.default_rng(5)
    items, outs, refs, keep = [], [], [], []
    for P, N, B in [(30, 126, 70), (30, 127, 70), (30, 222, 16), (30, 223, 16), (30, 223, 17),
                    (30, 300, 130), (30, 301, 130), (700, 301, 200), (40, 50, 300)]:
        pop = synth.uneven_population(rng, (20, 20), (N, N), (1, 1), with_inputs=False)
        who = np.arange(P) % pop.P
        tn, tc = torch.from_numpy(pop.nodes[who]).cuda(), torch.from_numpy(pop.conns[who]).cuda()
        x = torch.from_numpy(rng.standard_normal((P, B, pop.I), dtype=np.float32)).cuda()
        d = neat.dims_of(tn, tc, pop.I, pop.O)
        _, _, _, prog = neat.topo_sort(tn, tc, pop.I, pop.O, want_order=False)
        refs.append(neat.forward(d, prog, x, B, variant=neat.FWD_LDS))
        outs.append(torch.empty_like(refs[-1]))
        own = torch.empty_like(prog)  # written by the batch's transformation
        items.append(neat.batch_item(d, own, outs[-1], inputs=x, B=B, nodes=tn, conns=tc))
        keep.append((tn, tc, x, own))  # items hold addresses only
    plan = neat.BatchPlan()
    for _ in range(3):
        for y in outs:
            y.fill_(7.0)
        neat.forward_batch_noalloc(items) if no_alloc else plan.run(items)
        torch.cuda.synchronize()
        for y, r in zip(outs, refs):
            assert torch.equal(y.isnan(), r.isnan())
            assert torch.equal(y.nan_to_num(0.0).view(torch.int32),
                               r.nan_to_num(0.0).view(torch.int32))
    del keep
