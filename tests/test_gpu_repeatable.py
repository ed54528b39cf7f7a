"""GPU: repeated launches over full-size populations, where thousands of waves
share every compute unit, give the same bits: the register blocks of small
populations (four samples per lane; the recurrent ones of 32, 52 and 64 slots),
the launch that holds every class and the launches per class, levels and grid
queries, on mixed networks and on networks of sines only (the longest activation
block).  (The blocks of 64 slots of a population of 50 rows are in
test_gpu_parity.py.)"""
from __future__ import annotations

import numpy as np
import pytest

import paper_2404_01817_amd as neat
from tests.test_forward_plan import GRAPH, kinds, plan  # noqa: F401
from workloads import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

WORK = {"mixed": (synth.CONTROL_ACTS, synth.ALL_AGGS), "sine": ((synth.ACT_SIN,), (synth.AGG_SUM,))}


def _population(seed, work, P, N, I, O, recurrent=False):
    rng = np.random.default_rng(seed)
    acts, aggs = WORK[work]
    base = synth.make_population(rng, 64, N, 4 * N, I, O, N - I - O, synth._k_density(4 * N), acts,
                                 aggs, recurrent=recurrent)
    base.nodes[::3, :, 2] = rng.uniform(0.5, 2.0, base.nodes[::3, :, 2].shape)  # responses
    who = torch.from_numpy(rng.integers(0, 64, P)).cuda()
    tn = torch.from_numpy(base.nodes).cuda()[who].contiguous()
    tc = torch.from_numpy(base.conns).cuda()[who].contiguous()
    _, _, status, prog = neat.topo_sort(tn, tc, I, O, want_order=False, recurrent=recurrent)
    assert int(status.abs().sum()) == 0
    return neat.dims_of(tn, tc, I, O), prog


def _repeat(call, what):
    first = call().view(torch.int32).clone()
    for rep in range(3):
        differ = int((call().view(torch.int32) != first).sum())
        print(what, "repeat", rep, "differing words", differ, flush=True)
        assert differ == 0


@pytest.mark.parametrize("work", sorted(WORK))
@pytest.mark.parametrize("P,N,I,O,B,variant,want", [
    (10000, 30, 8, 4, 1000, neat.FWD_AUTO, ["r32x4"]),
    (4000, 127, 17, 6, 300, neat.FWD_REG2, ["r64x2", "r128", "r224"]),
    (3000, 300, 17, 6, 300, neat.FWD_AUTO, ["any"]),
    (3000, 300, 17, 6, 300, neat.FWD_REG2, ["r64x2", "r128", "r224", "lds"]),
    (2000, 600, 9, 4, 60, neat.FWD_AUTO, ["any"]),
    (2000, 900, 9, 4, 40, neat.FWD_AUTO, ["lvl"]),
])
def test_forward(plan, work, P, N, I, O, B, variant, want):  # noqa: F811
    planned, = plan([(GRAPH, [dict(P=P, N=N, I=I, O=O, B=B, variant=variant)])])
    assert kinds(planned) == want
    d, prog = _population(N + B, work, P, N, I, O)
    x = torch.randn((P, B, I), device="cuda", generator=torch.Generator("cuda").manual_seed(N))
    _repeat(lambda: neat.forward(d, prog, x, B, variant=variant), "%s %s" % (work, want))


@pytest.mark.parametrize("work", sorted(WORK))
@pytest.mark.parametrize("P,N,B,want", [(10000, 30, 500, "r32rec"), (10000, 50, 500, "r52rec"),
                                        (6000, 62, 500, "r64rec")])
def test_recurrent(plan, work, P, N, B, want):  # noqa: F811
    planned, = plan([(GRAPH, [dict(P=P, N=N, I=8, O=4, B=B, recurrent=1)])])
    assert kinds(planned) == [want]
    d, prog = _population(N, work, P, N, 8, 4, recurrent=True)
    x = torch.randn((P, B, 8), device="cuda", generator=torch.Generator("cuda").manual_seed(N))
    _repeat(lambda: neat.forward_recurrent(d, prog, x, B, 4), "%s %s" % (work, want))


@pytest.mark.parametrize("work", sorted(WORK))
@pytest.mark.parametrize("P,N", [(1000, 30), (600, 62)])
def test_grid(work, P, N):
    d, prog = _population(N, work, P, N, 5, 1)
    _repeat(lambda: neat.forward_grid(d, prog, 16, 0, 65536), "%s grid N %d" % (work, N))
