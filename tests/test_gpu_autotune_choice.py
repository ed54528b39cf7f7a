"""GPU: autotuning where NEAT_FWD_AUTO launches none of the five candidates
(four samples per lane; every class in one launch): the recorded winner is no
slower than the candidates' reported times say, and tuned calls and batches
give the bits of untuned ones."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import paper_2404_01817_amd as neat
from tests.parity import assert_parity
from workloads import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CANDIDATES = [neat.FWD_REG, neat.FWD_REG2, neat.FWD_LDS, neat.FWD_LVL, neat.FWD_SEG]


@pytest.fixture(autouse=True)
def _clean_tune_table():
    yield
    neat.tune_clear()


@pytest.mark.parametrize("P,N,B", [(3000, 20, 500), (60, 200, 130), (2500, 160, 200)])
def test_automatic_choice_is_timed_beside_the_candidates(P, N, B):
    print("case", P, N, B, flush=True)
    rng = np.random.default_rng(P + N + B)
    base = synth.uneven_population(rng, (24, 24), (N, N), (1, 1), with_inputs=False)
    who = rng.integers(0, base.P, P)
    nodes, conns = base.nodes[who].copy(), base.conns[who].copy()
    x = rng.standard_normal((P, B, base.I), dtype=np.float32)
    tn, tc, tx = (torch.from_numpy(a).cuda() for a in (nodes, conns, x))
    _, _, _, prog = neat.topo_sort(tn, tc, base.I, base.O, want_order=False)
    d = neat.dims_of(tn, tc, base.I, base.O)
    untuned = neat.forward(d, prog, tx, B)
    y = torch.empty_like(untuned)
    v, ms = neat.autotune_forward(d, prog, tx, B, outputs=y, reps=3)
    vt = neat.tuned_variant(d, B, throughput=True)
    print("recorded", v, vt, ms, flush=True)
    assert all(m > 0 for m in ms) and neat.tuned_variant(d, B) == v
    for got, times in ((v, ms[:5]), (vt, ms[5:])):
        assert got == neat.FWD_AUTO or times[CANDIDATES.index(got)] == min(times)
    tuned = neat.forward(d, prog, tx, B, variant=neat.FWD_TUNED)
    plan = neat.BatchPlan()
    yb, yc = torch.empty_like(untuned), torch.empty_like(untuned)
    plan.run([neat.batch_item(d, prog, yb, inputs=tx, B=B),
              neat.batch_item(d, prog, yc, inputs=tx, B=B)])
    torch.cuda.synchronize()
    for got, name, var in ((y, "outputs", v), (tuned, "tuned", v), (yb, "batch", vt)):
        if var == neat.FWD_SEG:
            y64, beta = oracle.forward(nodes[:8], conns[:8], x[:8], base.I, base.O)
            assert_parity(got[:8].cpu().numpy(), y64, beta, name)
        else:
            assert torch.equal(got.view(torch.int32), untuned.view(torch.int32)), name
    plan.free()
