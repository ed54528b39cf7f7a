"""GPU: edit lists that are not sorted by genome.  What applies is a run at the
front of a genome's part of the list; every entry of applied is written, and the
call costs about what a sorted list costs (shuffled lists of 80,000 edits once
took 15 ms for 20 us, growing with the square of the list)."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import paper_2404_01817_amd as neat

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _orders(rng, g):
    yield "sorted", g
    yield "shuffled", rng.permutation(g)
    yield "reversed", g[::-1].copy()
    yield "two halves", np.r_[g[::2], g[1::2]]
    yield "last first", np.r_[g[-1:], g[:-1]]
    yield "large then small", np.r_[np.full(len(g) // 2, g.max()), np.zeros_like(g[len(g) // 2:])]


@pytest.mark.parametrize("out_of_range", [False, True])
@pytest.mark.parametrize("P,n", [(1, 300), (7, 65), (300, 64), (300, 4097), (20000, 400000)])
def test_any_order(P, n, out_of_range):
    N, C = 5, max(16, 2 * n // P + 2)
    C = min(C, 400)
    rng = np.random.default_rng(P + n)
    genomes = np.sort(rng.integers(-2 if out_of_range else 0, P + 3 if out_of_range else P, n))
    for name, g in _orders(rng, genomes.astype(np.int32)):
        print("case", P, n, out_of_range, name, flush=True)
        e = np.zeros(n, oracle.EDIT_DTYPE)
        e["genome"], e["op"], e["column"] = g, oracle.CONN_SET, 3
        # a place of its own for every edit of a genome, as far as there are rows
        order = np.argsort(g, kind="stable")
        first = np.r_[0, np.flatnonzero(np.diff(g[order])) + 1]
        nth = np.empty(n, np.int64)
        nth[order] = np.arange(n) - np.repeat(first, np.diff(np.r_[first, n]))
        e["row"] = nth % C
        e["v"][:, 0] = np.arange(n)
        conns = torch.zeros((P, C, 4), device="cuda")
        nodes = torch.zeros((P, N, 5), device="cuda")
        te = torch.from_numpy(e.view(np.uint8).copy()).cuda()
        applied = torch.full((n,), 7, dtype=torch.int32, device="cuda")
        neat.edit(nodes, conns, te, applied=applied)
        ga, gc = applied.cpu().numpy(), conns.cpu().numpy()
        inside = (g >= 0) & (g < P)
        assert set(np.unique(ga)) <= {0, 1} and not ga[~inside].any()
        if name == "sorted":
            assert ga[inside].all()
        want = np.zeros((P, C, 4), np.float32)
        for k in np.flatnonzero(ga):
            want[g[k], e["row"][k], 3] = k
        assert np.array_equal(gc, want)
        # the applied edits of a genome lie side by side
        for x in np.unique(g[ga == 1])[:50]:
            at = np.flatnonzero((ga == 1) & (g == x))
            assert at[-1] - at[0] == len(at) - 1
        a, b = torch.cuda.Event(True), torch.cuda.Event(True)
        a.record()
        neat.edit(nodes, conns, te, applied=applied)
        b.record()
        torch.cuda.synchronize()
        print("us", 1e3 * a.elapsed_time(b), flush=True)
        if P == 20000:
            assert a.elapsed_time(b) < 30.0  # ms
