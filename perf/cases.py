"""The work that a program built on this framework has it do, as cases that can be timed.

A case is a dict of plain values.  ``kind`` names the entry points that its pass goes through:

* ``step``: the transformation and the calculation of one population, as an evaluation loop
  calls them (``topo_sort``, ``forward``);
* ``batch``: many uneven populations in one recorded batch (``BatchPlan``), their
  transformations included;
* ``serve``: a burst of requests for resident populations (``Server``), until its last result;
* ``grid``: CPPN queries over all pairs of a substrate's points (``forward_grid``);
* ``substrate``: CPPN weights and the substrate layer (``substrate_forward``);
* ``recurrent``: the transformation and K sweeps of networks with cycles
  (``topo_sort(recurrent=True)``, ``forward_recurrent``);
* ``species``: compatibility distances to the species' representatives (``distance``);
* ``offspring``: children by crossover and their mutations (``crossover``, ``edit``).

Everything is float32, the one type that the framework computes in.  Buffers that a program
keeps from one generation to the next (programs, status words, outputs) are made in
``prepare``.
"""
from __future__ import annotations

import math

import torch

import paper_2404_01817_amd as neat

# codes of the node encoding
IDENTITY, TANH, SIGMOID, RELU, SIN, GAUSS, ABS = range(7)
SUM, PRODUCT, MAX, MIN, MEAN = range(5)
CONTROL_ACTS = (SIGMOID, TANH, RELU, IDENTITY, SIN)
CPPN_ACTS = (SIN, GAUSS, ABS, TANH, SIGMOID)
ALL_AGGS = (SUM, PRODUCT, MAX, MIN, MEAN)
DEVICE = "cuda"


def listed():
    return [
        # the smallest evaluation: 16 tiny networks on 32 shared inputs, where only latency counts
        {"name": "step_tiny", "kind": "step", "P": 16, "N": 8, "C": 16, "I": 3, "O": 1, "B": 32,
         "shared": True, "order": False},
        # a small experiment with odd sizes, order and levels wanted (a program that inspects
        # its networks)
        {"name": "step_small_odd", "kind": "step", "P": 157, "N": 37, "C": 149, "I": 11, "O": 3,
         "B": 321, "shared": False, "order": True},
        # a control policy search at the paper's largest population: 17 observations, 6 actions
        {"name": "step_control", "kind": "step", "P": 10000, "N": 50, "C": 200, "I": 17, "O": 6,
         "B": 1000, "shared": False, "order": False},
        # large networks on few inputs each
        {"name": "step_large_nets", "kind": "step", "P": 700, "N": 365, "C": 1460, "I": 20, "O": 6,
         "B": 18, "shared": False, "order": False},
        # an experiment server that evaluates 24 searches of unlike sizes at once
        {"name": "batch_uneven", "kind": "batch", "pops": 24, "P": 2048, "N": 400, "B": 512,
         "mix": 7},
        # 16 resident populations and a burst of 48 requests
        {"name": "serve_burst", "kind": "serve", "pops": 16, "P": 2048, "N": 256, "B": 256,
         "requests": 48, "mix": 3},
        # HyperNEAT: the weights of 1000 substrates of 16 x 16 points
        {"name": "grid_cppn", "kind": "grid", "P": 1000, "N": 30, "C": 120, "side": 16,
         "first": 0, "Q": 65536},
        # HyperNEAT: weights and layer of 500 substrates, 256 input planes
        {"name": "substrate_layer", "kind": "substrate", "P": 500, "N": 30, "C": 120, "side": 16,
         "B": 256, "theta": 0.2},
        # recurrent control policies, four sweeps
        {"name": "recurrent_control", "kind": "recurrent", "P": 5000, "N": 50, "C": 200, "I": 17,
         "O": 6, "B": 500, "K": 4},
        # speciation of 10000 genomes against 64 species
        {"name": "species_control", "kind": "species", "P": 10000, "N": 50, "C": 200, "Q": 64},
        # the next generation of 10000 genomes, 8 edits each
        {"name": "offspring_control", "kind": "offspring", "P": 10000, "N": 50, "C": 200,
         "edits": 8},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: a kind, then sizes over its range, the whole no larger than its listed
    case."""
    kind = rng.choice(("step", "step", "step", "batch", "serve", "grid", "substrate",
                       "recurrent", "species", "offspring"))
    if kind in ("step", "recurrent"):
        N = _log_int(rng, 8, 400 if kind == "step" else 160)
        I = rng.randint(2, min(24, N // 2))
        O = rng.randint(1, min(8, N - I - 1))
        B = _log_int(rng, 1, 1000)
        top = 8e6 if kind == "step" else 2e6  # genome-inputs of networks of 50 rows
        P = max(16, min(_log_int(rng, 16, 10000), int(top * 50 / (max(B, 100) * N))))
        case = {"kind": kind, "P": P, "N": N, "C": rng.randint(2 * N, 4 * N), "I": I, "O": O,
                "B": B}
        if kind == "recurrent":
            return dict(case, K=rng.randint(1, 6))
        return dict(case, shared=rng.random() < 0.25, order=rng.random() < 0.25)
    if kind == "batch":
        return {"kind": kind, "pops": rng.randint(2, 24), "P": _log_int(rng, 100, 2048),
                "N": _log_int(rng, 10, 400), "B": _log_int(rng, 1, 512),
                "mix": rng.randrange(1 << 20)}
    if kind == "serve":
        return {"kind": kind, "pops": rng.randint(2, 16), "P": _log_int(rng, 64, 2048),
                "N": _log_int(rng, 10, 256), "B": _log_int(rng, 1, 256),
                "requests": rng.randint(1, 48), "mix": rng.randrange(1 << 20)}
    if kind == "grid":
        side = rng.randint(5, 24)
        first = rng.randrange(side ** 4 // 2)
        Q = rng.randint(1, side ** 4 - first)
        N = rng.randint(10, 30)
        return {"kind": kind, "P": max(1, min(_log_int(rng, 16, 1000), 65536000 // Q)), "N": N,
                "C": rng.randint(2 * N, 4 * N), "side": side, "first": first, "Q": Q}
    if kind == "substrate":
        side = rng.choice((8, 16, 24, 32))
        B = _log_int(rng, 1, 400)
        P = min(_log_int(rng, 16, 500), int(500 * (16 / side) ** 4 * 256 / max(B, 256)))
        N = rng.randint(10, 30)
        return {"kind": kind, "P": P, "N": N, "C": rng.randint(2 * N, 4 * N), "side": side,
                "B": B, "theta": rng.choice((0.0, 0.2))}
    N = _log_int(rng, 8, 400)
    C = rng.randint(2 * N, 4 * N)
    P = min(_log_int(rng, 32, 10000), 10000 * 50 // N)
    if kind == "species":
        return {"kind": kind, "P": P, "N": N, "C": C, "Q": _log_int(rng, 1, 64)}
    return {"kind": kind, "P": P, "N": N, "C": C, "edits": rng.randint(1, 8)}


# ------------------------------------------------------------------ random populations
class Nets:
    """P random genomes: their tensors, and the same networks by topological index (inputs
    0 .. I-1, then the M = O + hidden computed nodes in an order that every edge follows), which
    is what ``exact`` evaluates."""


def _rand(g, *shape):
    return torch.rand(shape, generator=g, device=DEVICE)


def _pick(g, codes, *shape):
    return torch.tensor(codes, device=DEVICE)[torch.randint(len(codes), shape, generator=g,
                                                            device=DEVICE)]


def make_nets(g, P, N, C, I, O, acts, aggs, dense=False, recurrent=False):
    """Genomes with 0 .. N-I-O hidden nodes and 1 .. C connections (``dense``: 10 to 60 % of
    the possible ones), 70 % of them enabled; NaN rows anywhere.  Weights and biases are
    N(0, 1), responses 1, as the paper's experiments start from."""
    H = N - I - O
    R = I + O
    M = O + H
    n = Nets()
    n.P, n.N, n.C, n.I, n.O = P, N, C, I, O
    hid = torch.randint(H + 1, (P,), generator=g, device=DEVICE)
    m = hid + O  # computed nodes of each genome
    live = torch.arange(M, device=DEVICE) < m[:, None]
    # computed node j: outputs 0 .. O-1, then hidden ones with distinct increasing keys
    step = (16 * N - R) // max(H, 1)
    keys = torch.cat([torch.arange(I, R, device=DEVICE).expand(P, O),
                      R + step * torch.arange(H, device=DEVICE)
                      + torch.randint(max(step, 1), (P, H), generator=g, device=DEVICE)], 1)
    rows = torch.cat([torch.arange(I, R, device=DEVICE).expand(P, O),
                      R + _rand(g, P, H).argsort(1)], 1)
    bias = torch.randn((P, N), generator=g, device=DEVICE)
    act, agg = _pick(g, acts, P, N), _pick(g, aggs, P, N)
    every = torch.stack([torch.zeros_like(bias), bias, torch.ones_like(bias), act.float(),
                         agg.float()], 2)
    nodes = torch.full((P, N, 5), float("nan"), device=DEVICE)
    nodes[:, :I] = every[:, :I]
    nodes[:, :I, 0] = torch.arange(I, device=DEVICE)
    computed = torch.gather(every, 1, rows[:, :, None].expand(P, M, 5)).clone()
    computed[:, :, 0] = keys
    computed[~live] = float("nan")
    nodes.scatter_(1, rows[:, :, None].expand(P, M, 5), computed)
    # a random topological order of the computed nodes, absent ones last
    order = (_rand(g, P, M) + (~live) * 2.0).argsort(1)
    # connections: pairs drawn from the allowed ones, repeats dropped
    pairs = I * m + (m * m if recurrent else m * (m - 1) // 2)
    cap = pairs.clamp(max=C)
    share = 0.1 + 0.5 * _rand(g, P) if dense else _rand(g, P)
    count = ((share * cap).long() + 1).minimum(cap)
    q = (torch.rand((P, C), generator=g, device=DEVICE, dtype=torch.float64)
         * pairs[:, None]).long()
    q[torch.arange(C, device=DEVICE) >= count[:, None]] = 1 << 40
    q = q.sort(1).values
    there = q < (1 << 40)
    there[:, 1:] &= q[:, 1:] != q[:, :-1]
    q[~there] = 0
    from_in = q < (I * m)[:, None]
    r = q - (I * m)[:, None]
    mm = m[:, None].clamp(min=1)
    if recurrent:
        a, b = r // mm, r % mm
    else:
        b = ((1 + (1 + 8 * r.clamp(min=0).double()).sqrt()) / 2).long()
        b = torch.where(b * (b - 1) // 2 > r, b - 1, b)
        b = torch.where(b * (b + 1) // 2 <= r, b + 1, b)
        a = r - b * (b - 1) // 2
    # topological indices of the ends
    src = torch.where(from_in, q // mm, I + a.clamp(0, M - 1))
    dst = torch.where(from_in, q % mm, b).clamp(0, M - 1)
    on = _rand(g, P, C) < 0.7
    weight = torch.randn((P, C), generator=g, device=DEVICE)
    key_of = torch.cat([torch.arange(I, device=DEVICE).expand(P, I),
                        torch.gather(keys, 1, order)], 1)
    conns = torch.stack([torch.gather(key_of, 1, src).float(),
                         torch.gather(key_of, 1, I + dst).float(), on.float(), weight], 2)
    conns[~there] = float("nan")
    place = _rand(g, P, C).argsort(1)
    n.nodes = nodes.contiguous()
    n.conns = torch.gather(conns, 1, place[:, :, None].expand(P, C, 4)).contiguous()
    at = torch.gather(rows, 1, order)
    n.M, n.live = M, torch.gather(live, 1, order)
    n.bias, n.act, n.agg = (torch.gather(t, 1, at) for t in (bias, act, agg))
    n.src, n.dst, n.weight, n.on = src, dst, weight, there & on
    # topological index of every output
    n.out = I + torch.argsort(order, 1)[:, :O]
    return n


def _pops(case):
    """Sizes of the populations of a ``batch`` or ``serve`` case: the first has the case's rows and
    inputs, the others spread below them (fixed by ``mix``)."""
    r = torch.Generator().manual_seed(case["mix"])

    def below(hi, lo):
        lo = min(lo, hi)
        return int(round(lo * (hi / lo) ** float(torch.rand((), generator=r))))

    got = []
    for k in range(case["pops"]):
        # the largest networks and the longest inputs come with a smaller population
        P = below(case["P"], 100)
        N, B = (below(case["N"], 10), below(case["B"], 1)) if k else (case["N"], case["B"])
        I = 2 + int(float(torch.rand((), generator=r)) * (min(24, N // 2) - 1))
        O = 1 + int(float(torch.rand((), generator=r)) * min(8, N - I - 1))
        got.append((P, N, 4 * N, I, O, B))
    return got


def _requests(case):
    """(population, inputs per genome) of every request of a ``serve`` case."""
    r = torch.Generator().manual_seed(case["mix"] + 1)
    got = []
    for _ in range(case["requests"]):
        k = int(torch.randint(case["pops"], (), generator=r))
        got.append((k, int(round(case["B"] ** float(torch.rand((), generator=r))))))
    return got


def _family(g, P, N, C):
    """A population of relatives: each genome is one of up to 64 ancestors with new weights and
    a fifth of its hidden genes and connections lost."""
    A = min(64, P)
    I, O = max(1, min(17, N // 3)), max(1, min(6, N // 6))
    base = make_nets(g, A, N, C, I, O, CONTROL_ACTS, ALL_AGGS)
    who = torch.randint(A, (P,), generator=g, device=DEVICE)
    who[:A] = torch.arange(A, device=DEVICE)
    nodes, conns = base.nodes[who], base.conns[who]
    nodes[:, :, 1] += 0.3 * torch.randn((P, N), generator=g, device=DEVICE)
    conns[:, :, 3] += 0.3 * torch.randn((P, C), generator=g, device=DEVICE)
    gone = _rand(g, P, N) < 0.2
    gone[:, :I + O] = False
    nodes[gone] = float("nan")
    conns[_rand(g, P, C) < 0.2] = float("nan")
    return nodes.contiguous(), conns.contiguous()


def _edits(g, P, N, C, each):
    """``each`` mutations of every genome, sorted by genome: 36-byte records (genome, op, row,
    column, five values) as int32 words."""
    n = P * each
    rec = torch.zeros((n, 9), dtype=torch.int32, device=DEVICE)
    rec[:, 0] = torch.arange(n, device=DEVICE) // each
    # weights change most; genes are added and lost
    op = _pick(g, (5, 5, 5, 5, 4, 4, 2, 2, 3, 0, 1), n)
    node = (op == 0) | (op == 1) | (op == 4)
    rec[:, 1] = op
    rec[:, 2] = (_rand(g, n) * torch.where(node, N, C)).int()
    rec[:, 3] = torch.where(op == 4, 1, 3)
    v = torch.zeros((n, 5), device=DEVICE)
    weight = torch.randn(n, generator=g, device=DEVICE)
    fresh = torch.randint(16 * N, (n, 2), generator=g, device=DEVICE)
    v[:, 0] = torch.where((op == 0) | (op == 2), fresh[:, 0].float(), weight)
    v[:, 1] = torch.where(op == 2, fresh[:, 1].float(), weight)
    v[:, 2] = 1.0
    v[:, 3] = torch.where(op == 2, weight, 1.0)
    rec[:, 4:] = v.view(torch.int32)
    return rec.contiguous()


# ------------------------------------------------------------------ the program's side
class State:
    pass


def _gen(seed):
    return torch.Generator(device=DEVICE).manual_seed(seed)


def _inputs(case, seed):
    """Everything drawn from the seed: what ``prepare`` and ``exact`` share."""
    g, k, s = _gen(seed), case["kind"], State()
    if k in ("step", "recurrent"):
        large = case["N"] > 62
        s.nets = make_nets(g, case["P"], case["N"], case["C"], case["I"], case["O"], CONTROL_ACTS,
                           ALL_AGGS, dense=large, recurrent=k == "recurrent")
        shared = case.get("shared", False)
        shape = (case["B"], case["I"]) if shared else (case["P"], case["B"], case["I"])
        s.x = torch.randn(shape, generator=g, device=DEVICE)
    elif k in ("batch", "serve"):
        s.nets = [make_nets(g, P, N, C, I, O, CONTROL_ACTS, ALL_AGGS, dense=True)
                  for P, N, C, I, O, B in _pops(case)]
        if k == "batch":
            jobs = [(j, p[5]) for j, p in enumerate(_pops(case))]
        else:
            jobs = _requests(case)
        s.x = [torch.randn((s.nets[j].P, B, s.nets[j].I), generator=g, device=DEVICE)
               for j, B in jobs]
        s.jobs = jobs
    elif k in ("grid", "substrate"):
        s.nets = make_nets(g, case["P"], case["N"], case["C"], 5, 1, CPPN_ACTS, (SUM,))
        if k == "substrate":
            s.x = 2 * _rand(g, case["B"], case["side"] ** 2) - 1
    else:
        P, N, C = case["P"], case["N"], case["C"]
        s.nodes, s.conns = _family(g, P, N, C)
        if k == "species":
            who = torch.randint(P, (case["Q"],), generator=g, device=DEVICE)
            s.rnodes, s.rconns = s.nodes[who].contiguous(), s.conns[who].contiguous()
        else:
            s.pairs = torch.randint(P, (P, 2), generator=g, device=DEVICE, dtype=torch.int32)
            s.rn, s.rc = _rand(g, P, N), _rand(g, P, C)
            s.edits = _edits(g, P, N, C, case["edits"])
    return s


def _dims(n):
    return neat.dims_of(n.nodes, n.conns, n.I, n.O)


def _ints(n):
    return torch.empty(n, dtype=torch.int32, device=DEVICE)


def _program(d):
    return _ints(neat.program_bytes(d) // 4)


def prepare(case, seed):
    k, s = case["kind"], _inputs(case, seed)
    s.case = case
    if k in ("step", "recurrent", "grid", "substrate"):
        n = s.nets
        s.nodes, s.conns, s.I, s.O = n.nodes, n.conns, n.I, n.O
        s.d = _dims(n)
        s.status, s.program = _ints(n.P), _program(s.d)
        if k in ("grid", "substrate"):
            neat.topo_sort(n.nodes, n.conns, n.I, n.O, program=s.program, status=s.status,
                           want_order=False)
        S = case.get("side", 0) ** 2
        if k == "substrate":
            s.w = torch.empty((n.P, S, S), device=DEVICE)
            s.y = torch.empty((n.P, case["B"], S), device=DEVICE)
        else:
            s.y = torch.empty((n.P, case["Q"] if k == "grid" else case["B"], n.O), device=DEVICE)
    elif k == "batch":
        s.plan, s.items, s.y, s.status, s.keep = neat.BatchPlan(), [], [], [], []
        for n, x, (_, B) in zip(s.nets, s.x, s.jobs):
            d = _dims(n)
            program, status = _program(d), _ints(n.P)
            y = torch.empty((n.P, B, n.O), device=DEVICE)
            s.items.append(neat.batch_item(d, program, y, inputs=x, B=B, nodes=n.nodes,
                                           conns=n.conns, status=status))
            s.y.append(y)
            s.status.append(status)
            s.keep.append((program, n.nodes, n.conns))
    elif k == "serve":
        torch.cuda.synchronize()  # the server copies the populations on streams of its own
        s.server = neat.Server(cap_bytes=32 << 30, max_inflight=4)
        ids = [s.server.register(n.nodes, n.conns, n.I, n.O) for n in s.nets]
        s.y = [torch.empty((s.nets[j].P, B, s.nets[j].O), device=DEVICE) for j, B in s.jobs]
        s.requests = [s.server.request(ids[j], y, inputs=x, B=B, I=s.nets[j].I)
                      for (j, B), x, y in zip(s.jobs, s.x, s.y)]
    elif k == "species":
        s.y = torch.empty((case["P"], case["Q"]), device=DEVICE)
    else:
        s.cn, s.cc = torch.empty_like(s.nodes), torch.empty_like(s.conns)
        s.applied = _ints(s.edits.shape[0])
    if hasattr(s, "nets"):
        del s.nets  # what is left of the genomes is what the program holds
    return s


def run(s):
    c = s.case
    k = c["kind"]
    if k == "step":
        order, level, status, program = neat.topo_sort(
            s.nodes, s.conns, s.I, s.O, program=s.program, status=s.status,
            want_order=c["order"])
        y = neat.forward(s.d, program, s.x, c["B"], shared_inputs=c["shared"], outputs=s.y)
        return (y, status, order, level) if c["order"] else (y, status)
    if k == "recurrent":
        _, _, status, program = neat.topo_sort(
            s.nodes, s.conns, s.I, s.O, program=s.program, status=s.status, want_order=False,
            recurrent=True)
        return neat.forward_recurrent(s.d, program, s.x, c["B"], c["K"], outputs=s.y), status
    if k == "batch":
        s.plan.run(s.items)
        return s.y, s.status
    if k == "serve":
        for t in s.server.submit_many(s.requests):
            s.server.wait(t)
        return s.y
    if k == "grid":
        return neat.forward_grid(s.d, s.program, c["side"], c["first"], c["Q"], outputs=s.y)
    if k == "substrate":
        return neat.substrate_forward(s.d, s.program, c["side"], s.x, c["theta"], weights=s.w,
                                      outputs=s.y)
    if k == "species":
        return neat.distance(s.nodes, s.conns, s.rnodes, s.rconns, out=s.y)
    neat.crossover(s.nodes, s.conns, s.pairs, s.rn, s.rc, child_nodes=s.cn, child_conns=s.cc)
    neat.edit(s.cn, s.cc, s.edits, applied=s.applied)
    return s.cn, s.cc, s.applied


# ------------------------------------------------------------------ what it cannot do without
def _net_work(P, N, C, I, O, B, sort=True, sweeps=1, x_bytes=None, edges=None):
    """Genomes read once, inputs read once and outputs written once; two operations per enabled
    connection, two per computed node and about four for its activation."""
    hidden = (N - I - O) / 2
    if edges is None:
        edges = 0.7 * 0.5 * C
    flops = sweeps * P * B * (2 * edges + 6 * (O + hidden))
    x_bytes = 4 * P * B * I if x_bytes is None else x_bytes
    return (P * (20 * N + 16 * C + 4) * sort + x_bytes + 4 * P * B * O, flops)


def work(case):
    c, k = case, case["kind"]
    if k in ("step", "recurrent"):
        x = 4 * c["B"] * c["I"] if c.get("shared") else None
        b, f = _net_work(c["P"], c["N"], c["C"], c["I"], c["O"], c["B"],
                         sweeps=c.get("K", 1), x_bytes=x)
    elif k in ("batch", "serve"):
        pops = _pops(c)
        jobs = [(j, p[5]) for j, p in enumerate(pops)] if k == "batch" else _requests(c)
        each = [_net_work(*pops[j][:5], B, sort=k == "batch") for j, B in jobs]
        b, f = sum(e[0] for e in each), sum(e[1] for e in each)
    elif k == "grid":
        b, f = _net_work(c["P"], c["N"], c["C"], 5, 1, c["Q"], x_bytes=0)
    elif k == "substrate":
        S = c["side"] ** 2
        b, f = _net_work(c["P"], c["N"], c["C"], 5, 1, S * S, x_bytes=0)
        b += 4 * c["B"] * S + 4 * c["P"] * c["B"] * S
        f += 2 * c["P"] * c["B"] * S * S
    else:
        P, genome = c["P"], 20 * c["N"] + 16 * c["C"]
        if k == "species":
            b, f = (P + c["Q"]) * genome + 4 * P * c["Q"], P * c["Q"] * 3 * (c["N"] + c["C"])
        else:
            # two parents and the numbers read, the child written, the edits read
            b, f = P * (3 * genome + 4 * (c["N"] + c["C"]) + 40 * c["edits"]), 0
    return {"bytes": b, "flops": f}


# ------------------------------------------------------------------ the same in 64 bits
def _act64(z, code):
    """act_code(z) for z [G, B], code [G]."""
    out = torch.empty_like(z)
    fns = (lambda v: v, torch.tanh, torch.sigmoid, torch.relu, torch.sin,
           lambda v: torch.exp(-v * v), torch.abs)
    for a, fn in enumerate(fns):
        at = code == a
        out[at] = fn(z[at])
    return out


def _dense64(n, at):
    """Weights [G, M, I + M] of the enabled connections of genomes ``at`` and their mask."""
    G, T = at.numel(), n.I + n.M
    w = torch.zeros((G, n.M, T), dtype=torch.float64, device=DEVICE)
    on = torch.zeros((G, n.M, T), dtype=torch.bool, device=DEVICE)
    g, e = n.on[at].nonzero(as_tuple=True)
    d, s = n.dst[at][g, e], n.src[at][g, e]
    w[g, d, s] = n.weight[at][g, e].double()
    on[g, d, s] = True
    return w, on


def _node64(n, at, j, w, on, v):
    """Computed node j of every genome ``at`` from the values v [G, I + M, B]."""
    wj, oj, agg = w[:, j], on[:, j], n.agg[at, j]
    deg = oj.sum(1).double()
    z = torch.bmm(wj[:, None], v)[:, 0]
    mean = agg == MEAN
    z[mean] /= deg[mean].clamp(min=1)[:, None]
    for code in (PRODUCT, MAX, MIN):
        sel = ((agg == code) & (deg > 0)).nonzero()[:, 0]
        if sel.numel():
            t = wj[sel][:, :, None] * v[sel]
            none = ~oj[sel][:, :, None]
            if code == PRODUCT:
                z[sel] = t.masked_fill_(none, 1.0).prod(1)
            elif code == MAX:
                z[sel] = t.masked_fill_(none, -math.inf).amax(1)
            else:
                z[sel] = t.masked_fill_(none, math.inf).amin(1)
    z = z + n.bias[at, j].double()[:, None]
    return _act64(z, n.act[at, j])


def _forward64(n, x, sweeps=None):
    """Outputs [P, B, O] in 64 bits for inputs x [P or 1, B, I]."""
    P, B = n.P, x.shape[1]
    y = torch.empty((P, B, n.O), dtype=torch.float64, device=DEVICE)
    T = n.I + n.M
    step = max(1, min(P, int(2.5e8 / (T * (B + n.M)))))
    for p in range(0, P, step):
        at = torch.arange(p, min(P, p + step), device=DEVICE)
        G = at.numel()
        xs = x.expand(P, -1, -1)[p:p + G].double().transpose(1, 2)
        v = torch.zeros((G, T, B), dtype=torch.float64, device=DEVICE)
        v[:, :n.I] = xs
        w, on = _dense64(n, at)
        for _ in range(1 if sweeps is None else sweeps):
            prev = v if sweeps is None else v.clone()
            for j in range(n.M):
                v[:, n.I + j] = _node64(n, at, j, w, on, prev) * n.live[at, j][:, None]
        y[p:p + G] = torch.gather(v, 1, n.out[at][:, :, None].expand(G, n.O, B)).transpose(1, 2)
    return y


def _queries64(side, first, Q):
    c = (2.0 * torch.arange(side, device=DEVICE, dtype=torch.float64) - (side - 1)) / (side - 1)
    q = torch.arange(first, first + Q, device=DEVICE)
    a, b = q // side ** 2, q % side ** 2
    x = torch.stack([c[a % side], c[a // side], c[b % side], c[b // side], torch.ones_like(c[a % side])], 1)
    return x.float()[None]  # the coordinates are float32 numbers


def _genes64(nodes, conns):
    """Codes (NaN rows: -1) and columns of the node and connection genes."""
    def code(k):
        return torch.where(k.isnan(), torch.full_like(k, -1.0), k).long()
    nk, ck = code(nodes[:, :, 0]), code(conns[:, :, 0]) * (1 << 24) + code(conns[:, :, 1])
    ck[conns[:, :, 0].isnan()] = -1
    return (nk, nodes.double()), (ck, conns.double())


def _distance64(s):
    A, B = _genes64(s.nodes, s.conns), _genes64(s.rnodes, s.rconns)
    P, Q = s.nodes.shape[0], s.rnodes.shape[0]
    y = torch.zeros((P, Q), dtype=torch.float64, device=DEVICE)
    for kind in range(2):
        (ka, xa), (kb, xb) = A[kind], B[kind]
        na = (ka >= 0).sum(1)
        for q in range(Q):
            keys, at = kb[q].sort(stable=True)
            j = torch.searchsorted(keys, ka).clamp(max=keys.numel() - 1)
            hit = (keys[j] == ka) & (ka >= 0)
            z = xb[q][at[j]]
            if kind == 0:
                d = ((xa[..., 1] - z[..., 1]).abs() + (xa[..., 2] - z[..., 2]).abs()
                     + (xa[..., 3] != z[..., 3]) + (xa[..., 4] != z[..., 4]))
            else:
                d = (xa[..., 3] - z[..., 3]).abs() + (xa[..., 2] != z[..., 2])
            d = torch.where(hit, d, torch.zeros_like(d)).sum(1)
            nb = (kb[q] >= 0).sum()
            most = torch.maximum(na, nb)
            total = 1.0 * (na + nb - 2 * hit.sum(1)) + 0.5 * d
            y[:, q] += torch.where(most > 0, total / most.clamp(min=1), torch.zeros_like(total))
    return y


def exact(case, seed):
    k, s = case["kind"], _inputs(case, seed)
    if k == "step":
        x = s.x[None] if case["shared"] else s.x
        y = _forward64(s.nets, x)
        return (y, None, None, None) if case["order"] else (y, None)
    if k == "recurrent":
        return _forward64(s.nets, s.x, sweeps=case["K"]), None
    if k in ("batch", "serve"):
        y = [_forward64(s.nets[j], x) for (j, _), x in zip(s.jobs, s.x)]
        return (y, [None] * len(y)) if k == "batch" else y
    if k == "grid":
        return _forward64(s.nets, _queries64(case["side"], case["first"], case["Q"]))
    if k == "substrate":
        S = case["side"] ** 2
        w = _forward64(s.nets, _queries64(case["side"], 0, S * S)).view(-1, S, S)
        pruned = torch.where(w.abs() < case["theta"], torch.zeros_like(w), w)
        x = s.x.double()
        return torch.stack([torch.tanh(x @ p) for p in pruned]), w
    if k == "species":
        return _distance64(s)
    return None  # genes are moved, not computed
