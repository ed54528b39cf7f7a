"""CPU: the forward planner (forward_plan and the rules of NEAT_FWD_AUTO,
csrc/forward.hip), called from a small host program linked against libneat.so
(tests/plan_probe.cpp): what each call launches, without a GPU."""
from __future__ import annotations

import json
import os
import subprocess

import numpy as np
import pytest

import paper_2404_01817_amd as neat
from paper_2404_01817_amd._lib import LIB_PATH

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LDS = 163840
AS_IS, GRAPH, IN_ORDER, TUNE_ALONE, TUNE_FULL = -1, 0, 1, 2, 3


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    if not os.path.exists(LIB_PATH):
        from paper_2404_01817_amd import build
        build.build()
    exe = str(tmp_path_factory.mktemp("plan") / "plan_probe")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", rocm + "/include",
                        "-I", os.path.join(ROOT, "include"),
                        "-I", os.path.join(ROOT, "paper_2404_01817_amd", "csrc"),
                        os.path.join(ROOT, "tests", "plan_probe.cpp"), LIB_PATH,
                        "-Wl,-rpath," + os.path.dirname(LIB_PATH) + ":" + rocm + "/lib", "-L", rocm + "/lib",
                        "-lamdhip64", "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr

    def run(plans):
        """plans: (how, jobs); job: dict of P, N, B, and optionally C, I, O, side, variant,
        recurrent, aligned."""
        text = ""
        for how, jobs in plans:
            text += "%d %d %d\n" % (how, LDS, len(jobs))
            for j in jobs:
                full = dict(dict(C=4 * j["N"], I=5, O=2, side=0, variant=neat.FWD_AUTO, recurrent=0,
                                 aligned=1), **j)
                text += " ".join(str(full[k]) for k in ("P", "N", "C", "I", "O", "B", "side",
                                                        "variant", "recurrent", "aligned")) + "\n"
        r = subprocess.run([exe], input=text, capture_output=True, text=True, timeout=60)
        assert r.returncode == 0, r.stderr
        out = [json.loads(l) for l in r.stdout.splitlines()]
        assert len(out) == len(plans)
        return out
    return run


def kinds(p):
    return [l["kind"] for l in p["launches"]]


PER_CLASS = {50: [], 100: ["r128"], 200: ["r128", "r224"], 300: ["r128", "r224", "lds"]}


@pytest.mark.parametrize("how", [AS_IS, GRAPH, IN_ORDER])
@pytest.mark.parametrize("N", sorted(PER_CLASS))
@pytest.mark.parametrize("P,B", [(3, 1), (50, 65), (4000, 300)])
def test_explicit_variants_are_launches_per_class(plan, how, N, P, B):
    """NEAT_FWD_REG and NEAT_FWD_REG2 mean the stores that their names say,
    alone and beside other populations, whatever the sizes."""
    for variant, first in ((neat.FWD_REG, "r64"), (neat.FWD_REG2, "r64x2")):
        for others in ([], [dict(P=7, N=60, B=3, variant=neat.FWD_SEG)]):
            got, = plan([(how, [dict(P=P, N=N, B=B, variant=variant)] + others)])
            assert got["rc"] == 0
            assert kinds(got) == [first] + PER_CLASS[N] + (["seg"] if others else [])


CANDIDATES = [neat.FWD_REG, neat.FWD_REG2, neat.FWD_LDS, neat.FWD_LVL, neat.FWD_SEG]


@pytest.mark.parametrize("N", [8, 30, 31, 62, 63, 126, 140, 151, 222, 223, 300, 500, 1000])
def test_the_autotuner_times_what_untuned_calls_launch(plan, N):
    """For every population the launches of NEAT_FWD_AUTO, alone and beside others on one
    stream, are those of a timed candidate, or timed beside them."""
    plans, sizes = [], []
    for P in (1, 40, 700, 5000, 40000):
        for B in (1, 9, 64, 65, 192, 1000):
            job = dict(P=P, N=N, B=B, I=4, O=2)
            full = max(1, min(64, -(-16384 // (P * -(-B // 64)))))
            for copies, how, tune in ((1, IN_ORDER, TUNE_ALONE), (full, IN_ORDER, TUNE_FULL)):
                if copies == 1 and tune == TUNE_FULL:
                    continue
                sizes.append((P, B, copies))
                plans.append((how, [job] * copies))
                plans.append((tune, [job] * copies))
                plans += [(AS_IS, [dict(job, variant=v)] * copies) for v in CANDIDATES]
    out = plan(plans)
    step = 2 + len(CANDIDATES)
    own = 0
    for k, size in enumerate(sizes):
        untuned, tuned, *cands = out[step * k:step * k + step]
        if tuned["tune"] == -1:
            assert any(c["launches"] == untuned["launches"] for c in cands), size
        else:
            own += 1
            assert tuned["launches"] == untuned["launches"], size
            assert all(c["launches"] != untuned["launches"] for c in cands), size
    # four samples per lane, and one launch for every class, are no candidate's (past 740 rows
    # every population goes by levels)
    assert (own > 0) == (N <= 30 or 62 < N <= 740)


def test_batches_are_refused_exactly_when_their_launches_per_class_are(plan):
    """Populations whose inputs and outputs fit a wave's LDS one by one and not together, and
    others near that limit: what a batch launches for them by size changes nothing in what is
    accepted."""
    rng = np.random.default_rng(5)
    lists = [[dict(P=100, N=400, I=300, O=10, B=64), dict(P=100, N=400, I=10, O=300, B=1000)],
             [dict(P=100, N=310, I=300, O=10, B=100), dict(P=100, N=310, I=10, O=300, B=100)]]
    for _ in range(400):
        jobs = []
        for _ in range(rng.integers(2, 5)):
            N = int(rng.choice([130, 200, 320, 400, 640, 1000]))
            I = int(rng.integers(1, min(N - 1, 340)))
            jobs.append(dict(P=int(rng.choice([1, 100, 5000])), N=N, I=I,
                             O=int(rng.integers(1, min(N - I, 340) + 1)),
                             B=int(rng.choice([5, 64, 65, 1000]))))
        lists.append(jobs)
    for how in (GRAPH, IN_ORDER):
        out = plan([(AS_IS, l) for l in lists] + [(how, l) for l in lists])
        n = len(lists)
        codes = [(a["rc"], b["rc"]) for a, b in zip(out[:n], out[n:])]
        assert all(a == b for a, b in codes), [l for l, (a, b) in zip(lists, codes) if a != b][:3]
        assert len(set(codes)) == 2  # some are accepted and some refused
        assert all(l["lds"] <= LDS for p in out for l in p["launches"])


@pytest.mark.parametrize("B,samples", [(64, 64), (65, 128), (5000, 128)])
@pytest.mark.parametrize("N", [1000, 1024])
def test_grid_queries_up_to_the_lds_of_their_staging(plan, N, B, samples):
    """A wave holds a tile's five inputs, 256 coordinates and a tile's outputs: every O for
    which these fit is accepted, with the table of the samples' offsets beside them, or where
    that does not fit by tiles of half the samples or by LDS rows."""
    top = (LDS // 4 - 256 - 5 * samples) // samples  # outputs
    outs = [1, 100, top - 2, top - 1, top, top + 1]
    got = plan([(AS_IS, [dict(P=3, N=N, I=5, O=O, B=B, side=16)]) for O in outs])
    small = "r64" if samples == 64 else "r64x2"
    for O, g in zip(outs, got):
        assert (g["rc"] == 0) == (O <= top), O
        if O < top:
            assert kinds(g) == [small, "r128", "r224", "lds32"]
        elif O == top:
            assert kinds(g) == (["lds32"] if samples == 64 else ["r64", "r128", "r224", "lds32"])
            assert [i["cls"] for l in g["launches"] for i in l["items"]] == \
                ([-1] if samples == 64 else [0, 1, 2, 3])
        for l in g["launches"]:
            s = {"r64x2": 128, "lds": 0, "lds32": 0}.get(l["kind"], 64)
            assert not s or l["wave_floats"] == s * (6 + O) + 256


def test_wave_areas_start_at_16_bytes(plan):
    """Inputs arrive in LDS and outputs leave it 16 bytes at a time: every wave's area and its
    output staging start at a multiple of that, whatever the rows of the level mapping that
    may share them."""
    plans = [(how, [dict(P=P, N=N, I=I, O=O, B=B, variant=v)])
             for how in (AS_IS, IN_ORDER) for v in (neat.FWD_AUTO, neat.FWD_REG)
             for N in (31, 63, 127, 223, 365, 511, 512, 513, 601, 1022, 1023, 1024)
             for I, O in ((1, 1), (3, 2), (9, 4)) for P in (3, 2500)
             for B in (1, 2, 3, 30, 70, 300)]
    for (_, (job,)), got in zip(plans, plan(plans)):
        assert got["rc"] == 0
        for l in got["launches"]:
            if l["kind"] in ("lvl", "seg"):
                continue  # words only
            assert l["wave_floats"] % 4 == 0 and l["stage_floats"] % 4 == 0, (job, l)


# (P, N, B), what a call's only population launches: both sides of every line of the rule
ALONE = [
    ((3072, 31, 64), ["r64"]), ((1536, 50, 100), ["r64"]), ((1537, 50, 100), ["r64x2"]),
    ((1024, 62, 192), ["r64"]), ((1025, 62, 192), ["r64x2"]), ((2731, 62, 192), ["r64"]),
    ((2730, 62, 192), ["r64x2"]), ((100, 30, 100), ["r64x2"]),
    ((3000, 120, 4), ["r64", "r128"]), ((3000, 121, 4), ["lvl"]), ((3000, 121, 9), ["r64", "r128"]),
    ((2000, 130, 4), ["any"]), ((2000, 131, 4), ["lvl"]),
    ((2048, 130, 64), ["any"]), ((2049, 130, 64), ["r64", "r128", "r224"]),
    ((2049, 131, 64), ["any"]), ((8192, 150, 64), ["any"]),
    ((8193, 150, 64), ["r64", "r128", "r224"]), ((8193, 151, 64), ["any"]),
    ((512, 200, 32), ["lvl"]), ((513, 200, 32), ["any"]), ((2000, 510, 300), ["any"]),
    ((100, 530, 300), ["lvl"]), ((101, 530, 300), ["r64x2", "r128", "r224", "lds"]),
    ((2000, 530, 32), ["any"]), ((2000, 530, 33), ["r64", "r128", "r224", "lds"]),
    ((300, 531, 300), ["lvl"]), ((301, 660, 300), ["r64x2", "r128", "r224", "lds32"]),
    ((2000, 640, 64), ["any"]), ((2000, 640, 65), ["r64x2", "r128", "r224", "lds32"]),
    ((1000, 661, 300), ["lvl"]), ((1001, 740, 300), ["any"]), ((9000, 741, 300), ["lvl"]),
]


def test_a_lone_population_takes_the_mapping_measured_best(plan):
    out = plan([(GRAPH, [dict(P=P, N=N, B=B)]) for (P, N, B), _ in ALONE])
    got = {k: kinds(o) for (k, _), o in zip(ALONE, out)}
    assert got == dict(ALONE)


def test_several_populations_past_510_rows(plan):
    other = dict(P=9, N=20, B=5)
    for how in (GRAPH, IN_ORDER):
        for (P, N, B), want in [((500, 530, 32), ["any"]),
                                ((500, 530, 33), ["r128", "r224", "lds"]),
                                ((500, 640, 64), ["any"]), ((500, 640, 16), ["lvl"]),
                                ((500, 640, 300), ["r64x2", "r128", "r224", "lds32"]),
                                ((500, 661, 300), ["lvl"]), ((50000, 900, 300), ["lvl"])]:
            got, = plan([(how, [dict(P=P, N=N, B=B), other])])
            assert [k for k in kinds(got) if k != "r64"] == want, (how, P, N, B)


def test_launches_come_in_the_order_of_the_kernels(plan):
    """Whatever the order of the jobs (in-order batches run them so)."""
    jobs = [dict(P=10, N=300, B=300, variant=neat.FWD_REG2), dict(P=10, N=20, B=5),
            dict(P=10, N=40, I=5, O=1, B=50, side=16), dict(P=9, N=100, B=3, variant=neat.FWD_SEG),
            dict(P=9, N=100, B=3, variant=neat.FWD_LVL), dict(P=3000, N=30, B=500)]
    a, b = plan([(AS_IS, jobs), (AS_IS, jobs[::-1])])
    order = [(l["kind"], l["grid_mode"]) for l in a["launches"]]
    assert order == [("r64", 0), ("r64", 1), ("r64x2", 0), ("r128", 0), ("r224", 0), ("lds", 0),
                     ("lvl", 0), ("seg", 0), ("r32x4", 0)]
    assert [(l["kind"], l["grid_mode"]) for l in b["launches"]] == order


def test_one_population_is_one_item_of_every_launch(plan):
    """A call over one population passes its items inline: no launch of it may hold two."""
    sizes = [(N, O) for N in (8, 30, 31, 62, 63, 127, 223, 330, 700, 1000, 1024)
             for O in (1, 2, 20, 312, 313, 314, 629, 630, 631, 900) if 5 + O <= N]
    plans = [(how, [dict(P=P, N=N, O=O, B=B, side=side, variant=v)])
             for N, O in sizes for side in (0, 3, 16) for P in (1, 5000) for B in (1, 64, 65, 300)
             for how, v in ((AS_IS, neat.FWD_AUTO), (GRAPH, neat.FWD_AUTO), (AS_IS, neat.FWD_REG),
                            (AS_IS, neat.FWD_REG2), (AS_IS, neat.FWD_LDS), (AS_IS, neat.FWD_LVL),
                            (AS_IS, neat.FWD_SEG))]
    accepted = 0
    for (_, (job,)), got in zip(plans, plan(plans)):
        accepted += got["rc"] == 0
        assert all(len(l["items"]) == 1 for l in got["launches"]), (job, kinds(got))
    assert accepted > len(plans) // 2
