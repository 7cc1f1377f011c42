"""GPU parity of the incremental FlowCutter path (maximal sink side,
piercing with warm-started flows, the FlowCutter loop) against the CPU
oracle, through the C ABI.

Every quantity compared is determined by the terminal sets alone (flow
value, minimal source side, maximal sink side) or by the deterministic
piercing rule on top of them (the FlowCutter trace), so the GPU must match
the oracle exactly although it warm starts and the oracle solves every
iteration from scratch.
"""
import json
import os
import sys

import numpy as np
import pytest

from paper_2201_01556_amd import inputs

pytestmark = pytest.mark.gpu

HERE = os.path.dirname(os.path.abspath(__file__))


def _say(msg):
    print(f"[gpu-cutter] {msg}", flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def hf():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2201_01556_amd import hyperflow
    hyperflow.load_library()
    return hyperflow


def _with_terminals(hg, S, T):
    return inputs.Hypergraph(hg.num_vertices, hg.net_offsets, hg.pins, hg.net_weights,
                             hg.vertex_weights, np.asarray(sorted(S), dtype=np.int32),
                             np.asarray(sorted(T), dtype=np.int32))


def balance_limit(total):
    """floor(103 * ceil(c(V) / 2) / 100): eps = 0.03 on two blocks."""
    return (103 * (-(-int(total) // 2))) // 100


@pytest.mark.parametrize("block", range(2))
def test_sink_side_tiny_vs_oracle(hf, oracle_mod, block):
    for seed in range(block * 150, block * 150 + 150):
        hg = inputs.tiny_hypergraph(seed)
        _say(f"tiny seed {seed}")
        r = oracle_mod.maxflow(hg, sink_side=True)
        with hf.FlowProblem.from_hypergraph(hg) as p:
            assert p.solve() == r.flow
            t = p.sink_side()
        assert (t.astype(bool) == r.sink_side.astype(bool)).all(), seed


def test_sink_side_uniform_vs_oracle(hf, oracle_mod):
    for seed in range(10):
        hg = inputs.uniform_hypergraph(seed)
        r = oracle_mod.maxflow(hg, sink_side=True)
        with hf.FlowProblem.from_hypergraph(hg, group_lanes=[4, 8, 16][seed % 3]) as p:
            assert p.solve() == r.flow
            t = p.sink_side()
        assert (t.astype(bool) == r.sink_side.astype(bool)).all(), seed


@pytest.mark.parametrize("side", [0, 1])
def test_pierce_warm_start_vs_oracle(hf, oracle_mod, side):
    """Solve, pierce (S_r or T_r plus one vertex), solve again warm with the
    invariant checker on: flow and both sides equal a fresh oracle solve of
    the new terminal sets."""
    for seed in range(12):
        hg = inputs.uniform_hypergraph(seed, num_vertices=600, num_nets=900, num_sources=20,
                                       num_sinks=20)
        _say(f"pierce side {side} seed {seed}")
        with hf.FlowProblem.from_hypergraph(hg, debug_checks=1) as p:
            p.solve()
            vs, _ = p.source_side()
            ts = p.sink_side()
            free = np.nonzero(~vs.astype(bool) & ~ts.astype(bool))[0]
            pick = int(free[len(free) // 2]) if free.size else None
            if side == 0:
                S = set(np.nonzero(vs)[0].tolist()) | ({pick} if pick is not None else set())
                T = set(hg.sinks.tolist())
            else:
                S = set(hg.sources.tolist())
                T = set(np.nonzero(ts)[0].tolist()) | ({pick} if pick is not None else set())
            p.pierce(side, [] if pick is None else [pick])
            F = p.solve()
            vs2, ns2 = p.source_side()
            ts2 = p.sink_side()
        r = oracle_mod.maxflow(_with_terminals(hg, S, T), sink_side=True)
        assert F == r.flow, seed
        assert (vs2.astype(bool) == r.vertex_side.astype(bool)).all(), seed
        assert (ns2 == r.net_side).all(), seed
        assert (ts2.astype(bool) == r.sink_side.astype(bool)).all(), seed


def test_pierce_errors(hf):
    hg = inputs.uniform_hypergraph(3, num_vertices=300, num_nets=450, num_sources=10,
                                   num_sinks=10)
    with hf.FlowProblem.from_hypergraph(hg) as p:
        with pytest.raises(hf.HyperflowError) as ei:
            p.pierce(0, [1])
        assert ei.value.name == "FP_ERR_STATE"
        F = p.solve()
        with pytest.raises(hf.HyperflowError) as ei:
            p.pierce(0, [int(hg.sinks[0])])
        assert ei.value.name == "FP_ERR_INVALID"
        with pytest.raises(hf.HyperflowError) as ei:
            p.pierce(1, [hg.num_vertices])
        assert ei.value.name == "FP_ERR_INVALID"
        # nothing changed: the handle is still solved with the same flow
        assert p.solve() == F


def _cutter_cases():
    with open(os.path.join(HERE, "golden", "flowcutter.json")) as f:
        return json.load(f)["cases"]


@pytest.mark.parametrize("case", _cutter_cases(), ids=lambda c: c["name"])
def test_flowcutter_fixtures(hf, case):
    hg = inputs.hypergraph_from_nets(case["V"], case["nets"], case["w"], case["S"], case["T"])
    c = np.asarray(case.get("c", np.ones(case["V"])))
    with hf.FlowProblem.from_hypergraph(hg) as p:
        res, x, trace = p.flowcutter(c, case["max_source"], case["max_sink"],
                                     bulk_percent=case.get("bulk_percent", 0),
                                     most_balanced=case.get("most_balanced", False))
    if "first_balanced" in case:
        assert res["first_balanced"] == case["first_balanced"]
    assert res["status"] == case["status"]
    assert res["flow"] == case["F"]
    assert res["iterations"] == case["iterations"]
    assert np.nonzero(x)[0].tolist() == case["x"]
    assert [list(t) for t in trace] == case["trace"]
    counts = case.get("counts", [1] * (case["iterations"] - 1) + [0])
    assert res["counts"] == counts


def _compare_cutter(hf, oracle_mod, hg, c, Ls, Lt, max_iter, tag, bulk_percent=0,
                    most_balanced=False, **opts):
    ref = oracle_mod.flowcutter(hg, c, Ls, Lt, max_iterations=max_iter,
                                bulk_percent=bulk_percent, most_balanced=most_balanced)
    with hf.FlowProblem.from_hypergraph(hg, **opts) as p:
        res, x, trace = p.flowcutter(c, Ls, Lt, max_iterations=max_iter,
                                     bulk_percent=bulk_percent, most_balanced=most_balanced)
    assert res["iterations"] == ref.iterations, tag
    assert res["first_balanced"] == ref.first_balanced, tag
    assert [tuple(t) for t in trace] == [tuple(t) for t in ref.trace], tag
    assert res["counts"] == ref.counts, tag
    assert res["status"] == ref.status, tag
    assert res["flow"] == ref.flow, tag
    assert (x.astype(bool) == ref.vertex_side.astype(bool)).all(), tag
    return res


def _random_region(seed):
    """14..23 vertices, 1..3 nets per vertex of 2..3 pins, unit weights;
    source 0, sink V-1 (shapes on which bulk piercing triggers)."""
    rng = np.random.default_rng(seed)
    V = int(rng.integers(14, 24))
    E = int(rng.integers(V, 3 * V))
    nets = [sorted(rng.choice(V, int(rng.integers(2, 4)), replace=False).tolist())
            for _ in range(E)]
    return inputs.hypergraph_from_nets(V, nets, [1] * E, [0], [V - 1])


def test_flowcutter_bulk_small_vs_oracle(hf, oracle_mod):
    """Bulk piercing (beta 55 %) on 120 small regions against the oracle,
    trace, pierced counts and result; some of them bulk-pierce."""
    bulked = 0
    for seed in range(120):
        hg = _random_region(seed)
        c = np.ones(hg.num_vertices)
        L = (hg.num_vertices + 1) // 2
        res = _compare_cutter(hf, oracle_mod, hg, c, L, L, 100, f"bulk small {seed}",
                              bulk_percent=55, debug_checks=1 if seed % 7 == 0 else 0)
        bulked += max(res["counts"]) > 1
    assert bulked >= 3


@pytest.mark.parametrize("seed", range(3))
def test_flowcutter_bulk_uniform_vs_oracle(hf, oracle_mod, seed):
    hg = inputs.uniform_hypergraph(seed)
    c = np.random.default_rng(seed).integers(1, 4, hg.num_vertices)
    L = balance_limit(c.sum())
    _say(f"bulk uniform {seed}")
    _compare_cutter(hf, oracle_mod, hg, c, L, L, 5000, f"bulk uniform {seed}",
                    bulk_percent=[55, 30, 80][seed])


def test_flowcutter_bulk_zipf_balanced(hf, oracle_mod):
    """The 200k-vertex instance with bulk piercing runs to a balanced cut;
    the returned side is a certificate: its cut weight is the flow value and
    both sides respect the bound."""
    hg = inputs.zipf_hypergraph(0, 200_000, 400_000, size_hi=200, vertex_weight_hi=3)
    c = hg.vertex_weights.astype(np.int64)
    L = balance_limit(c.sum())
    _say("zipf 200k with bulk piercing")
    with hf.FlowProblem.from_hypergraph(hg) as p:
        res, x, trace = p.flowcutter(c, L, L, max_iterations=100000, bulk_percent=55)
    x = x.astype(bool)
    _say(f"status {res['status']} after {res['iterations']} iterations, F {res['flow']}")
    assert res["status"] == "balanced"
    assert oracle_mod.cut_weight(hg, x) == res["flow"]
    assert int(c[x].sum()) <= L and int(c[~x].sum()) <= L
    assert max(res["counts"]) > 1


def test_flowcutter_tiny_vs_oracle(hf, oracle_mod):
    rng = np.random.default_rng(11)
    for seed in range(200):
        hg = inputs.tiny_hypergraph(seed)
        c = rng.integers(1, 4, hg.num_vertices)
        L = (int(c.sum()) + 1) // 2 + int(rng.integers(0, 3))
        _compare_cutter(hf, oracle_mod, hg, c, L, L, 100, f"tiny {seed}",
                        debug_checks=1 if seed % 5 == 0 else 0)


@pytest.mark.parametrize("seed", range(6))
def test_flowcutter_uniform_vs_oracle(hf, oracle_mod, seed):
    """2,000 vertices, 3,000 nets; vertex weights U{1..3}; eps = 0.03."""
    hg = inputs.uniform_hypergraph(seed)
    c = np.random.default_rng(seed).integers(1, 4, hg.num_vertices)
    L = balance_limit(c.sum())
    _say(f"uniform {seed}")
    res = _compare_cutter(hf, oracle_mod, hg, c, L, L, 5000, f"uniform {seed}",
                          group_lanes=[4, 8, 16][seed % 3])
    assert res["status"] == "balanced"


@pytest.mark.parametrize("seed", range(2))
def test_flowcutter_kept_labels_checked(hf, oracle_mod, seed):
    """A solve after an augmenting source pierce starts from the labels it
    has (paragraph "Maintain Distance Labels"); with the invariant checker
    after every round (preflow and label validity on every residual arc) the
    run still equals the oracle's, on 2,000-vertex instances whose runs
    pierce on both sides and augment."""
    hg = inputs.uniform_hypergraph(10 + seed)
    c = np.random.default_rng(seed).integers(1, 4, hg.num_vertices)
    L = balance_limit(c.sum())
    _say(f"kept labels, uniform {10 + seed}")
    res = _compare_cutter(hf, oracle_mod, hg, c, L, L, 5000, f"kept labels {seed}",
                          debug_checks=1)
    _say(f"{res['iterations']} iterations, {res['augmenting']} augmenting")
    assert res["augmenting"] > 0


def test_flowcutter_limit_returns_last_source_side(hf, oracle_mod):
    """A run stopped by its iteration limit returns the last iteration's
    S_r, also when that iteration pierced on the source side (the pierced
    vertex is not part of it): equal to the oracle's result at the same
    limit, for limits ending on source and on sink pierces."""
    hg = inputs.uniform_hypergraph(3)
    c = np.random.default_rng(3).integers(1, 4, hg.num_vertices)
    L = balance_limit(c.sum())
    full = oracle_mod.flowcutter(hg, c, L, L, max_iterations=5000)
    src = [i + 1 for i, t in enumerate(full.trace) if t[0] == 0][:2]
    snk = [i + 1 for i, t in enumerate(full.trace) if t[0] == 1][:1]
    assert src, "the run pierces on the source side"
    for k in src + snk:
        ref = oracle_mod.flowcutter(hg, c, L, L, max_iterations=k)
        assert ref.status == "cap"
        with hf.FlowProblem.from_hypergraph(hg) as p:
            res, x, trace = p.flowcutter(c, L, L, max_iterations=k)
        _say(f"limit {k}: last pierce on side {trace[-1][0]}")
        assert res["status"] == "cap" and res["flow"] == ref.flow
        assert [tuple(t) for t in trace] == [tuple(t) for t in ref.trace]
        assert (x.astype(bool) == ref.vertex_side.astype(bool)).all(), k
        assert oracle_mod.cut_weight(hg, x.astype(bool)) == res["flow"]


def test_flowcutter_block_pairs_vs_oracle(hf, oracle_mod):
    """Region problems of a partitioned hypergraph, balance = the k-way
    bound on both blocks (s and t carry the rest of their blocks)."""
    bp = inputs.block_pair_problems(0, num_vertices=20000, target_pins=100000, k=8,
                                    max_problems=6)
    for i, h in enumerate(bp.problems):
        _say(f"block pair {i}")
        res = _compare_cutter(hf, oracle_mod, h, h.vertex_weights, bp.lmax, bp.lmax, 3000,
                              f"pair {i}")
        assert res["flow"] >= 0


def test_flowcutter_zipf_prefix_vs_oracle(hf, oracle_mod):
    """The 200k-vertex incremental instance (Zipf sizes clamped to 200,
    vertex weights U{1..3}): the first 10 iterations match the oracle."""
    hg = inputs.zipf_hypergraph(0, 200_000, 400_000, size_hi=200, vertex_weight_hi=3)
    c = hg.vertex_weights
    L = balance_limit(c.sum())
    _say("zipf 200k prefix")
    ref = oracle_mod.flowcutter(hg, c, L, L, max_iterations=10)
    with hf.FlowProblem.from_hypergraph(hg) as p:
        res, x, trace = p.flowcutter(c, L, L, max_iterations=10)
    assert [tuple(t) for t in trace] == [tuple(t) for t in ref.trace]
    assert res["status"] == ref.status
    assert (x.astype(bool) == ref.vertex_side.astype(bool)).all()


def test_most_balanced_tiny_vs_oracle(hf, oracle_mod):
    """Most balanced cut on 200 tiny hypergraphs (loose bounds, so the
    balance phase has room): trace, first balanced iteration and result."""
    rng = np.random.default_rng(23)
    longer = 0
    for seed in range(200):
        hg = inputs.tiny_hypergraph(seed)
        c = rng.integers(1, 4, hg.num_vertices)
        L = (int(c.sum()) + 1) // 2 + int(rng.integers(0, 5))
        res = _compare_cutter(hf, oracle_mod, hg, c, L, L, 100, f"most balanced tiny {seed}",
                              most_balanced=True, debug_checks=1 if seed % 5 == 0 else 0)
        longer += res["iterations"] > res["first_balanced"] > 0
    assert longer >= 20


@pytest.mark.parametrize("seed", range(3))
def test_most_balanced_uniform_vs_oracle(hf, oracle_mod, seed):
    """2,000 vertices, 3,000 nets, vertex weights U{1..3}, eps = 0.03, with
    bulk piercing for the first seed (which then ends without a balanced
    cut: bulk pierces overshoot on this instance, in the oracle as well)."""
    hg = inputs.uniform_hypergraph(seed)
    c = np.random.default_rng(seed).integers(1, 4, hg.num_vertices)
    L = balance_limit(c.sum())
    _say(f"most balanced uniform {seed}")
    res = _compare_cutter(hf, oracle_mod, hg, c, L, L, 5000, f"most balanced uniform {seed}",
                          bulk_percent=55 if seed == 0 else 0, most_balanced=True,
                          group_lanes=[4, 8, 16][seed % 3])
    assert res["status"] == ("infeasible" if seed == 0 else "balanced")


def test_most_balanced_block_pairs_vs_oracle(hf, oracle_mod):
    bp = inputs.block_pair_problems(0, num_vertices=20000, target_pins=100000, k=8,
                                    max_problems=4)
    for i, h in enumerate(bp.problems):
        _say(f"most balanced block pair {i}")
        _compare_cutter(hf, oracle_mod, h, h.vertex_weights, bp.lmax, bp.lmax, 3000,
                        f"most balanced pair {i}", bulk_percent=55, most_balanced=True)


def test_most_balanced_zipf_improves_balance(hf, oracle_mod):
    """The 200k-vertex instance with bulk piercing: the most balanced cut
    keeps the first balanced cut's weight, is a certificate of it, respects
    the bound and has a heavier side no heavier than the first balanced
    cut's."""
    hg = inputs.zipf_hypergraph(0, 200_000, 400_000, size_hi=200, vertex_weight_hi=3)
    c = hg.vertex_weights.astype(np.int64)
    total = int(c.sum())
    L = balance_limit(total)
    _say("zipf 200k, first balanced cut")
    with hf.FlowProblem.from_hypergraph(hg) as p:
        r0, x0, _ = p.flowcutter(c, L, L, max_iterations=100000, bulk_percent=55)
    _say("zipf 200k, most balanced cut")
    with hf.FlowProblem.from_hypergraph(hg) as p:
        r1, x1, t1 = p.flowcutter(c, L, L, max_iterations=100000, bulk_percent=55,
                                  most_balanced=True)
    _say(f"first balanced at {r0['iterations']}: {r0['source_weight']}/{r0['sink_weight']}; "
         f"most balanced after {r1['iterations']}: {r1['source_weight']}/{r1['sink_weight']}")
    assert r0["status"] == r1["status"] == "balanced"
    assert r1["first_balanced"] == r0["iterations"]
    assert r1["flow"] == r0["flow"]
    x1 = x1.astype(bool)
    assert oracle_mod.cut_weight(hg, x1) == r1["flow"]
    cx = int(c[x1].sum())
    assert cx == r1["source_weight"] and total - cx == r1["sink_weight"]
    assert cx <= L and total - cx <= L
    assert max(cx, total - cx) <= max(r0["source_weight"], r0["sink_weight"])
    assert all(t[2] == r0["flow"] for t in t1[r0["iterations"] - 1:])


@pytest.mark.parametrize("seed", range(2))
def test_flowcutter_expanded_levels_vs_oracle(hf, oracle_mod, seed):
    """Every BFS level device-wide and expanded (provisional stamps plus the
    collect sweep on the source side, plain label stores on the relabel):
    the same traces, with bulk piercing and the most balanced cut."""
    hg = inputs.uniform_hypergraph(seed + 20)
    c = np.random.default_rng(seed).integers(1, 4, hg.num_vertices)
    L = balance_limit(c.sum())
    _say(f"expanded levels {seed}")
    _compare_cutter(hf, oracle_mod, hg, c, L, L, 5000, f"expanded levels {seed}",
                    bulk_percent=55 * seed, most_balanced=True, bottom_up_min=1,
                    tail_threshold=1)


@pytest.mark.parametrize("bulk,most_balanced", [(0, False), (55, False), (0, True), (55, True)])
def test_flowcutter_slices_equal_one_run(hf, oracle_mod, bulk, most_balanced):
    """A run cut into slices of 7 iterations (flow_problem_flowcutter_continue)
    gives the same trace, result and side as one uninterrupted run, and a
    finished run cannot be continued.  A most-balanced run that has no
    piercing vertex left is finished, not resumable (a run that reported
    itself resumable there kept this loop going without end)."""
    hg = inputs.uniform_hypergraph(5)
    c = np.random.default_rng(5).integers(1, 4, hg.num_vertices)
    L = balance_limit(c.sum())
    _say(f"slices bulk={bulk} most_balanced={most_balanced}")
    with hf.FlowProblem.from_hypergraph(hg) as p:
        r1, x1, t1 = p.flowcutter(c, L, L, max_iterations=5000, bulk_percent=bulk,
                                  most_balanced=most_balanced)
    assert r1["iterations"] < 5000 and not r1["resumable"]
    with hf.FlowProblem.from_hypergraph(hg) as p:
        r2, x2, t2 = p.flowcutter(c, L, L, max_iterations=7, bulk_percent=bulk,
                                  most_balanced=most_balanced)
        trace, slices = list(t2), 1
        while r2["resumable"]:
            assert r2["iterations"] == len(trace)
            assert slices <= r1["iterations"] // 7 + 1, "continued past the end of the run"
            r2, x2, t2 = p.flowcutter_continue(max_iterations=7)
            trace += t2
            slices += 1
        with pytest.raises(hf.HyperflowError) as ei:
            p.flowcutter_continue(max_iterations=7)
        assert ei.value.name == "FP_ERR_STATE"
    assert slices > 3
    assert trace == t1
    for k in ("flow", "source_weight", "sink_weight", "iterations", "status", "side",
              "augmenting", "first_balanced"):
        assert r1[k] == r2[k], k
    assert (x1 == x2).all()


def _checkpoint_vs_oracle(oracle_mod, hg, c, L, roles, step, tag):
    """The oracle solves the terminal sets of a checkpoint from scratch; its
    first FlowCutter iteration must be the GPU's next trace entry (flow
    value, c(S_r), c(T_r), side and smallest piercing vertex)."""
    hw = _with_terminals(hg, np.nonzero(roles == 1)[0], np.nonzero(roles == 2)[0])
    ref = oracle_mod.flowcutter(hw, c, L, L, max_iterations=1)
    assert tuple(ref.trace[0]) == tuple(step), f"{tag}: {ref.trace[0]} != {step}"
    return ref


@pytest.mark.parametrize("bulk", [55])
def test_flowcutter_zipf_checkpoints_vs_oracle(hf, oracle_mod, bulk):
    """The 200k-vertex incremental instance (Zipf sizes clamped to 200,
    vertex weights U{1..3}) run in slices to its balanced cut: at
    checkpoints spread over the run and at its last iteration, the oracle
    solves the GPU's current terminal sets from scratch and reproduces the
    next trace entry; at the end it reproduces the returned side."""
    hg = inputs.zipf_hypergraph(0, 200_000, 400_000, size_hi=200, vertex_weight_hi=3)
    c = hg.vertex_weights
    L = balance_limit(c.sum())
    _say(f"zipf 200k checkpoints bulk={bulk}")
    points = []
    with hf.FlowProblem.from_hypergraph(hg) as p:
        res, x, tr = p.flowcutter(c, L, L, max_iterations=1, bulk_percent=bulk)
        trace = list(tr)
        size = 1
        while res["resumable"]:
            roles = p.terminals()
            res, x, tr = p.flowcutter_continue(max_iterations=size)
            points.append((res["iterations"] - len(tr), roles, tr[0]))
            trace += tr
            size *= 4
        final_roles = p.terminals()
    _say(f"{len(trace)} iterations, {len(points)} checkpoints; {res['status']}")
    assert res["status"] == "balanced" and len(points) >= 3
    for it0, roles, step in points:
        _say(f"checkpoint after iteration {it0}")
        _checkpoint_vs_oracle(oracle_mod, hg, c, L, roles, step, f"after {it0}")
    _say("last iteration")
    ref = _checkpoint_vs_oracle(oracle_mod, hg, c, L, final_roles, trace[-1], "last")
    assert ref.status == "balanced"
    assert (x.astype(bool) == ref.vertex_side.astype(bool)).all()
    assert oracle_mod.cut_weight(hg, x.astype(bool)) == res["flow"]


@pytest.mark.parametrize("V,E,star,opts", [
    (31, 12, 0, {}), (32, 12, 0, {}), (33, 12, 0, {}), (63, 40, 0, {}), (65, 40, 9, {}),
    (1023, 300, 0, {}), (1025, 900, 40, dict(tail_threshold=8)), (1700, 300, 0, {}),
    (2500, 1200, 700, {}), (2500, 1200, 700, dict(tail_threshold=4096))], ids=str)
@pytest.mark.parametrize("most_balanced", [False, True])
def test_flowcutter_loop_edges_vs_oracle(hf, oracle_mod, V, E, star, opts, most_balanced):
    """Iterations run inside one workgroup: sparse networks, where most
    vertices are next to neither side and the pick falls back to the smallest
    vertex outside both; sizes around the words of the bitmaps; more iterations
    than one loop books; one net with many pins, whose growth is too large for
    the loop, or fits it and leaves more vertices to pierce than it takes."""
    rng = np.random.default_rng(V + E + star)
    nets = [sorted(rng.choice(V, size=int(rng.integers(2, 4)), replace=False).tolist())
            for _ in range(E)]
    if star:
        nets[E // 2] = sorted(rng.choice(V, size=star, replace=False).tolist())
    who = rng.permutation(V)[:6]
    hg = inputs.hypergraph_from_nets(V, nets, rng.integers(1, 4, E), who[:3], who[3:])
    c = rng.integers(1, 4, V)
    L = balance_limit(c.sum())
    _say(f"loop edges V={V} star={star} {opts} most_balanced={most_balanced}")
    _compare_cutter(hf, oracle_mod, hg, c, L, L, 4000, f"loop edges {V} {star}",
                    most_balanced=most_balanced, **opts)
