"""Batched search (vc_mvc_batch / vc_pvc_batch and their device forms) against the CPU
oracle, one graph at a time.

The bar is the single-graph bar, per graph: MVC size and PVC decision identical to the
oracle's; every cover checked edge by edge here; node counts identical where the tree does not
depend on the schedule (one workgroup that never donates; PVC graphs whose answer is no, in any
launch configuration). A graph's answer must not depend on the graphs it is batched with.
"""

import time

import numpy as np
import pytest

import graphs as G
import oracle

pytestmark = pytest.mark.gpu

KERNELS = {"auto": 0, "bitsets": 0x40, "degree_arrays": 0x20}


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return torch


@pytest.fixture(scope="module")
def solver(torch_cuda):
    import paper_2204_10402_amd as vc
    s = vc.Solver(0)
    yield s
    s.close()


def check_cover(g, cover, size):
    cover = np.asarray(cover)
    assert cover.shape == (g.n,)
    assert set(np.unique(cover).tolist()) <= {0, 1}
    assert oracle.is_cover(g, cover)
    assert int(cover.sum()) == size


def mixed_graphs(seed, count=24, n_hi=300):
    """Small random graphs of 1..4 bitset words and degree arrays (the batch tests also run
    them all on the degree-array kernels by flag)."""
    rng = np.random.default_rng(seed)
    out = []
    for i in range(count):
        n = int(rng.integers(5, n_hi + 1))
        p = float(rng.uniform(1.5, 5.0)) / n
        out.append(G.erdos_renyi(n, p, 1000 * seed + i))
    return out


@pytest.mark.parametrize("kernel", ["auto", "degree_arrays"])
@pytest.mark.parametrize("seed", range(4))
def test_mvc_batch_matches_oracle(solver, oracle_lib, seed, kernel):
    import paper_2204_10402_amd as vc
    gs = mixed_graphs(seed)
    res = solver.mvc_batch(gs, vc.Options(flags=KERNELS[kernel]))
    for i, g in enumerate(gs):
        o = oracle.mvc(g)
        assert res.status[i] == 0
        assert res.size[i] == o.size, i
        check_cover(g, res.cover_of(i), o.size)
    assert res.stats["nodes"] == int(res.nodes.sum())


@pytest.mark.parametrize("kernel", ["bitsets", "degree_arrays"])
def test_mvc_batch_single_workgroup_node_parity(solver, oracle_lib, kernel):
    """One workgroup that never donates walks the graphs one after another, each in the
    oracle's order: per-graph node counts equal the oracle's."""
    import paper_2204_10402_amd as vc
    gs = [G.erdos_renyi(20 + 9 * i, 0.12, 500 + i) for i in range(10)]
    res = solver.mvc_batch(gs, vc.Options(num_wg=1, wl_threshold=-1, flags=KERNELS[kernel]))
    for i, g in enumerate(gs):
        o = oracle.mvc(g)
        assert (res.size[i], res.nodes[i]) == (o.size, o.nodes), i
        check_cover(g, res.cover_of(i), o.size)


@pytest.mark.parametrize("kernel", ["auto", "degree_arrays"])
@pytest.mark.parametrize("seed", range(3))
def test_pvc_batch_decisions_and_no_node_counts(solver, oracle_lib, seed, kernel):
    import paper_2204_10402_amd as vc
    gs = mixed_graphs(100 + seed, count=20, n_hi=200)
    taus = [oracle.mvc(g).size for g in gs]
    ks = [max(t - (i % 3), 0) for i, t in enumerate(taus)]  # tau, tau-1, tau-2 in turn
    res = solver.pvc_batch(gs, ks, vc.Options(flags=KERNELS[kernel]))
    for i, g in enumerate(gs):
        want = ks[i] >= taus[i]
        assert res.status[i] == 0
        assert bool(res.yes[i]) == want, i
        if want:
            assert 0 <= res.size[i] <= ks[i]
            check_cover(g, res.cover_of(i), int(res.size[i]))
        else:
            # a no-instance's tree is searched whole, whatever the schedule
            assert res.size[i] == -1 and int(res.cover_of(i).sum()) == 0
            assert res.nodes[i] == oracle.pvc(g, ks[i]).nodes, i


def test_planted_batch_full_size(solver, oracle_lib):
    """4,096 planted-cover PVC instances (n uniform in [40, 400], average degree in [3, 12],
    |C| = 0.3n, k = |C| for even i and |C| - 1 for odd i) in one call: every decision equals
    the oracle's; no-instances visit exactly the oracle's nodes."""
    import paper_2204_10402_amd as vc
    batch = G.planted_batch(4096, 0)
    gs = [g for g, _ in batch]
    ks = [k for _, k in batch]
    res = solver.pvc_batch(gs, ks)
    assert (res.status == 0).all()
    # the instances above 256 vertices on the degree-array kernels too
    wide = [i for i, g in enumerate(gs) if g.n > 256]
    arr = solver.pvc_batch([gs[i] for i in wide], [ks[i] for i in wide],
                           vc.Options(flags=vc.OPT_DEGREE_ARRAYS))
    assert (arr.status == 0).all()
    assert [bool(x) for x in arr.yes] == [bool(res.yes[i]) for i in wide]
    for i, (g, k) in enumerate(batch):
        o = oracle.pvc(g, k)
        assert bool(res.yes[i]) == o.yes, i
        if o.yes:
            assert res.size[i] <= k
            check_cover(g, res.cover_of(i), int(res.size[i]))
        else:
            assert res.nodes[i] == o.nodes, i
    assert res.yes[0::2].all()  # k = |C| always has the planted cover


def test_batch_answers_do_not_depend_on_the_mix(solver, oracle_lib):
    import paper_2204_10402_amd as vc
    gs = mixed_graphs(7, count=12)
    alone = [solver.mvc(g) for g in gs]
    mixed = solver.mvc_batch(gs)
    rev = solver.mvc_batch(gs[::-1])
    for i, g in enumerate(gs):
        assert mixed.size[i] == alone[i].size == rev.size[len(gs) - 1 - i]
    ks = [max(r.size - 1, 0) for r in alone]
    pv = solver.pvc_batch(gs, ks, vc.Options(num_wg=17))
    for i, g in enumerate(gs):
        assert bool(pv.yes[i]) == (alone[i].size == 0)
        if not pv.yes[i]:
            assert pv.nodes[i] == solver.pvc(g, ks[i]).stats["nodes"]


def test_batch_with_rejected_empty_and_edgeless_graphs(solver, oracle_lib):
    import paper_2204_10402_amd as vc

    class Raw:
        pass
    bad = Raw()
    good = G.path(5)
    bad.n, bad.row_ptr = 5, good.row_ptr.copy()
    bad.col_idx = good.col_idx.copy()
    bad.col_idx[0] = 9  # out of range
    empty = G.empty(0)
    edgeless = G.empty(7)
    gs = [G.cycle(9), bad, empty, edgeless, G.complete(6), bad, G.erdos_renyi(150, 0.03, 3)]
    res = solver.mvc_batch(gs)
    want_status = [0, vc.ERR_INVALID_GRAPH, 0, 0, 0, vc.ERR_INVALID_GRAPH, 0]
    assert res.status.tolist() == want_status
    assert res.size[0] == 5 and res.size[2] == 0 and res.size[3] == 0 and res.size[4] == 5
    assert res.size[6] == oracle.mvc(gs[6]).size
    assert res.size[1] == -1 and int(res.cover_of(1).sum()) == 0
    for i in (0, 3, 4, 6):
        check_cover(gs[i], res.cover_of(i), int(res.size[i]))
    p = solver.pvc_batch(gs, [5, 3, 0, 0, 4, 3, 0])
    assert p.status.tolist() == want_status
    assert p.yes.tolist() == [True, False, True, True, False, False, False]


def test_batch_budget_is_per_graph(solver, oracle_lib):
    import paper_2204_10402_amd as vc
    hard = G.random_regular(120, 5, 0)
    easy = [G.cycle(11), G.erdos_renyi(80, 0.05, 1), G.path(30)]
    res = solver.mvc_batch([easy[0], hard, easy[1], easy[2]], vc.Options(node_budget=20000))
    assert res.status.tolist() == [0, vc.ERR_BUDGET, 0, 0]
    assert res.size[0] == 6 and res.size[3] == 15
    assert res.size[2] == oracle.mvc(easy[1]).size
    assert int(res.cover_of(1).sum()) == 0


def test_batch_device_form(solver, oracle_lib, torch_cuda):
    import paper_2204_10402_amd as vc
    torch = torch_cuda
    gs = mixed_graphs(9, count=16)
    n, nnz, rp, ci = vc.pack_batch(gs)
    rp_d = torch.from_numpy(rp).cuda()
    ci_d = torch.from_numpy(ci).cuda()
    cov = torch.zeros(int(n.sum()), dtype=torch.uint8, device="cuda")
    res = solver.mvc_batch_device(n, nnz, rp_d, ci_d, cov)
    host = solver.mvc_batch(gs)
    assert res.size.tolist() == host.size.tolist()
    c = cov.cpu().numpy()
    for i, g in enumerate(gs):
        check_cover(g, c[res.offsets[i]:res.offsets[i + 1]], int(res.size[i]))
    ks = np.maximum(res.size - 1, 0).tolist()
    pres = solver.pvc_batch_device(n, nnz, rp_d, ci_d, ks, cov)
    assert pres.yes.tolist() == (res.size == 0).tolist()
    assert int(cov.sum().item()) == 0


def test_empty_batch_and_bad_arguments(solver):
    import paper_2204_10402_amd as vc
    res = solver.mvc_batch([])
    assert res.status.size == 0
    with pytest.raises(vc.VCError) as ei:
        solver.pvc_batch([G.path(4)], [-1])
    assert ei.value.code == vc.ERR_INVALID_ARG
    with pytest.raises(vc.VCError) as ei:
        solver.mvc_batch([G.path(600)], vc.Options(flags=vc.OPT_BITSETS))
    assert ei.value.code == vc.ERR_INVALID_ARG


def test_autotuned_batches_keep_answers(torch_cuda, oracle_lib):
    """With VC_OPT_AUTOTUNE the first call times trial launches and later calls reuse the
    choice; answers and PVC-no node counts stay the oracle's either way."""
    import paper_2204_10402_amd as vc
    s = vc.Solver(0)  # a fresh context: nothing tuned yet
    try:
        gs = mixed_graphs(11, count=20)
        o = vc.Options(flags=vc.OPT_AUTOTUNE)
        first = s.mvc_batch(gs, o)
        second = s.mvc_batch(gs, o)
        for i, g in enumerate(gs):
            want = oracle.mvc(g).size
            assert first.size[i] == second.size[i] == want, i
            check_cover(g, second.cover_of(i), want)
        ks = [max(int(x) - 1, 0) for x in first.size]
        p = s.pvc_batch(gs, ks, o)
        for i, g in enumerate(gs):
            if not p.yes[i]:
                assert p.nodes[i] == oracle.pvc(g, ks[i]).nodes
        # explicit knobs switch the tuner off
        fixed = s.mvc_batch(gs, vc.Options(flags=vc.OPT_AUTOTUNE, num_wg=5))
        assert fixed.stats["num_wg"] <= 5 and fixed.size.tolist() == first.size.tolist()
    finally:
        s.close()


@pytest.mark.parametrize("count,team", [(40, 8), (700, 4), (1500, 2), (2500, 1)])
def test_bitset_team_sizes(solver, oracle_lib, count, team):
    """The wavefronts per workgroup follow the number of instances (a workgroup holds one instance
    at a time); the tree of a PVC-no answer is the oracle's node for node with every team size, so
    no sub-tree is lost or walked twice in a handover. Whole numbers: no tolerance."""
    base = [G.erdos_renyi(20 + 9 * i, 3.2 / (20 + 9 * i) + 0.02, 70 + i) for i in range(12)]
    taus = [oracle.mvc(g).size for g in base]
    want = [oracle.pvc(g, max(t - 1, 0)).nodes for g, t in zip(base, taus)]
    gs = [base[i % 12] for i in range(count)]
    res = solver.pvc_batch(gs, [max(taus[i % 12] - 1, 0) for i in range(count)])
    assert (res.status == 0).all() and not res.yes.any()
    assert res.nodes.tolist() == [want[i % 12] for i in range(count)]
    one = [g for g in gs if g.n <= 64]  # one kernel family
    r1 = solver.pvc_batch(one, [max(taus[base.index(g)] - 1, 0) for g in one])
    assert r1.nodes.tolist() == [want[base.index(g)] for g in one]
    mv = solver.mvc_batch(gs)
    assert mv.size.tolist() == [taus[i % 12] for i in range(count)]
    alone = solver.mvc_batch([base[4]] * count)
    assert alone.stats["wg_size"] == 64 * team and set(alone.size.tolist()) == {taus[4]}


@pytest.mark.parametrize("n", [257, 320, 321, 448, 511, 512, 513])
def test_pvc_family_by_size_and_options(solver, oracle_lib, n):
    """PVC takes the bitset kernels up to 512 vertices, unless an option asks for what only the
    degree-array kernels know; both families give the same decision, a valid cover and, for no,
    the oracle's node count. MVC keeps the degree arrays above 256. Whole numbers: no tolerance."""
    import paper_2204_10402_amd as vc
    torch = pytest.importorskip("torch")
    g = G.erdos_renyi(n, 3.0 / n, 4200 + n)
    tau = oracle.mvc(g, node_cap=200000).size
    want = oracle.pvc(g, tau - 1, node_cap=200000).nodes
    assert solver.mvc(g).stats["bitset_words"] == 0
    rp, ci = torch.from_numpy(g.row_ptr).to("cuda:0"), torch.from_numpy(g.col_idx).to("cuda:0")
    words = (n + 63) // 64 if n <= 512 else 0
    for kw, w in ((dict(), words), (dict(wg_size=64), 0), (dict(wg_size=128), 0),
                  (dict(flags=vc.OPT_CSR_GLOBAL), 0), (dict(flags=vc.OPT_DEGREE_ARRAYS), 0),
                  (dict(flags=vc.OPT_STACK_ONLY, start_depth=4), 0),
                  (dict(wl_threshold=-1, num_wg=1), words), (dict(num_wg=3, wl_capacity=1), words),
                  (dict(flags=vc.OPT_AUTOTUNE), words), (dict(timeout_ms=20000), words)):
        o = vc.Options(**kw)
        no = solver.pvc(g, tau - 1, o)
        assert not no.yes and no.stats["bitset_words"] == w and no.stats["nodes"] == want, kw
        yes = solver.pvc(g, tau, o)
        assert yes.yes and yes.size <= tau and oracle.is_cover(g, yes.cover), kw
        assert int(yes.cover.sum()) == yes.size
        if "flags" not in kw and "wg_size" not in kw:
            need = solver.workspace_bytes(g.n, g.col_idx.size, options=o)
            ws = torch.empty(need, dtype=torch.uint8, device="cuda:0")
            r = solver.pvc_device_ws(rp, ci, tau - 1, ws, options=o)
            assert not r.yes and r.stats["nodes"] == want, kw
            m = solver.mvc_device_ws(rp, ci, ws, options=o)
            assert m.size == tau and m.stats["bitset_words"] == 0, kw
    assert not solver.pvc_device_noalloc(rp, ci, tau - 1).yes
    with pytest.raises(vc.VCError) as e:
        solver.pvc(g, tau - 1, vc.Options(node_budget=1))
    assert e.value.code == vc.ERR_BUDGET or want <= 1


@pytest.mark.parametrize("count", [1, 2, 63, 64, 65, 130])
def test_results_of_batches_around_the_direct_limit(solver, oracle_lib, count):
    """Up to 64 graphs the cover check writes the results to host memory, above that a copy
    command brings them: sizes, decisions, node counts and covers are the oracle's either way, on
    a second call with other graphs too."""
    for seed in (0, 1):
        gs = [G.erdos_renyi(24 + (7 * i + 13 * seed) % 50, 0.09, 800 + 31 * seed + i)
              for i in range(count)]
        want = [oracle.mvc(g) for g in gs]
        mv = solver.mvc_batch(gs)
        assert mv.size.tolist() == [w.size for w in want]
        for i, g in enumerate(gs):
            c = np.asarray(mv.cover_of(i))
            assert oracle.is_cover(g, c) and int(c.sum()) == want[i].size, i
        ks = [max(w.size - 1, 0) for w in want]
        no = solver.pvc_batch(gs, ks)
        o = [oracle.pvc(g, k) for g, k in zip(gs, ks)]
        assert no.yes.tolist() == [x.yes for x in o]
        assert [int(no.nodes[i]) for i in range(count) if not o[i].yes] == \
            [x.nodes for x in o if not x.yes]


@pytest.mark.parametrize("way", ["option", "workspace"])
def test_failed_batch_leaves_nothing_running(oracle_lib, torch_cuda, way):
    """A batch that fails after some of its launches are queued (the graph above 256 vertices runs
    first, then the bitset group refuses a workgroup size; or a workspace that only holds the first
    kernel family) has stopped them when it returns: at once, although one of the searches would
    take far longer, and the next batch, staged in the same host memory, gets its own answers."""
    import paper_2204_10402_amd as vc
    hard = G.erdos_renyi(300, 0.06, 1)
    small = [G.erdos_renyi(60, 0.1, i) for i in range(3)]
    other = [G.erdos_renyi(30 + 7 * i, 0.12, 70 + i) for i in range(7)]
    with vc.Solver(0) as s:
        for _ in range(3):
            t = time.perf_counter()
            with pytest.raises(vc.VCError) as e:
                if way == "option":
                    s.mvc_batch(small + [hard], vc.Options(wg_size=128, timeout_ms=30000))
                else:
                    large = G.planted_cover(20000, 800, 60000, 0.75, 1)
                    n, nnz, rp, ci = vc.pack_batch(small + [large])
                    s.mvc_batch_device_ws(
                        n, nnz, torch_cuda.from_numpy(rp).to("cuda:0"),
                        torch_cuda.from_numpy(ci).to("cuda:0"),
                        torch_cuda.empty(4 << 20, dtype=torch_cuda.uint8, device="cuda:0"))
            assert e.value.code == (vc.ERR_INVALID_ARG if way == "option" else vc.ERR_NO_MEMORY)
            assert time.perf_counter() - t < 5.0
            res = s.mvc_batch(other)
            for i, g in enumerate(other):
                want = oracle.mvc(g)
                assert (res.status[i], res.size[i]) == (0, want.size), i
                check_cover(g, res.cover_of(i), want.size)
            res = s.pvc_batch(other, [oracle.mvc(g).size - 1 for g in other])
            for i, g in enumerate(other):
                o = oracle.pvc(g, oracle.mvc(g).size - 1)
                assert (res.status[i], bool(res.yes[i]), res.nodes[i]) == (0, False, o.nodes), i


@pytest.mark.parametrize("sizes", [(257, 320, 321, 384), (257, 384, 385, 448, 300), (300, 449, 512, 257, 385)])
def test_wide_bitset_graphs_share_a_launch(solver, oracle_lib, torch_cuda, sizes):
    """The graphs of 257 to 512 vertices of a PVC batch run in one bitset launch, as wide as the
    widest of them needs (a launch for each word count would run their searches in turn), beside
    the launches of the smaller ones. Node counts of no-answers are the oracle's, in a workspace
    of the stated size as well. Whole numbers: no tolerance."""
    import paper_2204_10402_amd as vc
    gs = [G.erdos_renyi(n, 2.6 / n, 60 + i) for i, n in enumerate(sizes)]
    for extra, launches in ([], 1), ([G.erdos_renyi(50, 0.08, 1), G.erdos_renyi(200, 0.015, 2)], 3):
        batch = gs + extra
        taus = [oracle.mvc(g, node_cap=200000).size for g in batch]
        no = solver.pvc_batch(batch, [t - 1 for t in taus])
        assert no.stats["launches"] == launches
        assert no.stats["bitset_words"] == (max(sizes) + 63) // 64
        want = [oracle.pvc(g, t - 1, node_cap=200000).nodes for g, t in zip(batch, taus)]
        assert not no.yes.any() and no.nodes.tolist() == want
        yes = solver.pvc_batch(batch, taus)
        for i, g in enumerate(batch):
            assert yes.yes[i] and yes.size[i] <= taus[i], i
            check_cover(g, yes.cover_of(i), int(yes.size[i]))
        n, nnz, rp, ci = vc.pack_batch(batch)
        ws = torch_cuda.empty(solver.batch_workspace_bytes(n, nnz), dtype=torch_cuda.uint8, device="cuda:0")
        r = solver.pvc_batch_device_ws(n, nnz, torch_cuda.from_numpy(rp).to("cuda:0"),
                                       torch_cuda.from_numpy(ci).to("cuda:0"), [t - 1 for t in taus], ws)
        assert r.stats["launches"] == launches and r.nodes.tolist() == want
        mv = solver.mvc_batch(gs, vc.Options(flags=vc.OPT_BITSETS))
        assert mv.stats["launches"] == 1 and mv.size.tolist() == taus[:len(gs)]


@pytest.mark.parametrize("budget", [0, 10 ** 5, 10 ** 12])
def test_node_counts_reported_on_the_way(solver, oracle_lib, budget):
    """A graph's node count is the oracle's whether its wavefronts report it when they leave the
    graph (no budget) or every few nodes (a budget that the tree does not use up)."""
    import paper_2204_10402_amd as vc
    g = G.erdos_renyi(90, 0.07, 5)
    k = oracle.mvc(g).size - 1
    want = oracle.pvc(g, k).nodes
    assert 200 < want < 10 ** 5
    for flags in (vc.OPT_BITSETS, vc.OPT_DEGREE_ARRAYS):
        r = solver.pvc(g, k, vc.Options(node_budget=budget, flags=flags))
        assert not r.yes and r.stats["nodes"] == want


@pytest.mark.parametrize("n", [50, 100, 160, 230])
def test_one_workgroup_visits_the_same_nodes_on_every_run(solver, oracle_lib, n):
    """num_wg = 1 with the bitset kernels is one wavefront: the node counts of MVC and of a PVC yes
    are the same on every run, and those of 64-thread workgroups."""
    import paper_2204_10402_amd as vc
    g = G.erdos_renyi(n, 4.6 / n, 11 + n)
    tau = oracle.mvc(g).size
    runs = []
    for o in [vc.Options(num_wg=1)] * 3 + [vc.Options(num_wg=1, wg_size=64)]:
        m, y, w = solver.mvc(g, o), solver.pvc(g, tau, o), solver.pvc(g, tau - 1, o)
        assert (m.size, y.yes, w.yes) == (tau, True, False)
        assert m.stats["wg_size"] == y.stats["wg_size"] == 64 and m.stats["num_wg"] == 1
        runs.append((m.stats["nodes"], y.stats["nodes"], w.stats["nodes"]))
    assert len(set(runs)) == 1 and runs[0][2] == oracle.pvc(g, tau - 1).nodes
