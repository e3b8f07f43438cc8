"""The kernels of the simulator (the order by iteration, the walk in LDS, the walk in global memory) at the places where
one hands over to the next or changes its layout: costs bit for bit equal to the CPU oracle's (both add fp64 times in
the order the rules fix)."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_2209_12769_amd import workloads as wl

pytestmark = pytest.mark.gpu

F = 16


@pytest.fixture(scope="module")
def B():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2209_12769_amd import binding
    binding.lib()
    return binding


def graph(n, edges):
    src, dst = (np.array(x, np.int64) for x in zip(*edges)) if edges else (np.zeros(0, np.int64),) * 2
    rp, ci = wl._csr_from_edges(n, src, dst)
    return wl.BaseGraph(n, n, rp, ci, np.zeros((n, F), np.float32))


def chain(n, extra=()):
    return graph(n, [(i, i + 1) for i in range(n - 1)] + list(extra))


def fan(n):
    """One op releases n - 2 others, which all precede the last."""
    return graph(n, [(0, i) for i in range(1, n - 1)] + [(i, n - 1) for i in range(1, n - 1)])


def tensors(n_op, n_ar):
    """A chain of ops whose last one produces n_ar tensors; the first tensor of the list has no predecessor."""
    return graph(n_op + n_ar, [(i, i + 1) for i in range(n_op - 1)] + [(n_op - 1, n_op + k) for k in range(1, n_ar)])


def sources(n):
    return graph(n + 1, [(i, n) for i in range(n)])


# name: (graph, mask of all-reduce nodes as a function of the node number, change of the op times)
CASES = {
    **{f"chain{n}": (chain(n), None, None) for n in (1, 2, 63, 64, 65, 128, 129, 200)},
    **{f"fan{n}": (fan(n), None, None) for n in (10, 65, 66, 67, 129, 130, 400)},
    **{f"sources{n}": (sources(n), None, None) for n in (15, 16, 17, 64, 65, 127, 128, 200)},
    **{f"tensors{k}": (tensors(70, k), lambda v: v >= 70, None) for k in (1, 63, 64, 65, 66, 129, 300)},
    "all_tensors": (graph(70, []), lambda v: v >= 0, None),
    "no_edges": (graph(300, []), lambda v: v % 7 == 0, None),
    "tensor_with_successor": (chain(90), lambda v: v % 10 == 5, None),
    "negative_time": (chain(90, [(3, 50)]), None, lambda t: np.where(np.arange(t.size) == 40, np.float32(-1), t)),
    "infinite_time": (chain(90), lambda v: v == 89, lambda t: np.where(np.arange(t.size) == 40, np.float32(np.inf), t)),
    "times_far_apart": (chain(500, [(3, 400)]), lambda v: v % 50 == 49 and v > 450, lambda t: t * np.where(np.arange(t.size) % 3 == 0, 1e6, 1e-6)),
    "times_at_the_limit": (chain(255), None, lambda t: np.where(np.arange(t.size) == 9, 2.0 ** -20, 1.0 + t)),
    "times_past_the_limit": (chain(255), None, lambda t: np.where(np.arange(t.size) == 9, 2.0 ** -24 * (1 + t), 1.0 + t)),
    "zero_times": (fan(100), lambda v: v == 99, lambda t: np.zeros_like(t)),
    "walked_in_memory": (chain(32000), None, None),
    "walked_in_memory_past_32768": (chain(33500), None, None),
    "wide_and_long": (wl.random_dag(31, 3000, 0.002, F), lambda v: v % 9 == 8, None),
}


def test_every_layout_gives_the_oracle_s_costs(B):
    import torch
    graphs = [c[0] for c in CASES.values()]
    labels = [np.arange(g.n, dtype=np.int32).reshape(1, -1) for g in graphs]
    w = wl.custom("walk", wl.ModelSpec(F, 32, 1, "f32"), graphs, labels, seed=1)
    ref = orc.contract(w, False)
    rng = wl.Rng(9, 1)
    op_time, ar_size = [], []
    for g, ar, change in CASES.values():
        t = (rng.uniform(g.n) + 0.01).astype(np.float32)
        is_ar = np.zeros(g.n, bool) if ar is None else np.asarray([ar(v) for v in range(g.n)], bool)
        op_time.append(t if change is None else change(t).astype(np.float32))
        ar_size.append(np.where(is_ar, 8 * rng.uniform(g.n), -1.0).astype(np.float32))
    op_time, ar_size = np.concatenate(op_time), np.concatenate(ar_size)
    ev = B.evaluator_for(w)
    nb, eb = sum(g.n for g in graphs), sum(g.e for g in graphs)
    batch = ev.contract_graphs(ev.to_device(w.cand_graph), ev.to_device(w.cand_off), ev.to_device(w.group_id),
                               ev.alloc_batch(w.n_cand, nb, nb, eb))
    t, x = torch.from_numpy(op_time).to(ev.device), torch.from_numpy(ar_size).to(ev.device)
    for c, d in ((0.25, 0.05), (0.0, 0.0), (3.0, 1.0)):
        want = orc.simulate(ref, op_time, ar_size, c, d)
        got = ev.simulate(batch, t, x, c, d).cpu().numpy()
        assert ev.check() == B.DC_OK
        for name, a, b in zip(CASES, got, want):
            assert a == b, (name, c, d, a, b)
    ev.close()


def _batch(B, graphs, copies):
    """`copies` times all the graphs as one contracted batch, unfused."""
    import torch
    w = wl.custom("walk", wl.ModelSpec(F, 32, 1, "f32"), graphs, [np.arange(g.n, dtype=np.int32).reshape(1, -1) for g in graphs], seed=1)
    nb, eb = copies * sum(g.n for g in graphs), copies * sum(g.e for g in graphs)
    ev = B.Evaluator(F, 32, 1, "f32", copies * len(graphs), nb, max(eb, 1))
    ev.set_base_graphs(w.g_node_off(), w.g_edge_off(), w.cat_rowptr(), w.cat_col(), w.cat_X())
    off = np.concatenate([[0], np.cumsum(np.tile([g.n for g in graphs], copies))])
    batch = ev.contract_graphs(ev.to_device(np.tile(w.cand_graph, copies)), ev.to_device(off),
                               torch.from_numpy(w.group_id).to(ev.device).repeat(copies),
                               ev.alloc_batch(copies * len(graphs), nb, nb, max(eb, 1)))
    return ev, batch, orc.contract(w, False)


def _times(ev, graphs, copies, is_ar, seed=3):
    """Host arrays of one copy, device arrays of all; is_ar: mask of all-reduce nodes by (graph, node number)."""
    import torch
    rng = wl.Rng(seed, 2)
    t = np.concatenate([rng.uniform(g.n) + 0.01 for g in graphs]).astype(np.float32)
    x = np.concatenate([np.where([is_ar(i, v) for v in range(g.n)], 8 * rng.uniform(g.n), -1.0)
                        for i, g in enumerate(graphs)]).astype(np.float32)
    return t, x, torch.from_numpy(np.tile(t, copies)).to(ev.device), torch.from_numpy(np.tile(x, copies)).to(ev.device)


def test_walked_modules_of_every_size_class_share_a_cu(B):
    """Ops wait for all-reduces, so every module is walked; about a dozen modules of six classes and of global memory
    fall to each workgroup."""
    graphs = [chain(n, [(1, n - 2), (n // 2, n - 1)]) for n in (5, 600, 680, 700, 1150, 1750, 2350, 3500, 3700, 5000)]
    copies = 310
    ev, batch, ref = _batch(B, graphs, copies)
    t, x, td, xd = _times(ev, graphs, copies, lambda i, v: v % 50 == 2)
    want = orc.simulate(ref, t, x, 0.25, 0.05)
    before = ev.walked_modules()
    got = ev.simulate(batch, td, xd, 0.25, 0.05).cpu().numpy()
    assert ev.check() == B.DC_OK
    assert np.array_equal(got.reshape(copies, -1), np.tile(want, (copies, 1)))
    assert ev.walked_modules() - before == copies * len(graphs)
    ev.close()


def test_small_walked_modules_fill_a_cu(B):
    """Ten working sets of 16 KB fit a CU's LDS: four times the modules of a batch that gives every CU two take little
    longer (0.27 and 0.32 ms); two to a CU whatever their size took four times as long."""
    g = chain(600)
    took = []
    for copies in (512, 2048):
        ev, batch, _ = _batch(B, [g], copies)
        _, _, td, xd = _times(ev, [g], copies, lambda i, v: v % 50 == 2)
        took.append(_milliseconds(ev, batch, td, xd))
        assert ev.walked_modules() == 6 * copies
        ev.close()
    print(took, flush=True)
    assert took[1] < 2.5 * took[0]


def layers(k, w, step=1):
    """k layers of w ops, each released by one op of the layer before: the same one for all, or w / step in turn."""
    return graph(k * w, [((a - 1) * w + (i * 7 % w) // step * step, a * w + i) for a in range(1, k) for i in range(w)])


def crossed(n):
    """Two ops whose n released ops each are numbered the other way round, then alternate."""
    e = [(0, 2 + n + i) for i in range(n)] + [(1, 2 + i) for i in range(n)]
    e += [(2 + n + 3, 2 + 2 * n + i) for i in range(0, n, 2)] + [(2 + 3, 2 + 2 * n + i) for i in range(1, n, 2)]
    return graph(2 + 3 * n, e)


TIED = {
    **{f"fan{n}": (fan(n), None) for n in (129, 130, 131, 250, 257, 700, 2100, 9000)},
    **{f"tensors{k}": (tensors(70, k), lambda v: v >= 70) for k in (128, 129, 130, 180, 700, 3000, 9000)},
    **{f"layers{k}x{w}/{s}": (layers(k, w, s), None) for k, w, s in ((12, 300, 1), (6, 1000, 500), (40, 129, 1), (3, 80, 1), (5, 260, 131))},
    **{f"crossed{n}": (crossed(n), None) for n in (60, 129, 200, 1500, 4000)},
    **{f"all_tensors{n}": (graph(n, []), lambda v: v >= 0) for n in (128, 129, 130, 1500, 5000)},
    "sources_and_tensors": (graph(4000, [(0, v) for v in range(2000, 3000)]), lambda v: v >= 1900),
}


def test_thousands_of_nodes_released_together(B):
    graphs = [g for g, _ in TIED.values()]
    ev, batch, ref = _batch(B, graphs, 1)
    t, x, td, xd = _times(ev, graphs, 1, lambda i, v: (list(TIED.values())[i][1] or (lambda v: False))(v))
    want = orc.simulate(ref, t, x, 0.25, 0.05)
    got = ev.simulate(batch, td, xd, 0.25, 0.05).cpu().numpy()
    assert ev.check() == B.DC_OK
    for name, a, b in zip(TIED, got, want):
        assert a == b, (name, a, b)
    assert ev.walked_modules() == 0
    ev.close()


def _milliseconds(ev, batch, td, xd):
    import torch
    cost = ev.simulate(batch, td, xd, 0.25, 0.05)
    best = np.inf
    for _ in range(5):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        ev.simulate(batch, td, xd, 0.25, 0.05, cost)
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b))
    return best


def test_tensors_of_one_op_take_the_time_of_tensors_of_many(B):
    """The work for nodes that become ready together is not the square of their number (6000: 5.1 ms so, 1.3 now; the
    same tensors spread over 70 ops 0.8)."""
    n = 6000
    spread = graph(70 + n, [(i, i + 1) for i in range(69)] + [(k % 70, 70 + k) for k in range(n)])
    took = []
    for g in (tensors(70, n), spread):
        ev, batch, _ = _batch(B, [g], 512)
        _, _, td, xd = _times(ev, [g], 512, lambda i, v: v >= 70)
        took.append(_milliseconds(ev, batch, td, xd))
        assert ev.walked_modules() == 0
        ev.close()
    print(took, flush=True)
    assert took[0] < 3 * took[1]


def chains(k, n):
    """k chains of n ops, numbered one after the other."""
    return graph(k * n, [(c * n + i, c * n + i + 1) for c in range(k) for i in range(n - 1)])


def renumbered(g, how):
    p = np.arange(g.n)[::-1] if how == "reversed" else np.random.default_rng(g.n).permutation(g.n)
    src = np.repeat(np.arange(g.n), np.diff(g.rowptr))
    return graph(g.n, list(zip(p[src].tolist(), p[g.col].tolist())))


def twice(g):
    src = np.repeat(np.arange(g.n), np.diff(g.rowptr))
    return graph(2 * g.n, list(zip(src.tolist(), g.col.tolist())) + list(zip((src + g.n).tolist(), (g.col + g.n).tolist())))


def blocks(n, lengths, shift=0):
    """n times: branches of these lengths between two ops, each branch numbered on its own."""
    e, at, new = [], 0, 1
    for _ in range(n):
        ends = []
        for m in lengths:
            p = at
            for _ in range(m):
                e.append((p, new))
                p, new = new, new + 1
            ends.append(p)
        e += [(p, new) for p in ends]
        at, new = new, new + 1
    return graph(new, e)


SMALL = wl.make("cfg2", 1).graphs[0]          # 729 nodes
SLOW = {
    **{f"chains{k}x{n}": chains(k, n) for k, n in ((2, 30), (2, 120), (2, 254), (2, 300), (8, 100), (3, 1000), (2, 4000), (2, 8000), (300, 40))},
    "reversed200": renumbered(chain(200), "reversed"),
    "reversed5000": renumbered(chain(5000, [(3, 4000)]), "reversed"),
    "permuted": renumbered(SMALL, "at random"),
    "twice": twice(SMALL),
    "blocks": twice(blocks(60, (3, 7, 5, 9))),
    "long_lists": renumbered(twice(wl.random_dag(5, 500, 0.02, F)), "reversed"),
}


def test_orders_far_from_the_numbering(B):
    """Parallel chains numbered one after the other, and numberings that follow no order: as many rounds from the index
    order as a chain is long, a handful from the depths."""
    graphs = list(SLOW.values())
    ev, batch, ref = _batch(B, graphs, 1)
    t, x, td, xd = _times(ev, graphs, 1, lambda i, v: graphs[i].rowptr[v] == graphs[i].rowptr[v + 1] and v % 3 == 0)
    want = orc.simulate(ref, t, x, 0.25, 0.05)
    got = ev.simulate(batch, td, xd, 0.25, 0.05).cpu().numpy()
    assert ev.check() == B.DC_OK
    for name, a, b in zip(SLOW, got, want):
        assert a == b, (name, a, b)
    assert ev.walked_modules() == 0
    ev.close()


def test_cycles_where_the_second_guess_is_needed(B):
    for n in (60, 600, 3000):
        g = chains(2, n)
        labs = np.stack([np.arange(2 * n)] * 3).astype(np.int32)
        labs[1, n - 5] = labs[1, n - 9]                      # late in the first chain
        labs[2, 2 * n - 1] = labs[2, 3]                      # no cycle: the ends of both
        w = wl.custom("cycles", wl.ModelSpec(F, 32, 1, "f32"), [g], [labs], seed=1)
        ref = orc.contract(w, False)
        t = (wl.Rng(n, 3).uniform(ref.ntot) + 0.01).astype(np.float32)
        x = np.full(ref.ntot, -1.0, np.float32)
        want = orc.simulate(ref, t, x, 0.25, 0.05)
        assert np.isinf(want[1]) and np.isfinite(want[[0, 2]]).all()
        ev = B.evaluator_for(w)
        batch = ev.contract_graphs(ev.to_device(w.cand_graph), ev.to_device(w.cand_off), ev.to_device(w.group_id),
                                   ev.alloc_batch(3, 6 * n, 6 * n, 6 * n))
        import torch
        got = ev.simulate(batch, torch.from_numpy(t).to(ev.device), torch.from_numpy(x).to(ev.device), 0.25, 0.05).cpu().numpy()
        assert ev.check() == B.DC_OK and ev.walked_modules() == 0
        assert np.array_equal(got, want), (n, got, want)
        ev.close()


def test_which_modules_are_walked(B):
    """Sizes at the ends of the classes, predecessor lists that overflow LDS, and an order that depths do not settle:
    every layer of three ops turns the order of the one before, so that a round settles one layer."""
    graphs = {
        **{f"chain{n}": chain(n) for n in (256, 257, 2048, 2049, 8192, 8193, 16384, 16385)},
        **{f"dense{n}": wl.random_dag(77, n, p, F) for n, p in ((256, 0.2), (2048, 0.02), (8192, 0.003), (16384, 0.0015))},
        "turning": graph(1500, [(3 * a - 1 - i, 3 * a + i) for a in range(1, 500) for i in range(3)]),
        "permuted_branches": renumbered(twice(SMALL), "at random"),
    }
    ev, batch, ref = _batch(B, list(graphs.values()), 1)
    t, x, td, xd = _times(ev, list(graphs.values()), 1, lambda i, v: False)
    want = orc.simulate(ref, t, x, 0.25, 0.05)
    got = ev.simulate(batch, td, xd, 0.25, 0.05).cpu().numpy()
    assert ev.check() == B.DC_OK
    for name, a, b in zip(graphs, got, want):
        assert a == b, (name, a, b)
    for g in list(graphs.values())[8:12]:                     # what lists longer than four keep in LDS does not fit it
        d = np.bincount(g.col, minlength=g.n)
        assert (d[d > 4] - 2).sum() > (256 if g.n <= 256 else 2048 if g.n <= 2048 else 8192 if g.n <= 8192 else 16384)
    assert ev.walked_modules() == 3                           # chain16385 and the last two
    ev.close()


def test_parallel_chains_do_not_take_a_round_per_op(B):
    """Two chains of 300 ops, 4096 modules: 4.4 ms with 256 rounds and then the walk, 0.33 now; one chain of 600 0.10."""
    took = []
    for g in (chains(2, 300), chain(600)):
        ev, batch, _ = _batch(B, [g], 4096)
        _, _, td, xd = _times(ev, [g], 4096, lambda i, v: False)
        took.append(_milliseconds(ev, batch, td, xd))
        ev.close()
    print(took, flush=True)
    assert took[0] < 6 * took[1]
