"""The layer kernel in which every wave works on 32 rows of its own, at the sizes where it can go wrong."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_2209_12769_amd import workloads as wl

pytestmark = pytest.mark.gpu
TOL = 2e-2          # bf16 against the plain oracle, as for every bf16 path


@pytest.fixture(scope="module")
def B():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2209_12769_amd import binding
    binding.lib()
    return binding


def _graph(n, kind, F):
    if kind == "sparse":
        return wl.random_dag(700 + n, n, min(1.0, 3.0 / max(n, 2)), F)
    if kind == "dense":      # a tile's lists exceed the 128 neighbour numbers that a wave keeps
        return wl.random_dag(800 + n, n, 0.2, F)
    # a chain, one source that feeds every node and one sink fed by every node
    edges = {(i, i + 1) for i in range(n - 1)} | {(0, i) for i in range(1, n)} | {(i, n - 1) for i in range(n - 1)}
    src, dst = (np.array(x) for x in zip(*sorted(edges)))
    rowptr = np.concatenate([[0], np.cumsum(np.bincount(src, minlength=n))]).astype(np.int32)
    X = np.random.default_rng(n).random((n, F), dtype=np.float32)
    return wl.BaseGraph(n, n, rowptr, dst.astype(np.int32), X)


@pytest.mark.parametrize("F,H,L", [(16, 32, 2), (32, 128, 3), (64, 64, 2), (128, 128, 2), (128, 32, 2), (128, 64, 1), (16, 128, 1),
                                   (64, 128, 2), (32, 64, 3)])
def test_equals_the_separate_kernels_bit_for_bit(B, F, H, L):
    model = wl.ModelSpec(F, H, L, "bf16")
    for n, kind, C in ((1, "sparse", 1), (31, "sparse", 1), (32, "sparse", 1), (33, "sparse", 1), (65, "sparse", 5),
                       (90, "dense", 3), (300, "hub", 2), (700, "sparse", 40)):
        g = _graph(n, kind, F)
        labs = np.tile(np.arange(g.n, dtype=np.int32), (C, 1))
        w = wl.with_time_like_head(wl.custom(f"wave-{kind}-{n}x{C}", model, [g], [labs], seed=9))
        ev = B.evaluator_for(w)
        cg, co, gid = ev.to_device(w.cand_graph), ev.to_device(w.cand_off), ev.to_device(w.group_id)
        print(F, H, L, n, kind, C, flush=True)
        fused = ev.eval_candidates(cg, co, gid).cpu().numpy()
        assert ev.check() == B.DC_OK
        ev.select_kernels(B.DC_KERNELS_SEPARATE_LAYERS)
        plain = ev.eval_candidates(cg, co, gid).cpu().numpy()
        assert ev.check() == B.DC_OK
        ev.close()
        assert np.array_equal(fused, plain), (n, kind, C, np.abs(fused - plain).max())
        want = orc.evaluate_parallel(w, False, 8, np.arange(1))
        assert abs(fused[0] - want[0]) <= TOL * abs(want[0]), (n, kind, fused[0], want[0])


@pytest.mark.parametrize("F,H,L", [(16, 32, 2), (32, 128, 2), (64, 64, 2), (128, 128, 1)])
def test_row_pointers_that_do_not_begin_at_zero(B, F, H, L):
    """A caller's batch may keep its edges anywhere in the edge arrays.  The first tiles have no neighbours at all: what
    they request in their place must be a row of the batch, whatever number the row pointers begin with."""
    import torch
    sparse = _graph(90, "sparse", F)
    X = np.random.default_rng(5).random((100, F), dtype=np.float32)
    lone = wl.BaseGraph(100, 100, np.zeros(101, np.int32), np.zeros(0, np.int32), X)
    graphs = [lone, sparse, lone]
    w = wl.with_time_like_head(wl.custom("moved", wl.ModelSpec(F, H, L, "bf16"), graphs,
                                         [np.arange(g.n, dtype=np.int32)[None] for g in graphs], seed=4))
    ev = B.evaluator_for(w)
    nb, eb = sum(g.n for g in graphs), sum(g.e for g in graphs)
    b = ev.contract_graphs(ev.to_device(w.cand_graph), ev.to_device(w.cand_off), ev.to_device(w.group_id),
                           ev.alloc_batch(w.n_cand, nb, nb, eb))
    want = ev.gnn_forward(b).cpu().numpy()
    assert ev.check() == B.DC_OK
    for pad in (1, nb + 7, 1 << 20):
        rps = [x + pad for x in (b.out_rowptr, b.in_rowptr)]
        cols = [torch.cat([torch.zeros(pad, dtype=torch.int32, device=ev.device), x]) for x in (b.out_col, b.in_col)]
        c = B.DcBatch(w.n_cand, nb, eb + pad, b.node_off.data_ptr(), b.edge_off.data_ptr(), b.new_id.data_ptr(),
                      rps[0].data_ptr(), cols[0].data_ptr(), rps[1].data_ptr(), cols[1].data_ptr(), b.Xc.data_ptr())
        moved = B.DeviceBatch(c, b.node_off, b.edge_off, b.new_id, rps[0], cols[0], rps[1], cols[1], b.Xc)
        got = ev.gnn_forward(moved).cpu().numpy()
        assert ev.check() == B.DC_OK
        assert np.array_equal(got, want), pad
    ev.close()


@pytest.mark.parametrize("F,H,L", [(16, 32, 2), (32, 128, 3), (64, 64, 2), (128, 128, 2), (128, 64, 1), (16, 128, 1), (64, 128, 1),
                                   (32, 64, 2), (64, 32, 1), (16, 64, 1)])
def test_waves_with_several_tiles(B, F, H, L):
    """At least two tiles of 32 rows for each of the grid's waves (sixteen of them on a CU, eight for the wider shapes),
    so that a tile's requests are made in the one before, across graphs with long lists, few and none."""
    import torch
    X = np.random.default_rng(6).random((41, F), dtype=np.float32)
    graphs = [_graph(150, "hub", F), _graph(700, "sparse", F), _graph(90, "dense", F), wl.BaseGraph(41, 41, np.zeros(42, np.int32), np.zeros(0, np.int32), X)]
    w = wl.with_time_like_head(wl.custom("tiles", wl.ModelSpec(F, H, L, "bf16"), graphs,
                                         [np.arange(g.n, dtype=np.int32)[None] for g in graphs], seed=8))
    per, edges = sum(g.n for g in graphs), sum(g.e for g in graphs)
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    copies = 2 * 16 * n_cu * 32 // per + 3
    ev = B.Evaluator(F, H, L, "bf16", 4 * copies, copies * per, copies * edges)
    ev.set_base_graphs(w.g_node_off(), w.g_edge_off(), w.cat_rowptr(), w.cat_col(), w.cat_X())
    ev.set_weights(w.weights)
    off = np.concatenate([[0], np.cumsum(np.tile([g.n for g in graphs], copies))])
    args = (ev.to_device(np.tile(w.cand_graph, copies)), ev.to_device(off), ev.to_device(w.group_id).repeat(copies))
    print(F, H, L, copies, flush=True)
    fused = ev.eval_candidates(*args).cpu().numpy()
    assert ev.check() == B.DC_OK
    ev.select_kernels(B.DC_KERNELS_SEPARATE_LAYERS)
    plain = ev.eval_candidates(*args).cpu().numpy()
    assert ev.check() == B.DC_OK
    ev.close()
    assert np.array_equal(fused, plain)
    want = orc.evaluate(w)
    assert np.all(np.abs(fused[:4] - want) <= TOL * np.abs(want))
