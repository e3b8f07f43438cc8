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
