"""GPU parity of the attention variant of the estimator (Sec. 3.3.1 with attention
coefficients, graph-attention reading) against the CPU oracle, through the C ABI."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_2209_12769_amd import workloads as wl

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-5, "bf16": 2e-2}     # against the plain oracle (fp32 storage, fp64 accumulation)
MIRROR_TOL = 6e-3                      # bf16 path against the oracle with the same bf16 storage points


def check(got, w, tag):
    want = orc.evaluate(w)
    err = rel_err(got, want)
    print(f"[attention] {tag} max rel err vs plain oracle {err.max():.3e}", flush=True)
    assert err.max() <= TOL[w.model.dtype]
    if w.model.dtype == "bf16":
        err = rel_err(got, orc.evaluate(w, bf16=True))
        print(f"[attention] {tag} max rel err vs oracle with bf16 storage points {err.max():.3e}", flush=True)
        assert err.max() <= MIRROR_TOL


@pytest.fixture(scope="module")
def B():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2209_12769_amd import binding
    binding.lib()
    return binding


def rel_err(got, ref):
    got = np.asarray(got, np.float64)
    ref = np.asarray(ref, np.float64)
    floor = 1e-3 * float(np.median(np.abs(ref))) if ref.size else 0.0
    return np.abs(got - ref) / np.maximum(np.maximum(np.abs(ref), floor), 1e-30)


def run(B, w):
    ev = B.evaluator_for(w)
    cg, co, gid = ev.to_device(w.cand_graph), ev.to_device(w.cand_off), ev.to_device(w.group_id)
    pred = ev.eval_candidates(cg, co, gid).cpu().numpy()
    assert ev.check() == B.DC_OK, B.dc_last_error(ev.ctx)
    again = ev.eval_candidates(cg, co, gid).cpu().numpy()
    assert np.array_equal(pred, again)
    ev.close()
    return pred


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("F,H,L,K", [(16, 32, 2, 4), (32, 64, 1, 2), (16, 128, 2, 8), (64, 256, 2, 4), (16, 512, 1, 1),
                                     (48, 64, 3, 8)])
def test_small_batches_every_width(B, dtype, F, H, L, K):
    g = wl.random_dag(7, 300, 0.02, F)
    labs = wl.random_labels(8, g.n, 90, C=7)
    w = wl.custom(f"att-{dtype}-{F}-{H}-{L}-{K}", wl.ModelSpec(F, H, L, dtype, "attention", K), [g], [labs], seed=3)
    if dtype == "bf16":
        # random signed weights let the last dot product cancel to a hundredth of its terms, where bf16
        # storage alone (the oracle with bf16 storage points against the plain one) is 3e-2 off; the
        # 2e-2 bound is about predictions that are sums of like-signed terms, as times are
        w = wl.with_time_like_head(w)
    check(run(B, w), w, w.name)


def test_long_neighbour_lists_and_two_cycles(B):
    # few groups on a dense graph: lists far longer than a lane group, neighbours that are both
    # predecessor and successor
    g = wl.random_dag(11, 500, 0.05, 16)
    labs = np.concatenate([wl.random_labels(12, g.n, 6, C=2), wl.random_labels(13, g.n, 60, C=2)])
    w = wl.custom("att-dense", wl.ModelSpec(16, 64, 2, "f32", "attention", 4), [g], [labs], seed=5)
    got = run(B, w)
    want = orc.evaluate(w)
    assert rel_err(got, want).max() <= TOL["f32"]


def test_zero_attention_vectors_equal_uniform_coefficients(B):
    g = wl.random_dag(17, 200, 0.03, 16)
    labs = wl.random_labels(18, g.n, 70, C=3)
    w = wl.custom("att-zero", wl.ModelSpec(16, 64, 2, "f32", "attention", 4), [g], [labs], seed=6)
    w.weights.att[:] = 0.0
    got = run(B, w)
    want = orc.evaluate(w)
    assert rel_err(got, want).max() <= TOL["f32"]


@pytest.mark.parametrize("name,n,heads", [("cfg1", 3, 4), ("cfg2", 64, 4), ("cfg3", 48, 8), ("cfg4", 12, 4)])
def test_configurations_with_attention(B, name, n, heads):
    w = wl.with_attention(wl.make(name, n), heads)
    check(run(B, w), w, f"{w.name} C={w.n_cand}")


def test_config_errors(B):
    for H, K in [(48, 4), (64, 3), (64, 16), (1024, 4)]:
        cfg = B.DcConfig(16, H, 1, B.DC_F32, 4, 100, 100, 0, 0, B.DC_AGG_ATTENTION, K)
        st, h = B.dc_create(cfg)
        assert st in (B.DC_ERR_UNSUPPORTED, B.DC_ERR_INVALID_ARG) and not h
    # the two weight calls are tied to the kind of context
    ev = B.Evaluator(16, 32, 1, "f32", 4, 100, 100)
    z = np.zeros(3 * 16 * 32 + 4 * 32 * 32 + 1000, np.float32)
    assert B.dc_set_attention_weights(ev.ctx, z, z, z, z) == B.DC_ERR_INVALID_ARG
    ev.close()
    ev = B.Evaluator(16, 32, 1, "f32", 4, 100, 100, agg="attention", heads=2)
    assert B.dc_set_weights(ev.ctx, z, z, z) == B.DC_ERR_INVALID_ARG
    ev.close()


def hub(n, F):
    """A chain, an op that precedes all others and one that follows all: lists of n - 1."""
    edges = {(i, i + 1) for i in range(n - 1)} | {(0, i) for i in range(1, n)} | {(i, n - 1) for i in range(n - 1)}
    src, dst = (np.array(x) for x in zip(*sorted(edges)))
    rowptr = np.concatenate([[0], np.cumsum(np.bincount(src, minlength=n))]).astype(np.int32)
    return wl.BaseGraph(n, n, rowptr, dst.astype(np.int32), np.random.default_rng(n).random((n, F), dtype=np.float32))


# (H, heads, dtype, waves per SIMD of the kernel, rows per wave and round): four rounds to a claim, two where a round has 16 rows
@pytest.mark.parametrize("H,K,dtype,waves,rows", [(256, 4, "bf16", 7, 2), (256, 4, "f32", 5, 2), (128, 1, "bf16", 7, 4),
                                                  (512, 2, "bf16", 7, 1), (64, 2, "f32", 5, 8), (32, 1, "bf16", 7, 16),
                                                  (32, 1, "f32", 5, 16)])
def test_rows_claimed_in_order(B, H, K, dtype, waves, rows):
    """A batch in which every XCD's eighth has sixteen rounds of rows for every wave, from where on the waves claim rows
    through a counter: every candidate gets the prediction of a batch of three, whose rows are dealt, bit for bit."""
    import torch
    F = 16
    graphs = [hub(150, F), wl.random_dag(901, 700, 0.004, F), wl.random_dag(902, 333, 0.01, F)]
    model = wl.ModelSpec(F, H, 2, dtype, "attention", K)
    w = wl.with_time_like_head(wl.custom("claims", model, graphs, [np.arange(g.n, dtype=np.int32)[None] for g in graphs], seed=6))
    want = run(B, w)
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    n_waves = (n_cu + 7) // 8 * waves * 4                     # on an XCD
    per, edges = sum(g.n for g in graphs), sum(g.e for g in graphs)
    copies = 8 * 16 * n_waves * rows // per + 2
    assert copies * per // 8 >= 16 * n_waves * rows > 2 * per
    ev = B.Evaluator(F, H, 2, dtype, 3 * copies, copies * per, copies * edges, agg="attention", heads=K)
    ev.set_base_graphs(w.g_node_off(), w.g_edge_off(), w.cat_rowptr(), w.cat_col(), w.cat_X())
    ev.set_weights(w.weights)
    off = np.concatenate([[0], np.cumsum(np.tile([g.n for g in graphs], copies))])
    args = (ev.to_device(np.tile(w.cand_graph, copies)), ev.to_device(off), ev.to_device(w.group_id).repeat(copies))
    print(H, K, dtype, copies, flush=True)
    for _ in range(2):
        got = ev.eval_candidates(*args).cpu().numpy().reshape(copies, 3)
        assert ev.check() == B.DC_OK
        assert np.array_equal(got, np.tile(want, (copies, 1)))
    ev.close()


# the score terms as columns of the product (up to four heads) and in a kernel of their own (eight, thirty-two); one row,
# the edges of its tiles of 128 rows, several tiles per workgroup
@pytest.mark.parametrize("F,K", [(64, 1), (64, 2), (256, 4), (64, 4), (64, 8), (64, 32)])
@pytest.mark.parametrize("n,C", [(1, 1), (43, 3), (127, 1), (129, 1), (640, 64)])
def test_score_columns(B, F, K, n, C):
    g = wl.random_dag(40 + n, n, min(1.0, 3.0 / n), F)
    w = wl.custom(f"att-columns-{F}-{K}", wl.ModelSpec(F, 256, 2, "bf16", "attention", K), [g],
                  [np.tile(np.arange(n, dtype=np.int32), (C, 1))], seed=K)
    w = wl.with_time_like_head(w)
    got = run(B, w)
    assert np.all(got == got[0])
    check(got[:1], w.subset([0]), w.name)
