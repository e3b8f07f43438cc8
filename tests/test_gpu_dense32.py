"""fp32 layers whose products run on the bf16 matrix cores in three pieces, against 64-bit sums: widths and numbers of
rows at the edges of their tiles, and values that the pieces cannot hold."""
import numpy as np
import pytest

from paper_2209_12769_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2209_12769_amd import binding
    binding.lib()
    return binding


def _sum_head(H):
    """A regression network that adds up the graph vector: no cancellation after the layer."""
    eye = np.eye(H, dtype=np.float32).reshape(-1)
    z = np.zeros(H, np.float32)
    return np.concatenate([eye, z, eye, z, np.ones(H, np.float32), np.zeros(1, np.float32)])


def _means(g, X):
    src = np.repeat(np.arange(g.n), np.diff(g.rowptr))
    out = []
    for own, nb in ((g.col, src), (src, g.col)):
        s = np.zeros_like(X)
        np.add.at(s, own, X[nb])
        out.append(s / np.maximum(np.bincount(own, minlength=g.n), 1)[:, None])
    return out


# columns: 32 (one block of 32 per wave), 64 (two), 128 and 256 (four), 160 (one); K = 3 F, whole and broken sections of 64
@pytest.mark.parametrize("F,H", [(48, 32), (64, 64), (80, 128), (96, 160), (64, 256), (112, 128)])
@pytest.mark.parametrize("n,C,values", [(n, C, v) for n, C in ((1, 1), (33, 1), (130, 3)) for v in ("plain", "wide", "largest", "inf", "nan")] +
                         [(33, 1100, "plain"), (33, 1100, "largest")])
def test_layer_against_64_bits(B, F, H, n, C, values):
    rng = np.random.default_rng(F * H + n)
    g = wl.random_dag(70 + n, n, 0.05, F)
    X = rng.standard_normal((n, F)).astype(np.float32)
    W = (rng.standard_normal((3 * F, H)) / np.sqrt(3 * F)).astype(np.float32)
    if values == "wide":
        X *= np.exp2(rng.integers(-40, 20, X.shape)).astype(np.float32)
    # the largest column: its first piece rounds to infinity although every product is finite
    if values == "largest":
        X[:, 5], X[0, 5] = 0.0, 3.4e38
        W[5::F] *= np.float32(1e-36)
    if values in ("inf", "nan"):
        X[0, 3] = {"inf": np.inf, "nan": np.nan}[values]
    model = wl.ModelSpec(F, H, 1, "f32")
    bias = rng.standard_normal(H).astype(np.float32)
    w = wl.custom("layer", model, [wl.BaseGraph(n, n, g.rowptr, g.col, X)], [np.tile(np.arange(n, dtype=np.int32), (C, 1))],
                  weights=wl.Weights(W.reshape(-1), bias, _sum_head(H)))
    ev = B.evaluator_for(w)
    print(F, H, n, C, values, flush=True)
    pred = ev.eval_candidates(ev.to_device(w.cand_graph), ev.to_device(w.cand_off), ev.to_device(w.group_id)).cpu().numpy()
    assert ev.check() == B.DC_OK
    ev.close()
    with np.errstate(invalid="ignore"):
        A = np.concatenate([X.astype(np.float64), *_means(g, X.astype(np.float64))], 1)
        h = np.fmax(A @ W.astype(np.float64) + bias, 0.0)
        ref = h.sum()
    assert np.all(pred == pred[0])
    if not np.isfinite(ref):
        # an infinite graph vector times the zeros of the head's matrices is not a number, and ReLU makes that 0
        assert not np.isfinite(pred[0]) or pred[0] == 0.0
        return
    # means and sums of products: at most 24 roundings per section of 64, one per section, two of the means and three of
    # the head, each of 2^-24 of the terms' size
    size = (np.abs(np.nan_to_num(A)) @ np.abs(W.astype(np.float64)) + np.abs(bias)).sum()
    roundings = 24 + (3 * F + 63) // 64 + 5
    assert abs(float(pred[0]) - ref) <= roundings * 2.0 ** -24 * size
