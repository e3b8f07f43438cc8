"""fp32 products on the bf16 matrix cores in three pieces, against 64-bit sums: whole graphs with widths and numbers of rows at
the edges of the tiles and values that the pieces cannot hold; single outputs of a layer through each form of the
product; the gradients."""
import numpy as np
import pytest

from oracle import oracle as orc
from oracle import train as ot
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


# ---- every output against 64 bits -------------------------------------------------------------------------------------
# A graph of three nodes in a row, of which only the middle one has a final embedding: the others carry a flag whose
# weights hold them below zero.  The head picks one column, so an estimate is one output of the layer's product.
# Error over the root mean square of the results, the products emulated in numpy: 1.0e-7 to 1.2e-7 (K = 32 to 816), with one of
# the six partial products of the pieces left out 2.4e-6 at least.  Twelve roundings of 2^-24 lie between.
BOUND = 12 * 2.0 ** -24


def _column_head(H, j):
    W1, W2, w3 = np.zeros((H, H), np.float32), np.zeros((H, H), np.float32), np.zeros(H, np.float32)
    W1[j, 0] = W2[0, 0] = w3[0] = 1.0
    z = np.zeros(H, np.float32)
    return np.concatenate([W1.reshape(-1), z, W2.reshape(-1), z, w3, np.zeros(1, np.float32)])


def _kernel_of(n_cu, C, F, H):
    """Which of the three forms of the product serves C graphs of three nodes."""
    tiles = (3 * C + 31) // 32 * (H // 32)
    if tiles <= (n_cu + 3) // 4 * 8 and (3 * F + 63) // 64 <= 12:
        return "four waves a tile"
    return "one wave a tile" if tiles <= 4 * n_cu else "tiles of 128 rows"


# K = 3 F below 128: the fp32 instructions, which have three forms for the same numbers of rows too
@pytest.mark.parametrize("F,H", [(16, 32), (32, 128), (32, 160), (48, 32), (272, 32), (64, 64), (112, 128), (96, 160), (64, 256), (512, 256)])
def test_every_output_of_a_layer(B, F, H):
    import torch
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    rng = np.random.default_rng(F + H)
    graphs, n_good = [], 61
    for i in range(n_good + 3):
        X = rng.standard_normal((3, F)).astype(np.float32)
        X[:, 0] = 1.0, 0.0, 1.0                              # the flag
        X[:, 5] = 0.0
        if i >= n_good:                                      # values that the pieces cannot hold
            X[1, 5] = (3.4e38, np.inf, np.nan)[i - n_good]
        graphs.append(wl.BaseGraph(3, 3, np.array([0, 1, 2, 2], np.int32), np.array([1, 2], np.int32), X))
    W = (rng.standard_normal((3 * F, H)) / np.sqrt(3 * F)).astype(np.float32)
    W[0], W[F], W[2 * F] = -1e6, 0.0, 0.0
    W[5::F] *= np.float32(1e-36)
    bias = rng.standard_normal(H).astype(np.float32)
    X = np.stack([g.X for g in graphs]).astype(np.float64)
    with np.errstate(invalid="ignore"):
        A = np.concatenate([X[:, 1], X[:, 0], X[:, 2]], 1)
        ref = np.maximum(A @ W.astype(np.float64) + bias, 0.0)
    sizes = [1, n_good]
    for tiles in (2.8 * n_cu, 4.6 * n_cu):
        sizes.append(int(tiles * 32 / (H // 32) / 3))
    if 3 * F < 128:
        forms = [2 if (3 * C + 15) // 16 * (H // 16) <= 8 * n_cu else 1 if (3 * C + 31) // 32 * (H // 32) <= 4 * n_cu else 0 for C in sizes]
        assert forms == [2, 2, 1, 0]
    elif F <= 256:
        assert [_kernel_of(n_cu, C, F, H) for C in sizes] == ["four waves a tile"] * 2 + ["one wave a tile", "tiles of 128 rows"]
    else:
        assert _kernel_of(n_cu, 1, F, H) == "one wave a tile"
    ev = B.Evaluator(F, H, 1, "f32", max(sizes), 3 * max(sizes), 2 * max(sizes))
    w = wl.custom("rows", wl.ModelSpec(F, H, 1, "f32"), graphs, [np.zeros((1, 3), np.int32)] * len(graphs))
    ev.set_base_graphs(w.g_node_off(), w.g_edge_off(), w.cat_rowptr(), w.cat_col(), w.cat_X())
    errors = []
    for j in sorted({0, 31, H // 2, H - 2, H - 1}):
        ev.set_weights(wl.Weights(W.reshape(-1), bias, _column_head(H, j)))
        alone = None
        for C in sizes[::-1]:
            for mixed in (False, True):
                cg = np.arange(C, dtype=np.int32) % n_good
                bad = np.zeros(C, bool)
                if mixed:                                    # the others share tiles with every one of these
                    bad[2::5] = True
                    cg[bad] = n_good + np.arange(bad.sum()) % 3
                print(F, H, j, C, mixed, flush=True)
                pred = ev.eval_candidates(ev.to_device(cg), ev.to_device(np.arange(0, 3 * C + 1, 3, dtype=np.int32)),
                                          ev.to_device(np.tile(np.arange(3, dtype=np.int32), C))).cpu().numpy()
                assert ev.check() == B.DC_OK
                if alone is None:
                    alone = pred[:n_good].copy()
                    errors.append(alone - ref[:n_good, j])
                # the same bits through each kernel, whatever else the batch holds
                assert np.array_equal(pred[~bad], alone[cg[~bad]])
                large = cg == n_good
                if large.any():                              # one after the other in fp32: a rounding of 2^-24 per term
                    terms = np.abs(A[n_good]) @ np.abs(W[:, j].astype(np.float64)) + abs(bias[j])
                    assert np.abs(pred[large] - ref[n_good, j]).max() <= (3 * F + 2) * 2.0 ** -24 * terms
    ev.close()
    errors, scale = np.concatenate(errors), np.sqrt(np.mean(ref[:n_good] ** 2))
    print(f"F {F} H {H}: error {np.sqrt(np.mean(errors ** 2)) / scale:.2e} largest {np.abs(errors).max() / scale:.2e}")
    assert np.sqrt(np.mean(errors ** 2)) <= BOUND * scale


# ---- the reverse pass ----------------------------------------------------------------------------------------------------
# Every unit passes (biases of 1, products a tenth of that), so that no sum near zero decides a derivative and the gradient is
# a chain of products: the first layer's weight gradient is X^T of what W1^T, W2^T and the layers' transposed matrices made
# of the estimates' derivatives.  X is signed: with operands of one sign the error of a lost piece would average out.  Emulated
# with fp32 instructions throughout: the first layer's matrix 1.5e-7 to 4.8e-7, tensors whose sums have one sign 2.5e-8 to 7.7e-8.
# With a partial product left out in the transposed products or in the weight gradients (emulated) the first is 1.9e-6 off or more.
# Five and one and a half roundings of 2^-24 hold only where the small partial products are added before the large one, what the
# matrix cores drop cancels, and slabs of few rows and the biases' sums are not rounded on the way (without: 3.0e-7 and 1.15e-7).
BOUND_REVERSE, BOUND_ONE_SIGN = 5 * 2.0 ** -24, 1.5 * 2.0 ** -24
def _all_pass(F, H, n, C, seed):
    rng = np.random.default_rng(seed)
    g = wl.random_dag(seed, n, min(1.0, 3.0 / n), F)
    X = [rng.standard_normal((n, F)).astype(np.float32) for _ in range(C)]
    graphs = [wl.BaseGraph(n, n, g.rowptr, g.col, x) for x in X]
    draw = lambda k, m, s: (s * rng.standard_normal((k, m)) / np.sqrt(k)).astype(np.float32)
    layers = [draw(3 * F, H, 0.1), draw(3 * H, H, 0.1)]
    W1, W2 = draw(H, H, 0.1), draw(H, H, 0.1)
    w3 = (1.0 + rng.random(H)).astype(np.float32) / H
    one = np.ones(H, np.float32)
    head = lambda: np.concatenate([W1.reshape(-1), n * one, W2.reshape(-1), n * one, w3, np.zeros(1, np.float32)])
    target = (n * np.exp(rng.uniform(1.5, 3.0, C))).astype(np.float32)     # above every estimate: no sum over samples cancels
    return graphs, layers, np.tile(one, (2, 1)), head, target


def _gradients(B, F, H, graphs, layers, biases, head, target):
    import torch
    C, n = len(graphs), graphs[0].n
    weights = wl.Weights(np.concatenate([W.reshape(-1) for W in layers]), biases.reshape(-1), head)
    model = wl.ModelSpec(F, H, 2, "f32")
    w = wl.custom("all-pass", model, graphs, [np.arange(n, dtype=np.int32)[None]] * C, weights=weights)
    ev = B.evaluator_for(w)
    nb, eb = C * n, C * graphs[0].e
    batch = ev.contract_graphs(ev.to_device(w.cand_graph), ev.to_device(w.cand_off), ev.to_device(w.group_id),
                               ev.alloc_batch(C, nb, nb, eb))
    ev.train_begin(1e-3, C, nb)
    _, _, grad = ev.loss_gradients(batch, torch.from_numpy(target).to(ev.device))
    assert ev.check() == B.DC_OK
    grad = grad.cpu().numpy().astype(np.float64)
    ev.close()
    _, _, ref = ot.loss_and_gradients(orc.contract(w), target, ot.Params.from_weights(weights, F, H, 2))
    return ot.Params.from_flat(grad, F, H, 2), ref


def _rms_error(got, ref):
    return np.sqrt(np.mean((got - ref) ** 2) / np.mean(ref ** 2))


# (up to 640 to 2048 rows, by width, slabs have at most sixteen rows; above: split products)
REVERSE = [(16, 32, 5, 3), (48, 64, 33, 80), (64, 96, 1, 40), (64, 128, 17, 60), (64, 128, 17, 150), (96, 160, 40, 65), (32, 32, 20, 140),
           (64, 256, 33, 160)]


@pytest.mark.parametrize("F,H,n,C", REVERSE)
def test_every_gradient_against_64_bits(B, F, H, n, C):
    graphs, layers, biases, head, target = _all_pass(F, H, n, C, F + H + n)
    got, ref = _gradients(B, F, H, graphs, layers, biases, head(), target)
    errors = {k: _rms_error(x, y) for k, x, y in
              (("W0", got.W[0], ref.W[0]), ("W1", got.W[1], ref.W[1]), ("b0", got.b[0], ref.b[0]), ("b1", got.b[1], ref.b[1]),
               ("head W1", got.W1, ref.W1), ("head W2", got.W2, ref.W2), ("head w3", got.w3, ref.w3))}
    print(F, H, n, C, {k: f"{e:.2e}" for k, e in errors.items()})
    assert errors.pop("W0") <= BOUND_REVERSE
    assert max(errors.values()) <= BOUND_ONE_SIGN, errors


# A column of X, or an entry of a layer's matrix, whose first piece rounds to infinity although the gradients are finite: what
# does not meet it keeps its bits, the rest has the gradient's value.
@pytest.mark.parametrize("F,H,n,C", REVERSE)
@pytest.mark.parametrize("where", ["X", "W"])
def test_gradients_with_values_that_the_pieces_cannot_hold(B, F, H, n, C, where):
    grads = []
    for scale in (-64, 0):
        graphs, layers, biases, head, target = _all_pass(F, H, n, C, F + H + n)
        k = 5
        if where == "X":                                     # that row meets no weight on the way up
            layers[0][k::F] = 0.0
            for g in graphs:
                g.X[:, k] = 0.0
            graphs[C // 2].X[n // 2, k] = np.float32(3.4e38) * np.float32(2.0 ** scale)
        else:                                                # h1[:, k] makes up for it: the same bits on the way up
            layers[0][:, k] = 0.0
            layers[1][k::H] = 0.0
            layers[1][k, 3] = np.float32(3.4e38) * np.float32(2.0 ** scale)
            biases[0, k] = np.float32(2.0 ** (-126 - scale))
        grads.append(_gradients(B, F, H, graphs, layers, biases, head(), target))
    (plain, _), (got, ref) = grads
    meets = np.zeros(got.W[0].shape, bool)
    if where == "X":
        meets[k::F] = True
    else:
        meets[:, k] = True
    assert np.isfinite(ref.W[0]).all() and np.isfinite(got.W[0]).all()
    assert _rms_error(got.W[0][~meets], ref.W[0][~meets]) <= BOUND
    assert np.abs(ref.W[0][meets]).max() > 1e20
    # one entry of dZ decides them all: its own error, not the average over many (1e-5: what gradients are held to elsewhere)
    assert _rms_error(got.W[0][meets] / 1e30, ref.W[0][meets] / 1e30) <= 1e-5
    assert np.array_equal(got.W[0][~meets], plain.W[0][~meets])
    for x, y in ((got.W[1], plain.W[1]), (got.W1, plain.W1), (got.W2, plain.W2)):
        keep = np.ones(x.shape, bool)
        if where == "W" and x is got.W[1]:
            keep[k::H] = False                               # their h differs
        assert np.array_equal(x[keep], y[keep])
