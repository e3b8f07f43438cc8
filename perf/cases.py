"""The work that a user of this framework has it do, as timed cases: candidate evaluation (contraction + estimator),
Cost(H'), the backtracking search and the training pass of the estimator, each through the public binding.

A case names a module (the base training DAG), a batch of candidates on it and an estimator.  The modules are those
of the repository's configurations: the 72-node layered DAG, the ResNet-50-shaped and the transformer-shaped training
DAG, and the heterogeneous set of power-law DAGs; drawn cases vary their size.  Graph structure depends on the case
only; features, profiled times, tensor sizes, weights, candidates and targets are made from the seed.
"""
import functools
import math

import numpy as np
import torch

from paper_2209_12769_amd import binding as B
from paper_2209_12769_amd import workloads as wl

DEV = "cuda:0"
AR_C, AR_D = 0.02, 0.01                  # T = C x + D of the all-reduce model, x in MiB
SEARCH = {"alpha": 1.05, "beta": 10}     # the defaults of the search
NODES_MOST = 4096 * 6563                 # labels of one batch: the benchmark's largest single-module batch

# The modules by size.  transformer: blocks and element-wise ops per major op; mixed: number of graphs and op range.
BERT = {"module": "transformer", "blocks": 12, "ew": 2, "embed": 5, "tail": 3}
LARGE = {"module": "transformer", "blocks": 24, "ew": 9, "embed": 10, "tail": 6}


def listed():
    def model(F, H, L, dtype, heads=0):
        return {"F": F, "H": H, "L": L, "dtype": dtype, "heads": heads}
    return [
        # one candidate of a small module at a time: what an interactive caller waits for; launches and latency
        {"name": "eval_tiny_one", "do": "eval", "module": "tiny", "cands": 1, "rule": "runs", "kmax": 2, **model(16, 32, 2, "f32")},
        # fp32 estimator on a ResNet-50-sized module
        {"name": "eval_resnet50_f32", "do": "eval", "module": "resnet50", "cands": 256, "rule": "chains", "kmax": 4, **model(32, 128, 3, "f32")},
        # the two halves of an evaluation called on their own, the contracted batch kept by the caller
        {"name": "contract_forward_bert", "do": "contract_forward", **BERT, "cands": 1024, "rule": "chains", "kmax": 4, **model(32, 128, 3, "bf16")},
        # a handful of candidates of a large module: a search that expands few parents per step
        {"name": "eval_large_few", "do": "eval", **LARGE, "cands": 7, "rule": "runs", "kmax": 8, **model(64, 256, 4, "bf16")},
        # the headline batch
        {"name": "eval_large", "do": "eval", **LARGE, "cands": 4096, "rule": "runs", "kmax": 8, **model(64, 256, 4, "bf16")},
        # candidates of 64 modules of very different size in one batch
        {"name": "eval_mixed", "do": "eval", "module": "mixed", "graphs": 64, "n_lo": 100, "n_hi": 20000, "cands": 8192, "rule": "geometric", "kmax": 0, **model(64, 256, 4, "bf16")},
        # the attention form of the estimator, an odd number of candidates
        {"name": "eval_attention", "do": "eval", **LARGE, "cands": 1001, "rule": "runs", "kmax": 8, **model(64, 256, 4, "bf16", 4)},
        # Cost(H') of fused modules
        {"name": "cost_large", "do": "cost", **LARGE, "cands": 4096, "rule": "runs", "kmax": 8, **model(64, 256, 4, "bf16")},
        # Cost(H') of the children that a search makes: modules close to the unfused one
        {"name": "cost_children", "do": "cost", **LARGE, "cands": 1000, "rule": "merges", "kmax": 24, **model(64, 256, 4, "bf16")},
        # the search itself, few parents per step
        {"name": "search_resnet50", "do": "search", "module": "resnet50", "parents": 8, "steps": 24, **model(32, 128, 3, "f32")},
        # forward, loss and reverse pass on a small and on a large batch of fused-op samples
        {"name": "train_resnet50", "do": "train", "module": "resnet50", "cands": 6, **model(32, 128, 3, "f32")},
        {"name": "train_large", "do": "train", **LARGE, "cands": 128, **model(64, 256, 4, "f32")},
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    do = rng.choice(["eval", "eval", "eval", "contract_forward", "cost", "cost", "search", "train"])
    case = {"do": do}
    kind = rng.choice(["tiny", "resnet50", "transformer", "transformer", "mixed"])
    if do in ("search", "train") and kind == "mixed":
        kind = "transformer"
    case["module"] = kind
    if kind == "transformer":
        case.update(blocks=log_int(1, 24), ew=rng.randint(1, 9), embed=rng.randint(2, 10), tail=rng.randint(1, 6))
    elif kind == "mixed":
        lo = log_int(60, 2000)
        case.update(graphs=rng.randint(2, 64), n_lo=lo, n_hi=min(20000, lo * rng.randint(2, 40)))
    # the configurations' widths most of the time, any supported one otherwise
    F, H, L = rng.choice([(16, 32, 2), (32, 128, 3), (64, 256, 4), (64, 256, 4), None, None]) or (
        16 * rng.randint(1, 6), rng.choice([32, 64, 128, 256] if do in ("eval", "contract_forward") else [32, 64, 96, 128, 160, 192, 256]), rng.randint(2, 5))
    dtype = "f32" if do in ("search", "train") else rng.choice(["f32", "bf16", "bf16"])
    heads = rng.choice([0, 0, 0, 2, 4]) if do in ("eval", "contract_forward") else 0
    case.update(F=F, H=H, L=L, dtype=dtype, heads=heads)
    n = sum(g.n for g in _module(_key(case))) / len(_module(_key(case)))
    # fp32 products run at a sixteenth of the bf16 rate: the batch shrinks so that no draw is longer than the largest
    # listed case
    most = NODES_MOST / (16 if dtype == "f32" else 1) / (4 if heads else 1)
    if do == "search":
        case.update(parents=log_int(1, 64), steps=min(rng.randint(4, 40), max(4, int(30000 / n))))
    elif do == "train":
        case["cands"] = min(log_int(2, 400), max(1, int(128 * 6563 / n)))
    else:
        case["rule"] = rng.choice(["runs", "runs", "chains", "geometric"] + (["merges"] if do == "cost" and kind != "mixed" else []))
        case["kmax"] = {"runs": rng.randint(2, 10), "chains": rng.randint(2, 6), "geometric": 0, "merges": rng.randint(1, 40)}[case["rule"]]
        if case["rule"] == "merges":
            most /= 4
        case["cands"] = max(1, min(log_int(1, 8192), int(most / n)))
        if kind == "mixed":
            case["cands"] = max(case["graphs"], case["cands"] // case["graphs"] * case["graphs"])
    return case


# ---- modules ---------------------------------------------------------------------------------------------------
def _key(case):
    return tuple(sorted((k, v) for k, v in case.items() if k in ("module", "blocks", "ew", "embed", "tail", "graphs", "n_lo", "n_hi")))


@functools.lru_cache(maxsize=32)
def _module(key):
    """The base graphs of a case, without features."""
    k = dict(key)
    if k["module"] == "tiny":
        return wl.cfg1(1).graphs
    if k["module"] == "resnet50":
        return wl.cfg2(1).graphs
    if k["module"] == "mixed":
        return wl.cfg5(k["graphs"], n_graphs=k["graphs"], n_lo=k["n_lo"], n_hi=k["n_hi"]).graphs
    n, n_op, src, dst = wl._transformer_dag(k["blocks"], k["ew"], k["embed"], k["tail"])
    rowptr, col = wl._csr_from_edges(n, src, dst)
    return [wl.BaseGraph(n, n_op, rowptr, col, np.zeros((n, 0), np.float32))]


def _with_features(graphs, F, rng):
    """Features as in the configurations: U(0,1); column 0 of an all-reduce node is its size in MiB (4 KB to 50 MB,
    log-uniform), column 1 tells ops from tensors."""
    out = []
    for g in graphs:
        X = rng.random((g.n, F), dtype=np.float32)
        X[:, 1] = np.arange(g.n) >= g.n_op
        X[g.n_op:, 0] = np.exp(rng.uniform(math.log(4e3), math.log(50e6), g.n - g.n_op)) / (1 << 20)
        out.append(wl.BaseGraph(g.n, g.n_op, g.rowptr, g.col, X))
    return out


# ---- candidates, made on the GPU ----------------------------------------------------------------------------------
def _run_starts(C, n, kmax, gen):
    """Start flags of runs of 1..kmax places (kmax = 0: geometric with mean 2.5)."""
    if kmax == 0:
        f = torch.rand((C, n), device=DEV, generator=gen) < 0.4
    else:
        lens = torch.randint(1, kmax + 1, (C, n), device=DEV, generator=gen, dtype=torch.int32)
        pos = torch.cumsum(lens, 1, dtype=torch.int32) - lens
        f = torch.zeros((C, n + 1), dtype=torch.bool, device=DEV)
        f.scatter_(1, pos.clamp_(max=n).long(), True)
        f = f[:, :n].contiguous()
    f[:, 0] = True
    return f


def _interval_labels(g, C, rule, kmax, gen):
    """Intervals of the topological order as fused ops (rule "chains": only along producer-consumer pairs), runs of
    neighbouring tensors as buckets; the label of a group is arbitrary."""
    f = _run_starts(C, g.n_op, kmax, gen)
    if rule == "chains":
        src = np.repeat(np.arange(g.n), np.diff(g.rowptr))
        linked = np.zeros(g.n, bool)
        linked[g.col[g.col == src + 1]] = True
        f |= ~torch.from_numpy(linked[:g.n_op]).to(DEV)
    if g.n > g.n_op:
        f = torch.cat([f, _run_starts(C, g.n - g.n_op, 0 if rule == "geometric" else 20, gen)], 1)
    run = torch.cumsum(f, 1, dtype=torch.int32) - 1
    perm = torch.argsort(torch.rand((C, g.n), device=DEV, generator=gen), 1)
    return torch.gather(perm, 1, run.long()).to(torch.int32).reshape(-1)


def _merged_labels(g, C, most, gen):
    """Children of a search after a few steps: on the unfused module up to `most` ops fused with their only predecessor
    (which leaves a module valid, as the entries of the search's queue are) and a few neighbouring tensors joined; one
    child in ten has fused the ends of some other dependency too, which mostly makes it invalid."""
    src = np.repeat(np.arange(g.n), np.diff(g.rowptr))
    indeg = np.bincount(g.col, minlength=g.n)
    every = np.nonzero(g.col < g.n_op)[0]
    sole = np.nonzero((g.col < g.n_op) & (indeg[g.col] == 1))[0]
    src, dst, every, sole = (torch.from_numpy(np.asarray(x, np.int64)).to(DEV) for x in (src, g.col, every, sole))
    lab = torch.arange(g.n, device=DEV, dtype=torch.int32).repeat(C, 1)
    times = torch.randint(1, most + 1, (C, 1), device=DEV, generator=gen)
    for k in range(most + 1):
        edges = sole if k < most else every
        on = times > k if k < most else torch.rand((C, 1), device=DEV, generator=gen) < 0.1
        e = edges[torch.randint(0, edges.numel(), (C,), device=DEV, generator=gen)]
        a, b = lab.gather(1, src[e][:, None]), lab.gather(1, dst[e][:, None])
        lab = torch.where((lab == a) & on, b, lab)
        if k % 3 == 0 and g.n - g.n_op > 1:
            t = torch.randint(g.n_op, g.n - 1, (C, 1), device=DEV, generator=gen)
            a, b = lab.gather(1, t), lab.gather(1, t + 1)
            lab = torch.where((lab == b) & on, a, lab)
    return lab.reshape(-1)


def _sample_labels(g, C):
    """Labelings whose groups are training samples: in most of the module an op joins one of its predecessors with
    probability 0.88, so that fused ops are connected and have about eight members and a long tail; the rest and the
    tensors stay single.  The same for every seed: the shapes of a training pass's results depend on them."""
    gen = torch.Generator(device=DEV).manual_seed(1)
    src = np.repeat(np.arange(g.n), np.diff(g.rowptr))
    order = np.argsort(g.col, kind="stable")
    pred = torch.from_numpy(np.append(src[order], 0)).to(DEV)
    deg = np.bincount(g.col, minlength=g.n)
    first = torch.from_numpy(np.cumsum(deg) - deg).to(DEV)
    deg = torch.from_numpy(deg).to(DEV)
    pick = first + (torch.rand((C, g.n), device=DEV, generator=gen, dtype=torch.float64) * deg).long().clamp_(max=g.n)
    p = pred[pick.clamp_(max=pred.numel() - 1)]
    area = torch.rand((C, g.n // 48 + 1), device=DEV, generator=gen).repeat_interleave(48, 1)[:, :g.n] < 0.66
    area[:, :48] = True
    own = torch.arange(g.n, device=DEV)
    join = area & area.gather(1, p) & (torch.rand((C, g.n), device=DEV, generator=gen) < 0.88) & (deg > 0) & (own < g.n_op)
    root = torch.where(join, p, own)
    for _ in range(max(1, int(math.ceil(math.log2(g.n))))):
        root = root.gather(1, root)
    return root.to(torch.int32).reshape(-1)


def _candidates(case, graphs, gen):
    """(cand_graph, cand_off, labels) on the GPU."""
    per = max(1, case["cands"] // len(graphs))
    parts = []
    for g in graphs:
        if case["do"] == "train":
            parts.append(_sample_labels(g, per))
        elif case["rule"] == "merges":
            parts.append(_merged_labels(g, per, case["kmax"], gen))
        else:
            parts.append(_interval_labels(g, per, case["rule"], case["kmax"], gen))
    cg = np.repeat(np.arange(len(graphs), dtype=np.int32), per)
    off = np.concatenate([[0], np.cumsum([graphs[b].n for b in cg])]).astype(np.int32)
    return torch.from_numpy(cg).to(DEV), torch.from_numpy(off).to(DEV), torch.cat(parts)


# ---- the cases -------------------------------------------------------------------------------------------------
def prepare(case, seed):
    rng = np.random.default_rng(seed)
    gen = torch.Generator(device=DEV).manual_seed(int(seed))
    graphs = _with_features(_module(_key(case)), case["F"], rng)
    model = wl.ModelSpec(case["F"], case["H"], case["L"], case["dtype"], "attention" if case["heads"] else "mean", max(1, case["heads"]))
    # a trained estimator puts out times: the last layer is taken non-negative
    w = wl.with_time_like_head(wl.custom("case", model, graphs, [np.zeros((1, g.n), np.int32) for g in graphs], seed=int(seed) % (1 << 20)))
    head = w.weights.head
    if case["do"] in ("cost", "search"):
        head[-(model.H + 1):] *= 0.02    # of a fused op: about the time of one of its ops, so that fusing pays
        head[-1] = 0.4
    else:
        head[-1] += 1.0
    n_most, e_most = max(g.n for g in graphs), max(g.e for g in graphs)
    s = {"do": case["do"]}
    if case["do"] == "search":
        C, nb, eb = 2 * case["parents"], 2 * case["parents"] * n_most, 2 * case["parents"] * e_most
    else:
        s["cand_graph"], s["cand_off"], s["labels"] = _candidates(case, graphs, gen)
        per = s["cand_graph"].numel() // len(graphs)
        C, nb, eb = per * len(graphs), per * sum(g.n for g in graphs), per * sum(g.e for g in graphs)
    keep = nb // 2 + 1 if case["do"] == "train" else C       # training: graphs of a batch are fused ops
    ev = s["ev"] = B.Evaluator(model.F, model.H, model.L, model.dtype, keep, nb, eb, device=DEV, agg=model.agg, heads=model.heads,
                               # intervals at least halve a large batch's nodes; a small one is not worth the thought
                               max_nodes=int(0.75 * nb) if case["do"] == "eval" and nb > 1 << 23 else 0)
    ev.set_base_graphs(w.g_node_off(), w.g_edge_off(), w.cat_rowptr(), w.cat_col(), w.cat_X())
    ev.set_weights(w.weights)
    if case["do"] in ("cost", "search", "train"):
        ev.set_profile(*wl.profile_of(w))
    if case["do"] == "contract_forward":
        s["batch"] = ev.alloc_batch(C, nb, nb, eb)
        for k in ("out_rowptr", "out_col", "in_rowptr", "in_col", "Xc"):
            getattr(s["batch"], k).zero_()                   # the part beyond the contracted batch is never written
    if case["do"] == "search":
        s["kw"] = dict(graph=0, n_nodes=n_most, seed=int(seed), ar_c=AR_C, ar_d=AR_D, parents=case["parents"],
                       max_steps=case["steps"], max_queue=max(64, 4 * case["parents"]), op_draw=B.DC_DRAW_OP, **SEARCH)
    if case["do"] == "train":
        s["batch"] = ev.fused_op_batch(s["cand_graph"], s["cand_off"], s["labels"], ev.alloc_batch(nb // 2 + 1, nb, nb, eb))
        K, M, _ = ev.last_fused_ops()
        size = (s["batch"].node_off[1:K + 1] - s["batch"].node_off[:K]).float()
        s["target"] = size.pow(0.8) * (0.3 + 0.6 * torch.rand(K, device=DEV, generator=gen))
        ev.train_begin(1e-4, K, M)
    return s


def run(s):
    ev = s["ev"]
    if s["do"] == "eval":
        return ev.eval_candidates(s["cand_graph"], s["cand_off"], s["labels"])
    if s["do"] == "contract_forward":
        b = ev.contract_graphs(s["cand_graph"], s["cand_off"], s["labels"], s["batch"])
        return [ev.gnn_forward(b), b.node_off, b.edge_off, b.new_id, b.out_rowptr, b.out_col, b.in_rowptr, b.in_col, b.Xc]
    if s["do"] == "cost":
        return ev.cost_candidates(s["cand_graph"], s["cand_off"], s["labels"], AR_C, AR_D)
    if s["do"] == "search":
        labels, r = ev.search(**s["kw"])
        return [labels, r.cost_in, r.cost_opt, r.steps, r.evaluated, r.valid, r.enqueued, r.improved, r.queued, r.unchanged]
    return list(ev.loss_gradients(s["batch"], s["target"]))


def _groups(case, g):
    """Expected (groups of ops, groups of tensors) of one candidate."""
    rule, n_ar = case["rule"], g.n - g.n_op
    if rule == "merges":
        return g.n_op - case["kmax"] / 2, n_ar - case["kmax"] / 6
    mean = 2.5 if rule == "geometric" else (case["kmax"] + 1) / 2
    if rule == "chains":
        src = np.repeat(np.arange(g.n), np.diff(g.rowptr))
        chains = g.n_op - int(np.count_nonzero((g.col == src + 1) & (g.col < g.n_op)))
        return chains + (g.n_op - chains) / mean, n_ar / 10.5
    return g.n_op / mean, n_ar / (2.5 if rule == "geometric" else 10.5)


def _rows(case, graphs):
    """Expected contracted nodes of the batch."""
    return max(1, case["cands"] // len(graphs)) * sum(sum(_groups(case, g)) for g in graphs)


def work(case):
    """Labels, base graphs and weights read once, results written once; products of the estimator's layers."""
    graphs = _module(_key(case))
    F, H, L = case["F"], case["H"], case["L"]
    blocks = 1 if case["heads"] else 3
    row = sum(2 * blocks * (F if l == 0 else H) * H for l in range(L)) + (8 * H * L if case["heads"] else 0)
    params = sum(blocks * (F if l == 0 else H) * H for l in range(L)) + 2 * H * H
    s = 4 if case["dtype"] == "f32" else 2
    by = params * s + sum(g.n * (4 * F + 4) + 4 * g.e for g in graphs)
    if case["do"] == "search":
        g = graphs[0]
        C = 2 * case["parents"] * case["steps"]
        rows = C / 2 * SEARCH["beta"]                        # half of the children fuse ops, about five pairs each
        return {"bytes": by + 4 * g.n, "flops": rows * row + rows / 2 * 4 * H * H}
    per = max(1, case["cands"] // len(graphs))
    C, nb = per * len(graphs), per * sum(g.n for g in graphs)
    by += 4 * nb + 4 * C
    if case["do"] == "train":
        rows = 0.55 * nb
        data = sum(2 * 3 * H * H for l in range(1, L))
        return {"bytes": by - 4 * nb + rows * (4 * F + 16) + 8 * params, "flops": rows * (2 * row + data) + rows / 8 * 12 * H * H}
    n = _rows(case, graphs)
    if case["do"] in ("eval", "contract_forward"):
        e = per * sum(g.e for g in graphs) * min(1.0, 1.6 * n / nb)
        more = 4 * nb + n * (F * s + 8) + 8 * e if case["do"] == "contract_forward" else 0
        return {"bytes": by + more, "flops": n * row + C * 4 * H * H}
    # Cost(H'): equal fused ops of a batch have one estimate; intervals of k ops have at most n_op different places
    rows = ops = 0.0
    for g in graphs:
        if case["rule"] == "merges":
            rows, ops = rows + per * case["kmax"], ops + per * case["kmax"] / 2
        else:
            k = case["kmax"] or 6
            rows += min(per * g.n_op * 0.8, g.n_op * (k * (k + 1) / 2 - 1))
            ops += min(per * _groups(case, g)[0] * 0.7, g.n_op * (k - 1))
    return {"bytes": by, "flops": rows * row + ops * 4 * H * H}


def tolerance(case):
    """About four times the distance from the same formulas with 64-bit sums: bf16 predictions up to 7e-4, summed
    features (rounded once) 1.7e-3, costs up to 2e-4; fp32 predictions and losses 2e-8 to 2e-7, gradients 3e-7 with
    single entries 4e-5 of the root mean square."""
    if case["dtype"] == "f32":
        return {"rel": 5e-6, "max": 4e-4}
    return {"rel": {"contract_forward": 7e-3, "cost": 1e-3}.get(case["do"], 3e-3)}
