"""The work that a program has this library do, as cases that can be timed and checked.

A case is one call, or the few calls that belong together, on a graph of one of the repository's families:

    spmm       Y = A_hat X (groot_spmm_execute): the aggregation of a GraphSAGE-mean layer, for inference and training
    spmm_t     dX = A_hat^T dY: the same call on the transposed graph, whose weights are explicit (backward pass)
    layer      one fused layer H = relu((A_hat X) Wn + X Ws + b) (inference)
    layer_dw   the fused layer's two weight gradients
    train      the last layer of a classifier in a training step: forward without an activation, the input gradient and
               the gradients of weights and bias from the loss gradient dZ
    partition  a graph cut into parts: every part with its re-grown boundary and its plan is built on the GPU, and its
               rows of Y = A_hat X are computed in place

Graphs: "csa" (carry-save multiplier AIG, 8 n^2 - 7 n nodes per copy), "booth" (radix-4 Booth multiplier AIG, more and
longer high-degree rows), "lut4" (carry-save array mapped to 4-input LUTs, rows of 7 entries, arrives as CSR arrays) and
"stress" (1 % of the rows hold nearly all entries, `bits` = log2 of its rows).  `batch` copies lie block-diagonally.
"""
import functools
import math

import numpy as np
import torch

import paper_2511_18297_amd as G
import workloads as wl

THRESHOLD = 32                       # degree threshold of the plans: the library's usual one


def listed():
    return [
        # the smallest aggregation a user runs: one 32-bit multiplier, 8 thousand rows; latency and launches
        dict(name="spmm_csa32_F32", op="spmm", graph="csa", bits=32, batch=1, F=32),
        # an ordinary verification run: one 256-bit multiplier, half a million rows, fits the last-level cache
        dict(name="spmm_csa256_F64", op="spmm", graph="csa", bits=256, batch=1, F=64),
        # the paper's kernel evaluation: Booth profile at 512 bits, embedding width 32
        dict(name="spmm_booth512x4_F32", op="spmm", graph="booth", bits=512, batch=4, F=32),
        # large batched graph: 1024-bit multiplier, 67 million rows, two matrices of 17 GB
        dict(name="spmm_csa1024x8_F64", op="spmm", graph="csa", bits=1024, batch=8, F=64),
        # polarized degrees: 2600 rows hold nearly all of the entries, widest embedding in use
        dict(name="spmm_stress18_F128", op="spmm", graph="stress", bits=18, batch=1, F=128),
        # a mapped netlist with longer rows and a width that is no power of two
        dict(name="spmm_lut256x8_F100", op="spmm", graph="lut4", bits=256, batch=8, F=100),
        # backward aggregation of an unfused training loop
        dict(name="spmm_t_csa512x4_F64", op="spmm_t", graph="csa", bits=512, batch=4, F=64),
        # inference layer at the hidden width, 8.4 million rows
        dict(name="layer_csa512x4_64_64", op="layer", graph="csa", bits=512, batch=4, F=64, F_out=64),
        # weight gradients at the hidden width, 8.4 million rows
        dict(name="layer_dw_csa512x4_64_64", op="layer_dw", graph="csa", bits=512, batch=4, F=64, F_out=64),
        # a training step on the small multipliers that models are trained on
        dict(name="train_csa64_32_32", op="train", graph="csa", bits=64, batch=1, F=32, F_out=32),
        # a training step on a large graph, narrowing layer
        dict(name="train_booth512x2_64_32", op="train", graph="booth", bits=512, batch=2, F=64, F_out=32),
        # a graph taken part by part
        dict(name="partition_csa512x4_8_F64", op="partition", graph="csa", bits=512, batch=4, F=64, parts=8),
    ]


# rows of one copy, and stored entries of a row on average (self-loops included)
_ROWS = {"csa": lambda b: 8 * b * b - 7 * b, "booth": lambda b: 8.28 * b * b, "lut4": lambda b: 2 * b * b + 6 * b,
         "stress": lambda b: 2 ** b}
_ENTRIES = {"csa": lambda b: 5.0, "booth": lambda b: 5.0, "lut4": lambda b: 8.9,
            "stress": lambda b: 11.6 * 2 ** (0.665 * (b - 14))}


def draw(rng):
    op = rng.choice(["spmm", "spmm", "spmm", "spmm_t", "layer", "layer_dw", "train", "partition"])
    graph = rng.choice({"spmm": ["csa", "booth", "lut4", "stress"], "spmm_t": ["csa", "booth"]}.get(op, ["csa", "booth"]))
    batch = rng.choice([1, 1, 2, 3, 4, 8])
    if graph == "stress":
        bits, batch = rng.randint(14, 18), 1
    else:
        low, high = {"spmm": (16, 512), "partition": (64, 384), "train": (8, 384)}.get(op, (16, 384))
        bits = int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))
        if graph == "booth":
            bits += bits % 2
    case = dict(op=op, graph=graph, bits=bits, batch=batch)
    if op in ("spmm", "spmm_t", "partition"):
        case["F"] = rng.choice([32, 64, 128, 32, 64, 128, 4 * rng.randint(1, 50)])
        if op == "partition":
            case["parts"] = rng.randint(2, 9)
    else:
        case["F"] = rng.choice([32, 64])
        case["F_out"] = rng.choice([32, 64] if op == "train" else [16, 32, 64])
    return case


# ---------------------------------------------------------------------------------------------------------------
# graphs: one copy's AIG or the CSR arrays, the same for every seed (a user has the netlist; the features change)
# ---------------------------------------------------------------------------------------------------------------
@functools.lru_cache(maxsize=None)
def _netlist(graph, bits, batch):
    if graph == "csa":
        return wl.csa_multiplier_aig(bits)
    if graph == "booth":
        return wl.booth_multiplier_aig(bits)
    if graph == "lut4":
        return wl.lut4_csa_graph(bits, batch)
    return wl.stress_graph(7, 2 ** bits, window=1024, dmax=2 ** (bits - 2))


def _graph(case):
    net = _netlist(case["graph"], case["bits"], case["batch"])
    if case["graph"] in ("csa", "booth"):
        return G.groot_graph_build(net.type, net.fanin0, net.fanin1, case["batch"])
    return G.groot_graph_from_csr(net.rowptr, net.col, net.val)


def _size(case):
    """(rows, stored entries) of the whole graph, about"""
    n = _ROWS[case["graph"]](case["bits"]) * case["batch"]
    return n, n * _ENTRIES[case["graph"]](case["bits"])


# ---------------------------------------------------------------------------------------------------------------
# inputs: features and weights as the repository's own model has them, U(-1, 1) and U(-1/8, 1/8); the loss gradient is
# that of a mean over all nodes
# ---------------------------------------------------------------------------------------------------------------
def _inputs(case, n, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)

    def uniform(rows, cols, scale):
        return torch.empty((rows, cols), device="cuda").uniform_(-scale, scale, generator=g)
    x = {"X": uniform(n, case["F"], 1.0)}
    if case["op"] in ("layer", "train"):
        x["Wn"], x["Ws"] = (uniform(case["F"], case["F_out"], 0.125) for _ in range(2))
        x["b"] = uniform(1, case["F_out"], 0.125)[0]
    if case["op"] in ("layer_dw", "train"):
        x["dZ"] = uniform(n, case["F_out"], 1.0 / n)
    return x


def prepare(case, seed):
    graph = _graph(case)
    if case["op"] == "spmm_t":
        graph = G.groot_graph_transpose(graph)
    plan = G.groot_spmm_plan(graph, THRESHOLD)
    G.groot_plan_upload(plan, max(case["F"], case.get("F_out", 0)))
    n, F = plan.n_rows, case["F"]
    s = dict(_inputs(case, n, seed), op=case["op"], plan=plan, n=n, parts=case.get("parts"), F=F)
    like = lambda rows, cols: torch.empty((rows, cols), device="cuda")  # noqa: E731
    if case["op"] in ("spmm", "spmm_t", "partition"):
        s["Y"] = like(n, F)
    elif case["op"] in ("layer", "train"):
        s["H"] = like(n, case["F_out"])
    if case["op"] in ("layer_dw", "train"):
        s["dW"] = torch.empty((2, F, case["F_out"]), device="cuda")
        s["work"] = torch.empty(G.groot_sage_layer_backward_weights_workspace(plan, F, case["F_out"]) // 4, device="cuda")
    if case["op"] == "train":
        s["scaled"], s["dX"] = like(n, case["F_out"]), like(n, F)
    return s


def run(s):
    op, plan = s["op"], s["plan"]
    if op in ("spmm", "spmm_t"):
        G.groot_spmm_execute(plan, s["X"], s["Y"])
        return s["Y"]
    if op == "layer":
        G.groot_sage_layer_forward_io(plan, s["X"], s["Wn"], s["Ws"], s["b"], True, s["H"])
        return s["H"]
    if op == "layer_dw":
        G.groot_sage_layer_backward_weights(plan, s["X"], s["dZ"], s["dW"][0], s["dW"][1], s["work"])
        return s["dW"]
    if op == "train":
        G.groot_sage_layer_forward_io(plan, s["X"], s["Wn"], s["Ws"], s["b"], False, s["H"])
        G.groot_rows_over_degree(plan, s["dZ"], s["scaled"])
        G.groot_sage_layer_backward_data(plan, s["scaled"], s["Wn"].t().contiguous(), s["Ws"].t().contiguous(), s["dX"])
        G.groot_sage_layer_backward_weights(plan, s["X"], s["dZ"], s["dW"][0], s["dW"][1], s["work"])
        return {"H": s["H"], "dX": s["dX"], "dW": s["dW"], "db": s["dZ"].sum(0)}
    counts = []
    for p in range(s["parts"]):
        part = G.groot_partition_regrow_device(plan, s["parts"], p)
        v = G.groot_dev_part_view(part)
        sub = G.groot_dev_part_plan(part, THRESHOLD, s["F"])
        G.groot_plan_use_global_columns(sub, v["global_id"], s["n"])
        G.groot_spmm_execute_rows(sub, s["X"], s["Y"], s["F"], v["n_owned"], v["global_id"])
        counts.append([v["n_owned"], v["n_halo"], v["n_crossing"], v["nnz"]])
    return {"Y": s["Y"], "counts": np.array(counts)}


def work(case):
    """The matrix as 8-byte row pointers and 4-byte columns (and 4-byte weights where they are explicit), every feature
    matrix once; partition: the parts' matrices are written once on top."""
    n, nnz = _size(case)
    F, Fo = case["F"], case.get("F_out", 0)
    matrix = 8 * n + 4 * nnz
    aggregate, dense = 2 * nnz * F, 2 * n * 2 * F * Fo
    if case["op"] == "spmm":
        return {"bytes": matrix + 8 * n * F, "flops": aggregate}
    if case["op"] == "spmm_t":
        return {"bytes": matrix + 4 * nnz + 8 * n * F, "flops": aggregate}
    if case["op"] == "layer":
        return {"bytes": matrix + 4 * n * (F + Fo), "flops": aggregate + dense}
    if case["op"] == "layer_dw":
        return {"bytes": matrix + 4 * n * (F + Fo), "flops": aggregate + dense}
    if case["op"] == "train":                            # X, dZ, H, dX once each
        return {"bytes": matrix + 4 * n * 2 * (F + Fo), "flops": aggregate + 2 * nnz * Fo + aggregate + 3 * dense}
    return {"bytes": 2 * matrix + 8 * n * F, "flops": aggregate}


def tolerance(case):
    """fp32 sums in an order of their own, as measured against exact(): 4.5e-8 for the aggregation, 1.5e-7 for a layer
    (2 F more terms), 1.3e-5 for weight gradients (sums over all rows whose terms mostly cancel)."""
    if case["op"] in ("spmm", "spmm_t", "partition"):
        return {"rel": 3e-7, "max": 3e-6}
    if case["op"] == "layer":
        return {"rel": 6e-7, "max": 1e-5}
    return {"rel": 6e-5, "max": 6e-4}


# ---------------------------------------------------------------------------------------------------------------
# the same in 64 bits with plain torch
# ---------------------------------------------------------------------------------------------------------------
def _entries(case):
    """(rows, columns, weights in fp64, rows of one copy, copies): one copy's stored entries, sorted by row and column"""
    net = _netlist(case["graph"], case["bits"], case["batch"])
    if case["graph"] in ("csa", "booth"):
        n, copies = int(net.type.shape[0]), case["batch"]
        f = torch.from_numpy(np.stack([net.fanin0, net.fanin1])).cuda().long()
        here = torch.arange(n, device="cuda").expand(2, n)
        src, dst = f[f >= 0] >> 1, here[f >= 0]
        every = torch.arange(n, device="cuda")
        key = torch.unique(torch.cat([src * n + dst, dst * n + src, every * n + every]))
        row, col = key // n, key % n
    else:
        n, copies = net.n, 1
        length = torch.from_numpy(np.diff(net.rowptr)).cuda()
        row = torch.repeat_interleave(torch.arange(n, device="cuda"), length)
        col = torch.from_numpy(net.col).cuda().long()
    w = 1.0 / torch.bincount(row, minlength=n).to(torch.float32)[row]     # fp32, as the library states its weights
    return row, col, w.double(), n, copies


def _product(entries, x, transposed=False):
    """A_hat x (or A_hat^T x) in fp64, copy by copy, a few million entries at a time"""
    row, col, w, n, copies = entries
    if transposed:
        row, col = col, row
    y = torch.zeros((n * copies, x.shape[1]), dtype=torch.float64, device="cuda")
    step = max(1, (1 << 28) // x.shape[1])
    for c in range(copies):
        xc, yc = x[c * n:(c + 1) * n], y[c * n:(c + 1) * n]
        for b in range(0, row.shape[0], step):
            e = slice(b, b + step)
            yc.index_add_(0, row[e], xc[col[e]].double() * w[e, None])
    return y


def exact(case, seed):
    e = _entries(case)
    x = _inputs(case, e[3] * e[4], seed)
    op = case["op"]
    if op in ("spmm", "spmm_t"):
        return _product(e, x["X"], op == "spmm_t")
    agg = _product(e, x["X"])
    if op == "partition":
        return {"Y": agg, "counts": None}
    X = x["X"].double()
    if op == "layer_dw":
        dZ = x["dZ"].double()
        return torch.stack([agg.t() @ dZ, X.t() @ dZ])
    Wn, Ws = x["Wn"].double(), x["Ws"].double()
    H = agg @ Wn + X @ Ws + x["b"].double()
    if op == "layer":
        return H.clamp_(min=0)
    dZ = x["dZ"].double()
    return {"H": H, "dX": _product(e, x["dZ"], True) @ Wn.t() + dZ @ Ws.t(),
            "dW": torch.stack([agg.t() @ dZ, X.t() @ dZ]), "db": dZ.sum(0)}
