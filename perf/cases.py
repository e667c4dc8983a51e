"""The framework's work as a list of timed cases: whole mini-batch passes (forward, training step) of every operator
the executor runs, through the entry points a user's program calls.

Each case is one mini-batch of a seeded synthetic graph, with the batch subgraph's plans, the feature table, the
history tables and the weights in hand (`prepare`), and one pass over it (`run`).  Graph shapes, widths and batch
shares are those of the benchmark configurations, of the overhead experiment and of the training benchmarks, plus a
training step on odd sizes.
"""
import math

import torch

import paper_2106_05609_amd as gas
from paper_2106_05609_amd import executor
from gas_inputs import batches, graphs

ALPHA = 0.1                       # GCNII's initial residual
LEARNING_RATE = 0.01
FORWARD, TRAIN = "forward", "train"


def _case(name, op, mode, graph, n, blocks, per_batch, degree, f_in, hidden, f_out, layers, dtype="f32", heads=1,
          outside=0):
    c = dict(op=op, mode=mode, graph=graph, n=n, blocks=blocks, per_batch=per_batch, degree=degree, f_in=f_in,
             hidden=hidden, f_out=f_out, layers=layers, dtype=dtype, heads=heads, outside=outside)
    return dict(c, name=name) if name else c


def listed():
    return [
        # a citation-sized graph: one batch of 512 nodes, two narrow layers.  Launches and host time are all there is:
        # what an interactive query or a small experiment's inner loop pays
        _case("tiny-gcn-forward", "gcn", FORWARD, "sbm", 2048, 4, 1, 5, 64, 64, 64, 2),
        _case("tiny-gcn-train", "gcn", TRAIN, "sbm", 2048, 4, 1, 5, 64, 64, 64, 2),
        # the runtime-overhead experiment: a 4-layer GIN, 4,000 nodes with 60 links each, as many nodes outside the batch
        _case("overhead-gin-forward", "gin", FORWARD, "links", 8000, 2, 1, 60, 256, 256, 256, 4, outside=4000),
        # bag-of-words features and a class count that nothing divides, a few thousand nodes: the odd sizes of small
        # text graphs, trained
        _case("ragged-gcn-train", "gcn", TRAIN, "sbm", 19997, 8, 2, 10, 1433, 256, 47, 3),
        # the mid-size community graph: inference over one batch of 50,000 nodes
        _case("mid-gcn-forward", "gcn", FORWARD, "sbm", 200_000, 40, 10, 10, 128, 256, 256, 3),
        # the two anisotropic operators on the same graph, trained
        _case("mid-pna-train", "pna", TRAIN, "sbm", 200_000, 40, 10, 10, 128, 256, 256, 3),
        _case("mid-gat-train", "gat", TRAIN, "sbm", 200_000, 40, 10, 10, 128, 256, 256, 3, heads=4),
        # the deep narrow model: 64 layers of width 64, inference and training
        _case("deep-gcnii-forward", "gcnii", FORWARD, "sbm", 170_000, 32, 4, 14, 128, 64, 64, 64),
        _case("deep-gcnii-train", "gcnii", TRAIN, "sbm", 170_000, 32, 4, 14, 128, 64, 64, 64),
        # the large power-law graph (2.4 M nodes, hubs of up to 20,000 links), trained
        _case("large-gcn-train", "gcn", TRAIN, "power", 2_400_000, 64, 16, 50, 100, 256, 256, 3),
        # a tenth of the huge power-law graph in bf16: inference over one batch (312,500 nodes) and a training step
        _case("huge-gin-forward", "gin", FORWARD, "power", 5_000_000, 512, 32, 30, 128, 256, 256, 3, dtype="bf16"),
        _case("huge-gin-train", "gin", TRAIN, "power", 5_000_000, 512, 32, 30, 128, 256, 256, 3, dtype="bf16"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["gcn", "gcn", "gin", "gcnii", "pna", "gat"])
    mode = rng.choice([FORWARD, TRAIN])
    dtype = rng.choice(["f32", "f32", "bf16"]) if op != "gcnii" else "f32"
    blocks = rng.randint(4, 64)
    per_batch = max(1, blocks // rng.choice([4, 6, 8, 16]))
    hidden = 8 * rng.randint(4, 32)
    f_in, f_out = _log_int(rng, 40, 1500), rng.randint(2, 256)
    if rng.random() < 0.5:
        f_in = 32 * max(2, min(8, f_in // 32))
    if op == "gcnii":
        hidden = rng.choice([32, 48, 64, 64, 96, 128])
        return _case(None, op, mode, "sbm", _log_int(rng, 4_000, 200_000), blocks, per_batch, rng.randint(4, 20), f_in,
                     hidden, hidden, rng.randint(8, 64))
    if op == "gin" and mode == FORWARD and rng.random() < 0.3:
        nb = _log_int(rng, 500, 8_000)
        outside = int(nb * rng.uniform(0.1, 2.5))
        return _case(None, op, mode, "links", nb + outside, 2, 1, rng.randint(10, 60), f_in, hidden, hidden, 4, dtype,
                     outside=outside)
    if op in ("pna", "gat"):
        heads = rng.choice([1, 2, 4]) if op == "gat" else 1
        if op == "pna" and mode == TRAIN:
            dtype = "f32"        # in bf16 many neighbours tie for an extreme: which one is met first decides its gradient
        hidden = 32 * rng.randint(2, 8)
        return _case(None, op, mode, "sbm", _log_int(rng, 4_000, 200_000), blocks, per_batch, rng.randint(4, 20), f_in,
                     hidden, hidden, 3, dtype, heads)
    graph = rng.choice(["sbm", "power"])
    n = _log_int(rng, 2_000, 300_000) if graph == "sbm" else _log_int(rng, 20_000, 1_500_000)
    return _case(None, op, mode, graph, n, blocks, per_batch, rng.randint(4 if graph == "sbm" else 20, 40), f_in, hidden, f_out,
                 rng.randint(2, 4), dtype)


def _sizes(c):
    """Expected (in-batch rows, halo rows, entries) of the case's batch; exact counts depend on the seed."""
    if c["graph"] == "links":
        nb = c["n"] - c["outside"]
        return nb, c["outside"], nb * c["degree"] + c["outside"] * c["degree"]
    nb = c["n"] * c["per_batch"] // c["blocks"]
    nnz = nb * c["degree"]
    out = c["n"] - nb
    links_out = nnz * (0.15 if c["graph"] == "sbm" else 1.0) * out / c["n"]
    # distinct nodes outside the batch that the links name; a power law repeats its hubs, so it names fewer
    nh = int(out * (1.0 - math.exp(-links_out / max(1, out))) * (1.0 if c["graph"] == "sbm" else 0.67))
    return nb, nh, nnz + (nb if c["op"] != "gin" else 0)


def work(case):
    """Every table row, activation, weight and gradient once, at the storage type's size; the entries of the pattern
    once per layer and direction; multiply-adds of the aggregations and the products."""
    c = case
    nb, nh, nnz = _sizes(c)
    s = 4 if c["dtype"] == "f32" else 2
    train = c["mode"] == TRAIN
    entry = 4 + (4 if c["op"] in ("gcn", "gcnii") else 0)
    nbytes = flops = 0.0
    for l in range(c["layers"]):
        fi = (c["hidden"] if c["op"] == "gcnii" else c["f_in"]) if l == 0 else c["hidden"]
        fo = c["f_out"] if l == c["layers"] - 1 else c["hidden"]
        rows = nb + nh
        if c["op"] == "pna":
            f1 = max(8, fo // 4)
            dense = 2.0 * fi * f1 * (rows + nb) + 2.0 * (fi + 9 * f1) * fo * nb
            weights = 2 * fi * f1 + (fi + 9 * f1) * fo
            agg = 3.0 * nnz * f1
        elif c["op"] == "gat":
            dense, weights, agg = 2.0 * fi * fo * rows, fi * fo + 2 * fo, 6.0 * nnz * fo
        elif c["op"] == "gin":
            dense, weights, agg = 2.0 * nb * c["hidden"] * (fi + fo), c["hidden"] * (fi + fo), 2.0 * nnz * fi
        else:
            dense, weights, agg = 2.0 * nb * fi * fo, fi * fo, 2.0 * nnz * fi
        push = nb * fo * s if l < c["layers"] - 1 else 0
        nbytes += rows * fi * s + nb * fo * s + push + nnz * entry + weights * s
        flops += dense + agg
        if train:
            # output gradients in, both operands of the weight gradients, the input gradient of every layer but the first
            nbytes += nb * (2 * fo + fi) * s + weights * 8 + (nb * fi * s + nnz * entry if l > 0 else 0)
            flops += dense + (dense + agg if l > 0 else 0)
    if c["op"] == "gcnii":
        nbytes += (nb + nh) * (c["f_in"] + c["hidden"]) * s
        flops += 2.0 * (nb + nh) * c["f_in"] * c["hidden"] * (2 if train else 1)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """About four times the largest difference seen over 80 cases of these ranges between a pass and the same pass with
    its nodes and its input features in another order (every sum of the aggregations, of the first layer's products and
    of the weight gradients in another order)."""
    c = case
    if c["dtype"] == "bf16":
        # one storage rounding per tensor; GIN's unnormalised sums carry it through hubs of thousands of neighbours, whose
        # rows set the scale (largest single difference seen: 0.19 of an output's root mean square)
        return {"rel": 1e-2, "max": 0.75} if c["op"] == "gin" else {"rel": 6e-3, "max": 0.06}
    if c["mode"] == FORWARD:
        return {"rel": 1e-5, "max": 1e-4}       # largest single difference seen: 2.4e-5, in rows below a hub
    # a hidden unit (GAT: a score, PNA: a tie for an extreme) within rounding of its threshold may fall on either side,
    # and its whole gradient with it: 2e-4 (GCN, GCNII), 6e-4 (PNA) and 9e-4 (GAT) of a gradient's norm seen
    return {"rel": 4e-3 if c["op"] in ("gat", "pna") else 1e-3, "max": 2e-2}


def _graph(c, seed, dev):
    if c["graph"] == "links":
        return graphs.batch_with_outside_links(c["n"] - c["outside"], c["outside"], c["degree"], seed, dev)
    if c["graph"] == "power":
        cap = max(64, min(20_000, c["n"] // 120))
        return graphs.chung_lu_bfs_blocks(c["n"], 2.1 if c["degree"] >= 40 else 2.2, float(c["degree"]), cap, c["blocks"],
                                          seed, dev)
    return graphs.sbm_partners(c["n"], c["blocks"], float(c["degree"]), 0.85, seed, dev)


def prepare(case, seed):
    c, dev = case, torch.device("cuda:0")
    dt = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)

    def normal(*shape):
        return torch.randn(*shape, generator=gen, device=dev, dtype=dt)

    def glorot(fi, fo, scale=1.0):
        a = scale * math.sqrt(6.0 / (fi + fo))
        return ((torch.rand(fi, fo, generator=gen, device=dev) * 2 - 1) * a).to(dt)

    g = _graph(c, seed, dev)
    # the blocks of the batch are the same for every seed (the graph, the values and so the batch's pattern are not):
    # blocks differ by a node in size, and by much in entries where one of them holds the hubs
    batch = torch.arange(int(g.block_ptr[1])) if c["graph"] == "links" else batches.split(g, c["per_batch"], 0)[0]
    op, L, train = c["op"], c["layers"], c["mode"] == TRAIN
    sg = batches.batch_subgraph(g, batch, self_loops=op in ("gcn", "gcnii", "gat"))
    bg = executor.BatchGraph(sg.nb, sg.n_id, sg.rowptr, sg.col, g.deg, sg.colptr if train else None,
                             sg.row if train else None, max_F=max(c["f_in"], c["hidden"], c["f_out"]),
                             normalise=op in ("gcn", "gcnii"), csc_pos=sg.csc_perm if train else None)
    bg.src                                       # built on first use otherwise; a program builds it once per batch
    if train and op in ("gcnii", "pna", "gat"):
        bg.plan_t_all
    widths = [c["hidden"] if op == "gcnii" else c["f_in"]] + [c["hidden"]] * (L - 1) + [c["f_out"]]
    s = {"case": c, "bg": bg, "x": normal(c["n"], c["f_in"])}
    # stored embeddings are outputs of a ReLU; one block of memory, a table per layer
    s["tables"] = normal(max(1, L - 1), c["n"], c["hidden"]).clamp_(min=0)
    s["hist"] = [s["tables"][l] for l in range(L - 1)]
    if op == "gin":
        # sums over `degree` neighbours: weights that keep the activations of order one, as normalisation or training would
        q = math.sqrt(1.0 / c["degree"])
        ws = [(glorot(widths[l], c["hidden"], q if l == 0 else 1.5 * q), glorot(c["hidden"], widths[l + 1])) for l in range(L)]
        s["weights"] = ws
    elif op == "pna":
        s["weights"] = [(glorot(2 * widths[l], max(8, widths[l + 1] // 4)),
                         glorot(widths[l] + 9 * max(8, widths[l + 1] // 4), widths[l + 1])) for l in range(L)]
        s["delta"] = float(torch.log(g.deg.double() + 1.0).mean())
    elif op == "gat":
        s["weights"] = [(glorot(widths[l], widths[l + 1]), 0.1 * normal(widths[l + 1]), 0.1 * normal(widths[l + 1]))
                        for l in range(L)]
    else:
        if op == "gcnii":
            s["stack"] = torch.stack([glorot(widths[l], widths[l + 1]) for l in range(L)])     # equal widths: one block
            s["weights"] = [s["stack"][l] for l in range(L)]
        else:
            s["weights"] = [glorot(widths[l], widths[l + 1]) for l in range(L)]
    if op in ("gcn", "gin", "gcnii"):
        w_in = glorot(c["f_in"], c["hidden"]) if op == "gcnii" else None
        s["model"] = executor.Model(op, s["weights"], w_in, ALPHA if op == "gcnii" else 0.0)
    if train:
        k = min(16, c["f_out"])
        labels = torch.randint(0, k, (sg.nb,), generator=gen, device=dev, dtype=torch.int32)
        labels[torch.rand(sg.nb, generator=gen, device=dev) < 0.5] = -1            # half of the nodes carry a label
        s["labels"], s["n_labelled"] = labels, int((labels >= 0).sum())
    return s


def run(s):
    c, bg = s["case"], s["bg"]
    op = c["op"]
    if c["mode"] == FORWARD:
        if op == "pna":
            y = executor.pna_forward_batch(s["weights"], s["delta"], bg, s["x"], s["hist"])
        elif op == "gat":
            y = executor.gat_forward_batch(s["weights"], bg, s["x"], s["hist"], heads=c["heads"])
        else:
            y = executor.forward_batch_fused(s["model"], bg, s["x"], s["hist"])
        return {"y": y, "tables": s["tables"]}
    if op in ("pna", "gat"):
        loss = torch.empty(1, device=s["x"].device)

        def loss_grad(y):
            g = torch.empty_like(y)
            gas.gas_softmax_xent(y, s["labels"], g, torch.empty(bg.nb, device=y.device), loss,
                                 scale=1.0 / max(1, s["n_labelled"]))
            return g
        if op == "pna":
            y, grads, _ = executor.pna_train_batch(s["weights"], s["delta"], bg, s["x"], s["hist"], loss_grad)
        else:
            y, grads, _ = executor.gat_train_batch(s["weights"], bg, s["x"], s["hist"], loss_grad, heads=c["heads"])
        executor.sgd_update(s["weights"], grads, LEARNING_RATE)
        return {"y": y, "loss": loss, "grads": [grads[l] for l in range(c["layers"])], "weights": s["weights"],
                "tables": s["tables"]}
    loss, _, y, grads = executor.train_step(s["model"], bg, s["x"], s["hist"], s["labels"], LEARNING_RATE,
                                            n_labelled=s["n_labelled"], fused=True)
    out = {"y": y, "loss": loss, "tables": s["tables"]}
    if op == "gcnii":            # the projection's gradient has come through every layer; the layers' weights are one block
        out.update(w_in=s["model"].w_in, g_in=grads["w_in"], weights=s["stack"],
                   grads=[grads[l] for l in range(0, c["layers"], 2)])
    else:
        out.update(weights=s["weights"], grads=[grads[l] for l in range(c["layers"])])
        if op == "gin":
            out["eps"] = grads["eps"]
    return out


def exact(case, seed):
    """The outputs, the loss and the pushed tables in 64 bits, with plain torch: Algorithm 1's forward pass over the batch
    from the same inputs.  Gradients and updated weights have no such value that two correct passes are near to: a hidden
    unit within rounding of its threshold takes its whole gradient with it (see `tolerance`)."""
    c, s = case, prepare(case, seed)
    bg, op, L, nb = s["bg"], c["op"], c["layers"], s["bg"].nb
    deg_rows = (bg.rowptr[1:] - bg.rowptr[:-1]).long()
    row = torch.repeat_interleave(torch.arange(nb, device=s["x"].device), deg_rows)
    col, n_id = bg.col.long(), bg.n_id.long()
    tables = s["tables"].double()

    def adjacency(val):
        return torch.sparse_csr_tensor(bg.rowptr.long(), col, val, size=(nb, bg.nv))

    def norm():
        # 1 / sqrt((deg v + 1) (deg w + 1)), degrees of the whole graph; prepare's pattern carries the self-loops
        deg = _graph(c, seed, s["x"].device).deg.double().to(s["x"].device) + 1.0
        q = deg[n_id].rsqrt()
        return q[row] * q[col]

    x = s["x"][n_id].double()
    if op in ("gcn", "gcnii"):
        a = adjacency(norm())
    elif op == "gin":
        a = adjacency(torch.ones_like(col, dtype=torch.float64))
    if op == "gcnii":
        h0 = x = torch.relu(x @ s["model"].w_in.double())
    for l in range(1, L + 1):
        w = s["weights"][l - 1]
        w = [m.double() for m in w] if isinstance(w, tuple) else w.double()
        if op == "gcn":
            y = (a @ x) @ w
        elif op == "gin":
            y = torch.relu((a @ x + x[:nb]) @ w[0]) @ w[1]
        elif op == "gcnii":
            beta = math.log(0.5 / l + 1.0)
            z = (1.0 - ALPHA) * (a @ x) + ALPHA * h0[:nb]
            y = (1.0 - beta) * z + beta * (z @ w)
        elif op == "pna":
            f, f1 = x.shape[1], w[0].shape[1]
            p = x @ w[0][f:]
            own = deg_rows.clamp(min=1)[:, None]
            index = row[:, None].expand(-1, f1)
            zero = torch.zeros(nb, f1, dtype=torch.float64, device=x.device)
            agg = [torch.zeros_like(zero).index_add_(0, row, p[col]) / own,
                   torch.zeros_like(zero).scatter_reduce_(0, index, p[col], "amin", include_self=False),
                   torch.zeros_like(zero).scatter_reduce_(0, index, p[col], "amax", include_self=False)]
            some = (deg_rows > 0)[:, None]
            agg = [torch.where(some, t + x[:nb] @ w[0][:f], zero) for t in agg]
            scale = torch.log(deg_rows.double() + 1.0)[:, None] / s["delta"]
            blocks = agg + [scale * t for t in agg] + [torch.where(some, t / scale, zero) for t in agg]
            y = torch.cat([x[:nb]] + blocks, 1) @ w[1]
        else:
            p, fh = x @ w[0], w[0].shape[1] // c["heads"]
            y = torch.zeros(nb, w[0].shape[1], dtype=torch.float64, device=x.device)
            for h in range(c["heads"]):
                k = slice(h * fh, (h + 1) * fh)
                score = torch.nn.functional.leaky_relu((p[:nb, k] @ w[1][k])[row] + (p[:, k] @ w[2][k])[col], 0.2)
                top = torch.full((nb,), -math.inf, dtype=torch.float64, device=x.device)
                e = torch.exp(score - top.scatter_reduce_(0, row, score, "amax")[row])
                total = torch.zeros(nb, dtype=torch.float64, device=x.device).index_add_(0, row, e)
                y[:, k] = adjacency(e / total[row]) @ p[:, k].contiguous()
        if l < L:
            y = torch.relu(y)
            tables[l - 1, n_id[:nb]] = y
            x = torch.cat([y, tables[l - 1, n_id[nb:]]])
    out = {"y": y, "tables": tables}
    if c["mode"] == TRAIN:
        known = s["labels"] >= 0
        loss = torch.logsumexp(y, 1) - y.gather(1, s["labels"].clamp(min=0).long()[:, None])[:, 0]
        out.update(loss=loss[known].sum()[None], grads=None, weights=None)
    return out
