"""Sequencing of the C-ABI calls for one mini-batch (paper, Algorithm 1).

Nothing is computed here: buffers are torch allocations and every step is a
gas_* call.  For layer l of a batch B with halo V_b \\ B:

    gas_spmm   Z      = aggregation of the mini-batch tensor X over the rows of G_b
    gas_linear Y      = transform(Z)            (gas_mlp2 for GIN), written into rows 0..nb-1 of the next X
    gas_push   H[l]   <- Y   for the in-batch nodes        (not for the last layer)
    gas_pull   X[nb:] <- H[l] for the halo nodes

The first layer's X is a gas_pull of all of V_b from the feature table (exact
inputs); GCNII first applies its graph-agnostic input projection to all rows.
"""
import itertools
import math

import torch

from . import binding as B


class _Kept:
    """An array, the stream that built it and the event after which it is complete."""

    def __init__(self, array, stream):
        self.array, self.stream, self.event, self.complete = array, stream, torch.cuda.Event(), False
        self.event.record(stream)


def plan_limits(rows, entries, longest):
    """Which rows of a pattern are cut into chunks, and how long a chunk is (gas_plan_options).  A wavefront, or a team of its lanes,
    walks a light row's entries, 0.1 us each, and a launch waits for the longest; a chunk's partial sum is written and read
    again, and any heavy row adds two launches.  So the line follows the batch: 256 entries where the whole takes half a
    millisecond and more, 64 where it takes 20 to 200 us, but no less than twice the mean (rows of like lengths hide each other's
    walks), and none where the longest row is hardly longer than that or its walk is short beside the launch.  Many rows hide a
    walk: from 131,072 rows of a middling batch 256, and from 262,144 the plan's own 512 and 256.  us, rows above
    512 by 256 entries and so, aggregations of power-law batches (and their adjoints), 256 floats, 64 floats, 256 bf16:
    - 250,000 rows of 40: 1,223 -> 1,192 (565 -> 553), 459 -> 417 (259 -> 245), 704 -> 659 (329 -> 321);
    - 15,000 rows of 43: 143 -> 83 (53 -> 41), 105 -> 43 (60 -> 33), 125 -> 53 (59 -> 38);
    - 3,750 rows of 24, the longest 269: 34 -> 29, 33 -> 22, 33 -> 25; by chunks of 128 50, 43, 49;
    - 25,000 rows of 18, the longest 141: whole 64, with 64 the line 75.
    Forward passes of two layers, 240 bf16, line and chunk: 37,000 rows of 47, whole rows 378, 256 and 128 304, 128 and 128 290, 64
    and 64 284; 100,000 rows of 43 756, 674, 654, 657; 350,000 rows of 68 2,915, 2,914, 2,917, 2,984; 117,000 rows of 17, the longest
    290, 414, 448, 446, 431.  Of three layers, 256 bf16 (256 floats), 128 and 64, 256 and 128, 512 and 256: 293,000 rows of 15 1,185, 1,160, 1,185
    (2,325, 2,299, 2,320), of 23 1,604, 1,555, 1,529 (3,092, 3,090, 3,083), of 31 1,980, 1,904, 1,852 (3,706, 3,696, 3,710), 391,000 rows of 20
    1,901, 1,853, 1,824; 195,000 rows of 26 1,276, 1,224, 1,239 (2,373, 2,369, 2,382), of 36 1,570, 1,500, 1,506 (2,837, 2,822, 2,891); 146,000
    of 28 1,018, 978, 1,039 (1,852, 1,851, 1,910); 98,000 of 45 1,055, 1,017, 1,038 (1,831, 1,840, 1,886)."""
    if rows == 0:
        return None
    size, chunk = (256, 128) if entries >= 10_000_000 else (128, 64) if entries >= 3_000_000 else (64, 64 if entries >= 200_000 else 32)
    if 3_000_000 <= entries < 10_000_000 and rows >= 131_072:
        size, chunk = (512, 256) if rows >= 262_144 else (256, 128)
    line = min(512, max(size, -(-2 * entries // rows)))
    if longest <= min(512, line + 144 + entries // 6000):
        return None
    return dict(heavy_threshold=line, chunk=chunk)


def _windowed(limits, max_F):
    """plan_limits with windows of 16 MiB of rows of max_F, at most 256 (a wide input layer's plan serves the layers behind it too), floats
    where chunks are short: a window of the plan's own 2 MiB cuts more of them, whose partial sums cost more than the reuse
    saves.  us of three layers forward with 2 and with 16 MiB, 256 bf16 (256 floats): 600,000 rows of 83 8,800 and 8,471 (13,793 and
    13,846), 200,000 of 86 3,222 and 3,114 (5,173 and 5,153), 117,000 of 109 2,483 and 2,392 (3,920 and 3,890), 37,500 of 190 1,320
    and 1,264 (1,815 and 1,854)."""
    if limits is None or limits["chunk"] > 128:
        return limits
    return dict(limits, window_rows=min(1 << 20, (16 << 20) // (4 * min(max_F, 256))))


class BatchGraph:
    """Device-side index structure of one batch subgraph plus its plans."""

    def __init__(self, nb, n_id, rowptr, col, deg=None, colptr=None, row=None, max_F=256, normalise=True, timed=False,
                 plan_options=None, csc_pos=None):
        """timed: wait for the device after each part of the per-batch set-up and keep its wall time in
        self.setup_ms (plans, coefficients, fused source indices); the benchmark reports it.
        plan_options: of all of the batch's plans (gas_plan_options).  A dict is taken as it is: a field that it doesn't
        name, and all of them in an empty one, has the library's default.  None: what suits the batch (plan_limits)."""
        import time
        self.setup_ms = {}

        def part(name, fn):
            if not timed:
                return fn()
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            out = fn()
            torch.cuda.synchronize()
            self.setup_ms[name] = round((time.perf_counter() - t0) * 1e3, 3)
            return out

        self._max_F, self._plan_options = max_F, plan_options
        self.nb, self.nv = int(nb), int(n_id.numel())
        self.n_id, self.rowptr, self.col = n_id, rowptr, col
        self.nnz = int(col.numel())
        self.max_row = int((rowptr[1:] - rowptr[:-1]).max().item()) if self.nb > 0 else 0
        self.plan = part("plan_csr", lambda: B.gas_plan_create(rowptr, self.nnz, max_F, ind=col,
                                                               options=self._options(self.nb, self.nnz, self.max_row)))
        self.val = None
        if normalise:
            self.val = torch.empty(self.nnz, dtype=torch.float32, device=col.device)
            part("gcn_norm_csr", lambda: B.gas_gcn_norm(rowptr, col, n_id, deg, self.val))
        self._src = self._src_first = self._groups = None
        self.csc_pos = csc_pos       # int32[nnz]: position of every CSC entry in the CSR arrays (PNA / GAT backward)
        self._n_id_host = None
        self._plan_t_all = None
        self.colptr, self.row, self.val_t, self.plan_t = colptr, row, None, None
        self.nnz_t, self.max_col = 0, 0          # entries of the in-batch columns, and of the longest of them
        if colptr is not None:
            # backward over the in-batch columns only: histories are constants
            if self.nb > 0:
                longest = (colptr[1:self.nb + 1] - colptr[:self.nb]).max()
                self.max_col, self.nnz_t = torch.stack((longest, colptr[self.nb])).tolist()    # one read-back
            self.plan_t = part("plan_csc", lambda: B.gas_plan_create(colptr[: self.nb + 1], self.nnz_t, max_F, n_rows=self.nb, ind=row,
                                                                     options=self._options(self.nb, self.nnz_t, self.max_col)))
            if normalise:
                self.val_t = torch.empty(self.nnz, dtype=torch.float32, device=col.device)
                part("gcn_norm_csc", lambda: B.gas_gcn_norm(colptr, row, n_id, deg, self.val_t))
        if timed:
            part("fuse_sources", lambda: self.src)
            self.setup_ms["total"] = round(sum(self.setup_ms.values()), 3)

    def _options(self, rows, entries, longest):
        if self._plan_options is not None:
            return self._plan_options
        return _windowed(plan_limits(rows, entries, longest), self._max_F)

    @property
    def plan_t_all(self):
        """Plan of the backward aggregation over ALL columns, halo included (GCNII's first layer: the gradient of
        the projected features of every node of V_b); built on first use, once per batch."""
        if self._plan_t_all is None:
            self._max_col_all = int((self.colptr[1:] - self.colptr[:-1]).max().item()) if self.nv > 0 else 0
            self._plan_t_all = B.gas_plan_create(self.colptr, self.nnz, self._max_F, ind=self.row,
                                                 options=self._options(self.nv, self.nnz, self._max_col_all))
        return self._plan_t_all

    @property
    def max_col_all(self):
        """Entries of the longest of all columns, halo included."""
        self.plan_t_all
        return self._max_col_all

    def _once(self, name, build):
        """self.<name>, an array of this batch that `build` makes on first use, without a wait of the host: streams other than the
        one that built it wait for it there.  While a graph is captured an array that is not known to be complete is built
        again, as a part of the graph, and not kept: it has no contents before the graph has run."""
        kept = getattr(self, name)
        if kept is not None and kept.complete:
            return kept.array
        if torch.cuda.is_current_stream_capturing():
            return build()
        cur = torch.cuda.current_stream()
        if kept is None:
            kept = _Kept(build(), cur)
            setattr(self, name, kept)          # another thread may have been here: the contents are the same
        else:
            kept.complete = kept.event.query()
            if not kept.complete and kept.stream != cur:
                cur.wait_event(kept.event)
        return kept.array

    @property
    def groups(self):
        """The in-batch rows by degree (gas_pna_groups; max_row is the largest), built on first use, once per batch."""
        return self._once("_groups", lambda: B.gas_pna_groups(self.rowptr, self.max_row))

    @property
    def n_id_host(self):
        """The node ids in host memory (index lists of tables on disk are read by host threads)."""
        if self._n_id_host is None:
            self._n_id_host = self.n_id.cpu()
        return self._n_id_host

    def _sources(self, nb):
        src = torch.empty_like(self.col)
        B.gas_fuse_sources(self.col, nb, self.n_id, src)
        return src

    @property
    def src(self):
        """Source indices for gas_spmm_hist (built on first use, once per batch)."""
        if self._src is None:
            self._src = self._sources(self.nb)
        return self._src

    @property
    def src_first(self):
        """Source indices of a first layer that reads the feature table in place (gas_spmm_table: GCN, and GIN without
        gradients), built on first use, once per batch; under capture as a part of the graph, and not kept: they have no
        contents before the graph has run."""
        first = self._src_first
        if first is None:
            first = self._sources(0)
            if not torch.cuda.is_current_stream_capturing():
                self._src_first = first
        return first


class Model:
    def __init__(self, op, weights, w_in=None, alpha=0.0, gin_eps=0.0):
        self.op, self.weights, self.w_in, self.alpha, self.gin_eps = op, weights, w_in, alpha, gin_eps

    @property
    def n_layers(self):
        return len(self.weights)

    def out_width(self, l):
        w = self.weights[l]
        return (w[1] if self.op == "gin" else w).shape[1]


# Rows longer than this keep the two-kernel form, whose plan splits them over wavefronts; the one-launch layer
# gives a row to one team of lanes (backward: _back_in_one_launch).
ONE_LAUNCH_MAX_ROW = 512


def _back_in_one_launch(width, rows, entries, longest) -> bool:
    """Whether the adjoint of the aggregation and the input gradient below it, `width` columns wide, are one launch
    (gas_spmm_t_relu_linear) and not two (gas_spmm_t_relu by its plan, gas_linear_bwd_input_add).  `rows` in-batch nodes,
    `entries` of the pattern, `longest` of one of them.  One team of lanes walks a row's entries, 0.09 us each, and the
    eight teams of a wavefront wait for the longest; the plan spreads a long row.  us, one launch and two:
    - short rows: 512 rows of up to 30 entries, 32 -> 32 columns, 5.5 and 7.1, 21,248 8.1 and 15.2; 10,000 of up to 40
      7.3 and 10.4;
    - few rows, where the host bounds a pass and a launch more is 10 us of its time: 512 rows of up to 60 8.4 and 7.8;
    - longer ones of like lengths where many rows hide them: 10,000 rows of up to 100 13.2 and 14.1, 21,248 of up to 200
      31.8 and 38.8; but 512 rows of up to 100 11.4 and 8.9;
    - power-law lengths up to 500 where rows have few entries (21,248 rows of 2.4 0.76-1.0 of the time, of 7.4 1.2-1.6);
    - 64 columns, 256-byte rows, up to 8,192 rows of any lengths up to ONE_LAUNCH_MAX_ROW: 5,000 rows of up to 100 14.9
      and 25.2, power law 0.8-1.0 of the time (21,248 rows 1.0-1.2);
    - more than 64 columns double the lanes of a row and halve the rows in flight: 21,248 rows of up to 30, 80 -> 80, 26.1
      and 30.8, 96 -> 96 28.6 and 28.8, of up to 60 39.3 and 40.4, 41.9 and 38.6, of up to 100 56.9 and 54.8.  128 columns,
      512-byte rows, have the better plan: 5,000 rows of up to 20 11.7 and 12.0, 8,192 12.6 and 12.8, 10,000 17.5 and 15.1,
      21,248 27.4 and 23.0."""
    if longest > ONE_LAUNCH_MAX_ROW:
        return False
    if longest <= (64 if rows <= 4096 else 48 if width <= 64 else 32):
        return width < 128 or rows <= 8192
    if width > 64:
        return False
    alike = longest * rows <= 4 * entries
    return (width == 64 and rows <= 8192) or (alike and 100 * longest <= rows) or (rows >= 16384 and entries <= 4 * rows)


def _layers_together(model: Model, bg, h0) -> bool:
    """Whether GCNII's layers (all of one width) go in groups by one call (gas_spmm_linear_layers): narrow fp32 layers without long
    rows, of few rows.  A layer takes the host 14 us by a call of its own and 7 in a group of four or eight.  16 layers of 64, one by one and in
    groups: 500 rows 245 and 143 us, 5,000 244 and 151, 12,500 246 and 208, 16,000 246 and 224; 21,248 287 and 289, where the card
    takes longer than either and a pass that starts on an idle one waits 14 us for its first groups."""
    return B.spmm_linear_supported(h0, h0.shape[1]) and bg.max_row <= ONE_LAUNCH_MAX_ROW and model.n_layers >= 2 and 0 < bg.nb <= 16384


def _layer_groups(count, most=8):
    """Ranges of layers that go in one call: 2, 2, 4 and then `most`: the card has work in hand while the host puts the next, larger
    call together."""
    first = 0
    while first < count:
        end = min(count, first + max(2, min(most, first)))
        yield range(first, end)
        first = end


def _forward_layers(model: Model, bg, h0, histories, ids, betas, ys, zs):
    """GCNII's layers by gas_spmm_linear_layers: layer l into ys[l], its aggregated rows into zs[l] (None: not kept); ids None:
    no Push."""
    L = model.n_layers
    tables, pushed = [None] + list(histories[:L - 1]), list(histories[:L - 1]) + [None]
    for g in _layer_groups(L):
        a, b = g.start, g.stop
        B.gas_spmm_linear_layers(bg.rowptr, bg.col if a == 0 else bg.src, bg.src, bg.val, h0 if a == 0 else ys[a - 1], model.weights[a:b],
                                 ys[a:b], tables[a:b], s_agg=1.0 - model.alpha, r=h0, s_res=model.alpha,
                                 c_identity=[1.0 - x for x in betas[a:b]], c_weight=betas[a:b], relu_last=b < L,
                                 z_outs=None if zs is None else zs[a:b], push_idx=ids, push_hists=None if ids is None else pushed[a:b])


def _mlp_in_two(z, w1, w2) -> bool:
    """Whether GIN's MLP is faster as two products with the hidden activation stored between them, which run on bf16 parts
    (csrc/split.h) where the fused fp32 kernel uses the fp32 instruction on 32 rows a workgroup: 4,000 rows of
    256 -> 256 -> 256 19 us against 33 fused, 64 -> 64 -> 64 11 against 13.  Narrow layers of few rows save a launch by the fused kernel: up to three
    steps of 32 of the two reduced widths, 32 output columns and a workgroup for every compute unit (4,000 rows: 32 -> 32 -> 32 8 us
    fused, 11 in two, 64 -> 32 -> 32 9.7 and 10.8; 128 -> 32 -> 32 12.7 and 10.9, 24,000 rows of 32 -> 32 -> 32 16.5 and 10.7).
    bf16 has fused kernels of its own."""
    if z.dtype != torch.float32:
        return False
    steps = -(-z.shape[1] // 32) + -(-w1.shape[1] // 32)
    return not (z.shape[0] <= 8192 and steps <= 3 and w2.shape[1] <= 32)


def _matrices(rows, widths, dtype, device):
    """A matrix of `rows` rows for every width.  Four or more of one width in a row share an allocation, each on a 512-byte boundary
    as if it had its own: a deep narrow model's pass has hundreds of matrices, and its launches are shorter than what
    allocating and slicing them one by one takes (2 us each)."""
    if len(widths) < 4:
        return [torch.empty((rows, width), dtype=dtype, device=device) for width in widths]
    out, size = [], torch.finfo(dtype).bits // 8
    for width, run in itertools.groupby(widths):
        n = len(list(run))
        if n < 4:
            out += [torch.empty((rows, width), dtype=dtype, device=device) for _ in range(n)]
            continue
        stride = -(-rows * width * size // 512) * (512 // size)
        out += torch.empty(n * stride, dtype=dtype, device=device).as_strided((n, rows, width), (stride, width, 1)).unbind(0)
    return out


class _WeightGrads:
    """The weight gradients of a backward pass.  Small ones wait for each other and share launches
    (gas_linear_bwd_weights): 21,248 rows of 64 x 64, 64 layers, 12 us each alone and 4 together.  A gradient matrix of
    more than 16 MB fills the chip by itself and is not kept waiting (it would only hold memory); bf16 has kernels
    of its own."""
    LARGEST, TOGETHER = 16 << 20, 16

    def __init__(self):
        self.waiting = []

    def add(self, z, g, dw=None, c=1.0):
        """dW = c * z^T g, complete after done()."""
        if dw is None:
            dw = torch.empty((z.shape[1], g.shape[1]), dtype=torch.float32, device=z.device)
        if z.dtype == torch.float32 and 4 * g.numel() <= self.LARGEST:
            self.waiting.append((z, g, dw, c))
            if len(self.waiting) == self.TOGETHER:
                self.done()
            return dw
        ws = torch.empty(max(1, B.gas_linear_bwd_weight_workspace(z.shape[0], z.shape[1], g.shape[1])),
                         dtype=torch.uint8, device=z.device)
        B.gas_linear_bwd_weight(z, g, dw, ws, c_weight=c)
        return dw

    def done(self):
        B.gas_linear_bwd_weights(self.waiting)
        self.waiting = []


def _pushes(do_push, table) -> bool:
    """Whether a training pass of GCN or GCNII, or a pass of PNA, lets the transform store its rows to the history table as well, and of
    GAT the aggregation: not to host memory, which gas_push_host writes with few workgroups.  (The other forward passes and GIN push from the transform
    there too: the link bounds both, 20,000 rows of 128 floats 199 us in one and 205 us in two, 50,000 of 256 981 and 982.)"""
    return do_push and not isinstance(table, B.HostTable)


def gcnii_beta(layer: int) -> float:
    return math.log(0.5 / layer + 1.0)


def forward_batch_fused(model: Model, bg: BatchGraph, x_feat, histories, do_push=True):
    """Same result as forward_batch, with the halo rows read in place by the
    aggregation (gas_spmm_hist) instead of being pulled into the mini-batch
    tensor, and the Push taken in the transform's epilogue: per layer
    aggregate(X_batch, H[l-1]) -> transform, rows stored to H[l] as well.
    Layer 1 reads all its rows from the feature table in place (gas_spmm_table: no copy of the in-batch rows; 5,000 rows of
    1,433 floats 22 us, of 512 rows a launch of three).  Copy and aggregation took 1.07 to 1.5 times as long in all of 520 cases
    (GCN and GIN, 500 to 75,000 rows of 6 to 45 entries, clustered and power law, 40 to 1,433 columns of both types, with and without
    the rows in the caches), the least with 75,000 power-law rows out of the caches: 212 and 194 us for 100 floats.  GCNII: its first layer aggregates the
    projected features of all of V_b, which no table holds, so that layer gathers from the mini-batch tensor; from
    layer 2 on the halo rows come from the history tables in place.  Narrow fp32 layers of GCN and GCNII (widths
    up to 128, no row above ONE_LAUNCH_MAX_ROW entries) take one launch each (gas_spmm_linear)."""
    dev, dt = x_feat.device, x_feat.dtype
    nb = bg.nb
    if model.op == "gcnii":
        return _forward_gcnii_fused(model, bg, x_feat, histories, do_push)
    ids = bg.n_id[:nb]
    x = x_feat
    L = model.n_layers
    y = None
    for l in range(1, L + 1):
        last = l == L
        table = x_feat if l == 1 else histories[l - 2]
        y = torch.empty((nb, model.out_width(l - 1)), dtype=dt, device=dev)
        push = not last and do_push          # the transform stores its rows to the next history table as well
        if model.op == "gcn" and B.spmm_linear_supported(x, y.shape[1]) and bg.max_row <= ONE_LAUNCH_MAX_ROW:
            # narrow layers: aggregation, transform and Push in one launch
            B.gas_spmm_linear(bg.rowptr, bg.src_first if l == 1 else bg.src, bg.val, x, model.weights[l - 1], y, hist=table,
                              relu=not last, push_idx=ids if push else None, push_hist=histories[l - 1] if push else None)
            x = y
            continue
        z = torch.empty((nb, x.shape[1]), dtype=dt, device=dev)
        if l == 1:
            B.gas_spmm_table(bg.plan, bg.rowptr, bg.src_first, bg.val if model.op == "gcn" else None, table, z,
                             diag=0.0 if model.op == "gcn" else 1.0 + model.gin_eps, own=bg.n_id)
        elif model.op == "gcn":
            B.gas_spmm_hist(bg.plan, bg.rowptr, bg.src, bg.val, x, table, z)
        else:
            B.gas_spmm_hist(bg.plan, bg.rowptr, bg.src, None, x, table, z, diag=1.0 + model.gin_eps)
        if model.op == "gcn":
            if push:
                B.gas_linear_push(z, model.weights[l - 1], y, ids, histories[l - 1], relu=True)
            else:
                B.gas_linear(z, model.weights[l - 1], y, relu=not last)
        else:
            w1, w2 = model.weights[l - 1]
            if _mlp_in_two(z, w1, w2):
                h = torch.empty((nb, w1.shape[1]), dtype=dt, device=dev)
                B.gas_mlp2_keep(z, w1, w2, y, h, idx=ids if push else None,
                                hist=histories[l - 1] if push else None, relu_out=not last)
            elif push:
                B.gas_mlp2_push(z, w1, w2, y, ids, histories[l - 1], relu_out=True)
            else:
                B.gas_mlp2(z, w1, w2, y, relu_out=not last)
        x = y
    return y


def _forward_gcnii_fused(model: Model, bg: BatchGraph, x_feat, histories, do_push):
    dev, dt = x_feat.device, x_feat.dtype
    nb, nv = bg.nb, bg.nv
    ids = bg.n_id[:nb]
    x0 = torch.empty((nv, x_feat.shape[1]), dtype=dt, device=dev)
    B.gas_pull(x_feat, bg.n_id, x0)
    h0 = torch.empty((nv, model.w_in.shape[1]), dtype=dt, device=dev)
    B.gas_linear(x0, model.w_in, h0, relu=True)
    x, y = h0, None
    L = model.n_layers
    if _layers_together(model, bg, h0):
        y = torch.empty((nb, h0.shape[1]), dtype=dt, device=dev)
        turns = [torch.empty_like(y) for _ in range(min(2, L - 1))]
        _forward_layers(model, bg, h0, histories, ids if do_push else None, [gcnii_beta(l) for l in range(1, L + 1)],
                        [turns[l % 2] for l in range(L - 1)] + [y], None)
        return y
    for l in range(1, L + 1):
        last = l == L
        y = torch.empty((nb, model.out_width(l - 1)), dtype=dt, device=dev)
        beta = gcnii_beta(l)
        push = not last and do_push
        if B.spmm_linear_supported(x, y.shape[1]) and bg.max_row <= ONE_LAUNCH_MAX_ROW:
            # narrow layers: aggregation, transform and Push in one launch
            B.gas_spmm_linear(bg.rowptr, bg.col if l == 1 else bg.src, bg.val, x, model.weights[l - 1], y,
                              hist=None if l == 1 else histories[l - 2], s_agg=1.0 - model.alpha, r=h0,
                              s_res=model.alpha, c_identity=1.0 - beta, c_weight=beta, relu=not last,
                              push_idx=ids if push else None, push_hist=histories[l - 1] if push else None)
            x = y
            continue
        z = torch.empty((nb, h0.shape[1]), dtype=dt, device=dev)
        if l == 1:
            B.gas_spmm(bg.plan, bg.rowptr, bg.col, bg.val, x, z, s_agg=1.0 - model.alpha, r=h0, s_res=model.alpha)
        else:
            B.gas_spmm_hist(bg.plan, bg.rowptr, bg.src, bg.val, x, histories[l - 2], z, s_agg=1.0 - model.alpha, r=h0,
                            s_res=model.alpha)
        if push:
            B.gas_linear_push(z, model.weights[l - 1], y, ids, histories[l - 1], c_identity=1.0 - beta,
                              c_weight=beta, relu=True)
        else:
            B.gas_linear(z, model.weights[l - 1], y, c_identity=1.0 - beta, c_weight=beta, relu=not last)
        x = y
    return y


def _aggregate_transform(model: Model, l, bg: BatchGraph, x, h0, z, y):
    """Layer l (1-based) on the mini-batch tensor x: aggregation into z, transform into y (ReLU unless last)."""
    last = l == model.n_layers
    if model.op == "gcn":
        B.gas_spmm(bg.plan, bg.rowptr, bg.col, bg.val, x, z)
        B.gas_linear(z, model.weights[l - 1], y, relu=not last)
    elif model.op == "gin":
        B.gas_spmm(bg.plan, bg.rowptr, bg.col, None, x, z, diag=1.0 + model.gin_eps)
        w1, w2 = model.weights[l - 1]
        B.gas_mlp2(z, w1, w2, y, relu_out=not last)
    elif model.op == "gcnii":
        B.gas_spmm(bg.plan, bg.rowptr, bg.col, bg.val, x, z, s_agg=1.0 - model.alpha, r=h0, s_res=model.alpha)
        beta = gcnii_beta(l)
        B.gas_linear(z, model.weights[l - 1], y, c_identity=1.0 - beta, c_weight=beta, relu=not last)
    else:
        raise ValueError(model.op)


def forward_batch(model: Model, bg: BatchGraph, x_feat, histories, do_push=True, keep_layers=False):
    """Run all layers for one batch.  Returns the last layer's [nb, F] output
    (and the list of mini-batch tensors if keep_layers)."""
    dev, dt = x_feat.device, x_feat.dtype
    nb, nv = bg.nb, bg.nv
    x = torch.empty((nv, x_feat.shape[1]), dtype=dt, device=dev)
    B.gas_pull(x_feat, bg.n_id, x)
    h0 = None
    if model.op == "gcnii":
        h0 = torch.empty((nv, model.w_in.shape[1]), dtype=dt, device=dev)
        B.gas_linear(x, model.w_in, h0, relu=True)
        x = h0
    layers = []
    L = model.n_layers
    y = None
    for l in range(1, L + 1):
        last = l == L
        f_in, f_out = x.shape[1], model.out_width(l - 1)
        z = torch.empty((nb, f_in), dtype=dt, device=dev)
        if last:
            y = torch.empty((nb, f_out), dtype=dt, device=dev)
        else:
            x_next = torch.empty((nv, f_out), dtype=dt, device=dev)
            y = x_next[:nb]
        _aggregate_transform(model, l, bg, x, h0, z, y)
        if last:
            break
        if do_push:
            B.gas_push(y, bg.n_id[:nb], histories[l - 1])
        if nv > nb:
            B.gas_pull(histories[l - 1], bg.n_id[nb:], x_next[nb:])
        x = x_next
        if keep_layers:
            layers.append(x)
    return (y, layers) if keep_layers else y


class HostPipeline:
    """Streams for histories kept in host memory (Section 5 "PyGAS" of the paper: history access runs beside the
    computation).  One stream carries the pulls, one the pushes, both at the default priority.  The mini-batch
    tensors the transfers touch belong to the pipeline: two sets, used by alternate batches, so that a batch can
    compute while the pushes of the one before still read its tensors.  Events: `table_pushed[l]`, the end of the
    last push into table l (a later pull from that table waits for it); `set_pushed[i]` / `set_read[i]`, the end
    of the pushes / of the computation that last read set i (the next writers of that set wait for them)."""

    def __init__(self, device):
        self.pull = torch.cuda.Stream(device)
        self.push = torch.cuda.Stream(device)
        self.turn = 0
        self.table_pushed = {}
        self.set_pushed = [None, None]
        self.set_read = [None, None]
        self._buffers = {}
        self._fresh = False

    def buffer(self, l, rows, width, dtype, device):
        """The mini-batch tensor of the current set that layer l writes and layer l + 1 reads; grown when a
        batch needs more rows."""
        key = (self.turn, l, width, dtype)
        t = self._buffers.get(key)
        if t is None or t.shape[0] < rows:
            if t is not None:                    # the transfer streams may still be using the old tensor
                t.record_stream(self.pull)
                t.record_stream(self.push)
            t = self._buffers[key] = torch.empty((rows, width), dtype=dtype, device=device)
            self._fresh = True                   # memory the compute stream may still be using
        return t[:rows]

    def join(self):
        """Make the current stream wait for every transfer issued so far."""
        cur = torch.cuda.current_stream()
        cur.wait_stream(self.pull)
        cur.wait_stream(self.push)


def forward_batch_host(model: Model, bg: BatchGraph, x_feat, histories, pipe: HostPipeline, do_push=True):
    """forward_batch for history tables in pinned host memory (binding.HostTable), with the transfers taken off
    the compute stream: the halo rows of every layer are pulled ahead on pipe.pull (they were pushed by earlier
    batches, so none depends on this batch's computation) and each layer's output is pushed on pipe.push while
    the next layer computes.  A layer waits only for its own halo rows, a pull only for the earlier pushes into
    its own table.  Same bits as forward_batch: in-batch and halo rows of a table are disjoint, so the order of
    this batch's pushes and pulls is immaterial (Algorithm 1).  The caller calls pipe.join() before it reads the
    tables or uses them outside this function."""
    dev, dt = x_feat.device, x_feat.dtype
    nb, nv = bg.nb, bg.nv
    L = model.n_layers
    cur = torch.cuda.current_stream()
    turn = pipe.turn = pipe.turn ^ 1
    pipe._fresh = False
    xs = [None] + [pipe.buffer(l, nv, model.out_width(l - 1), dt, dev) for l in range(1, L)]
    pulled = [None] * L
    if nv > nb:
        with torch.cuda.stream(pipe.pull):
            if pipe._fresh or pipe.set_read[turn] is None:
                pipe.pull.wait_stream(cur)
            else:
                pipe.pull.wait_event(pipe.set_read[turn])
            for l in range(1, L):
                if l - 1 in pipe.table_pushed:
                    pipe.pull.wait_event(pipe.table_pushed[l - 1])
                B.gas_pull(histories[l - 1], bg.n_id[nb:], xs[l][nb:])
                pulled[l] = torch.cuda.Event()
                pulled[l].record(pipe.pull)
    if pipe.set_pushed[turn] is not None:
        cur.wait_event(pipe.set_pushed[turn])    # pushes that still read the rows the layers overwrite
    x = torch.empty((nv, x_feat.shape[1]), dtype=dt, device=dev)
    B.gas_pull(x_feat, bg.n_id, x)
    h0 = None
    if model.op == "gcnii":
        h0 = torch.empty((nv, model.w_in.shape[1]), dtype=dt, device=dev)
        B.gas_linear(x, model.w_in, h0, relu=True)
        x = h0
    y = None
    for l in range(1, L + 1):
        last = l == L
        z = torch.empty((nb, x.shape[1]), dtype=dt, device=dev)
        y = torch.empty((nb, model.out_width(l - 1)), dtype=dt, device=dev) if last else xs[l][:nb]
        if l > 1 and pulled[l - 1] is not None:
            cur.wait_event(pulled[l - 1])
        _aggregate_transform(model, l, bg, x, h0, z, y)
        if last:
            break
        if do_push:
            done = torch.cuda.Event()
            done.record(cur)
            with torch.cuda.stream(pipe.push):
                pipe.push.wait_event(done)
                B.gas_push(y, bg.n_id[:nb], histories[l - 1])
                pipe.table_pushed[l - 1] = torch.cuda.Event()
                pipe.table_pushed[l - 1].record(pipe.push)
        x = xs[l]
    pipe.set_read[turn] = torch.cuda.Event()
    pipe.set_read[turn].record(cur)
    if do_push and L > 1:
        pipe.set_pushed[turn] = pipe.table_pushed[L - 2]
    return y


class DiskPipeline:
    """Mini-batch tensors for histories kept on disk (binding.DiskTable): two sets, used by alternate batches, so
    that a batch can compute while the pushes of the one before still read its tensors; `pushing[i]` lists the
    (table, ticket) pairs of the pushes that read set i."""

    def __init__(self):
        self.turn = 0
        self.pushing = [[], []]
        self._buffers = {}

    def buffer(self, l, rows, width, dtype, device):
        key = (self.turn, l, width, dtype)
        t = self._buffers.get(key)
        if t is None or t.shape[0] < rows:
            t = self._buffers[key] = torch.empty((rows, width), dtype=dtype, device=device)
        return t[:rows]

    def settle(self, turn):
        """Wait for the pushes that still read the tensors of set `turn`."""
        for table, ticket in self.pushing[turn]:
            table.wait(ticket)
        self.pushing[turn] = []

    def join(self):
        self.settle(0)
        self.settle(1)


def forward_batch_disk(model: Model, bg: BatchGraph, x_feat, tables, pipe: DiskPipeline, do_push=True):
    """forward_batch for history tables on disk (the tier the paper's "Conclusion and Future Work" names; transfer
    scheme of its Section 5 "PyGAS").  The halo rows of every layer are requested at the start of the batch (they
    were pushed by earlier batches; each table runs its transfers in the order queued, so a pull sees the pushes
    queued before it), a layer waits for its own halo rows only, and each layer's output goes to its table while
    the next layer computes.  Same bits as forward_batch.  The caller calls pipe.join() before it reads the tables."""
    dev, dt = x_feat.device, x_feat.dtype
    nb, nv = bg.nb, bg.nv
    L = model.n_layers
    turn = pipe.turn = pipe.turn ^ 1
    pipe.settle(turn)
    ids = bg.n_id_host
    xs = [None] + [pipe.buffer(l, nv, model.out_width(l - 1), dt, dev) for l in range(1, L)]
    pulled = [None] * L
    if nv > nb:
        # the transfer starts after the work queued so far, which includes the last readers of this set
        for l in range(1, L):
            pulled[l] = tables[l - 1].pull(ids[nb:], xs[l][nb:])
    x = torch.empty((nv, x_feat.shape[1]), dtype=dt, device=dev)
    B.gas_pull(x_feat, bg.n_id, x)
    h0 = None
    if model.op == "gcnii":
        h0 = torch.empty((nv, model.w_in.shape[1]), dtype=dt, device=dev)
        B.gas_linear(x, model.w_in, h0, relu=True)
        x = h0
    y = None
    for l in range(1, L + 1):
        last = l == L
        z = torch.empty((nb, x.shape[1]), dtype=dt, device=dev)
        y = torch.empty((nb, model.out_width(l - 1)), dtype=dt, device=dev) if last else xs[l][:nb]
        if l > 1 and pulled[l - 1] is not None:
            tables[l - 2].wait(pulled[l - 1])
        _aggregate_transform(model, l, bg, x, h0, z, y)
        if last:
            break
        if do_push:
            pipe.pushing[turn].append((tables[l - 1], tables[l - 1].push(y, ids[:nb])))
        x = xs[l]
    return y


def train_batch(model: Model, bg: BatchGraph, x_feat, histories, grad_out, do_push=True, fused=False):
    """Forward with the activations kept, then the backward pass through all layers (no optimiser step).
    Historical embeddings are constants, so gradients travel along in-batch rows only; GCNII's input projection
    is computed in-graph for the halo rows too and its gradient includes them.  GIN's MLP stores its hidden
    activation here (gas_mlp2_keep: the backward pass reads it again).  Returns (Y_L, grads, kept) with
    grads[l] = dW_l (float32; a pair for GIN), grads["w_in"] for GCNII, and kept = the stored activations the
    backward pass read (x0, h0, per layer (Z, hidden, Y)).  Y_L owns its memory; kept activations of one width share an
    allocation (_matrices), so keeping one of them keeps those, and the weight gradients of a model of one width share one of
    the size of its weights (64 layers of 64 x 64: 1 MB; one by one they took 1.4 us of host time each).  grad_out is
    dLoss/dY_L [nb, F_L], or a function that returns it given Y_L.  fused: the forward aggregations read their
    halo rows from the feature table / the history tables in place (gas_spmm_hist) and nothing is pulled; same
    bits.  GCNII's first layer gathers the projected features from the mini-batch tensor, its later layers from
    the histories.  Narrow fp32 layers of GCN and GCNII then take one launch each (gas_spmm_linear with Z kept;
    the row sums are taken in another order, so these agree with the other form to rounding, not bit for bit).  Every step is a gas_* call."""
    return _train_batch(model, bg, x_feat, histories, grad_out, do_push, fused, keep_input=True)


def _train_batch(model: Model, bg: BatchGraph, x_feat, histories, grad_out, do_push, fused, keep_input):
    """train_batch; keep_input False: a fused GCN, whose backward pass does not read its input, aggregates the feature
    table in place and returns no x0."""
    dev, dt = x_feat.device, x_feat.dtype
    nb, nv = bg.nb, bg.nv
    all_rows = not fused or model.op == "gcnii"      # GCNII projects the features of every node of V_b
    in_place = fused and model.op == "gcn" and not keep_input
    x0 = None
    if not in_place:
        x0 = torch.empty((nv if all_rows else nb, x_feat.shape[1]), dtype=dt, device=dev)
        B.gas_pull(x_feat, bg.n_id if all_rows else bg.n_id[:nb], x0)
    x, h0 = x_feat if in_place else x0, None
    if model.op == "gcnii":
        h0 = torch.empty((nv, model.w_in.shape[1]), dtype=dt, device=dev)
        B.gas_linear(x0, model.w_in, h0, relu=True)
        x = h0
    L = model.n_layers
    saved = []
    y = None
    ids = bg.n_id[:nb]
    widths = [model.out_width(l) for l in range(L)]
    ins = [x.shape[1]] + widths[:-1]
    zs = _matrices(nb, ins, dt, dev)
    # whole mini-batch tensors where the halo rows are pulled into them
    ys = _matrices(nb if fused else nv, widths[:-1], dt, dev) + [torch.empty((nb, widths[-1]), dtype=dt, device=dev)]
    betas = [gcnii_beta(l) for l in range(1, L + 1)] if model.op == "gcnii" else [1.0] * L
    short_rows = fused and model.op in ("gcn", "gcnii") and bg.max_row <= ONE_LAUNCH_MAX_ROW
    together = fused and model.op == "gcnii" and _layers_together(model, bg, h0)
    if together:
        _forward_layers(model, bg, h0, histories, ids if do_push else None, betas, ys, zs)
        saved, y = [(z, None, out) for z, out in zip(zs, ys)], ys[-1]
    for l in range(1, L + 1) if not together else ():
        last = l == L
        z, x_next = zs[l - 1], ys[l - 1]
        y = x_next if fused or last else x_next[:nb]
        h, pushed = None, False
        table = (x_feat if l == 1 else histories[l - 2]) if fused else None
        if fused and model.op == "gcnii" and l == 1:
            table = None                                  # layer 1 gathers the projected features from h0 itself
        if short_rows and B.spmm_linear_supported(x, widths[l - 1]):
            # narrow layers: aggregation, transform and Push in one launch; Z is kept for the weight gradient
            push = not last and do_push
            beta = betas[l - 1]
            kw = dict(s_agg=1.0 - model.alpha, r=h0, s_res=model.alpha, c_identity=1.0 - beta,
                      c_weight=beta) if model.op == "gcnii" else {}
            src = bg.col if table is None else bg.src_first if in_place and l == 1 else bg.src
            B.gas_spmm_linear(bg.rowptr, src, bg.val, x, model.weights[l - 1], y, hist=table, relu=not last, z_out=z,
                              push_idx=ids if push else None, push_hist=histories[l - 1] if push else None, **kw)
            saved.append((z, h, y))
            if last:
                break
            x = x_next
            continue
        if model.op == "gcn":
            if in_place and l == 1:
                B.gas_spmm_table(bg.plan, bg.rowptr, bg.src_first, bg.val, table, z)
            elif fused:
                B.gas_spmm_hist(bg.plan, bg.rowptr, bg.src, bg.val, x, table, z)
            else:
                B.gas_spmm(bg.plan, bg.rowptr, bg.col, bg.val, x, z)
            pushed = not last and _pushes(do_push, histories[l - 1])
            if pushed:
                B.gas_linear_push(z, model.weights[l - 1], y, ids, histories[l - 1], relu=True)
            else:
                B.gas_linear(z, model.weights[l - 1], y, relu=not last)
        elif model.op == "gin":
            if fused:
                B.gas_spmm_hist(bg.plan, bg.rowptr, bg.src, None, x, table, z, diag=1.0 + model.gin_eps)
            else:
                B.gas_spmm(bg.plan, bg.rowptr, bg.col, None, x, z, diag=1.0 + model.gin_eps)
            w1, w2 = model.weights[l - 1]
            h = torch.empty((nb, w1.shape[1]), dtype=dt, device=dev)
            # both products in one call, the hidden activation stored for the backward pass, the Push in its epilogue
            push = not last and do_push
            B.gas_mlp2_keep(z, w1, w2, y, h, idx=ids if push else None,
                            hist=histories[l - 1] if push else None, relu_out=not last)
            pushed = push
        else:
            if table is not None:
                B.gas_spmm_hist(bg.plan, bg.rowptr, bg.src, bg.val, x, table, z, s_agg=1.0 - model.alpha, r=h0,
                                s_res=model.alpha)
            else:
                B.gas_spmm(bg.plan, bg.rowptr, bg.col, bg.val, x, z, s_agg=1.0 - model.alpha, r=h0, s_res=model.alpha)
            beta = betas[l - 1]
            pushed = not last and _pushes(do_push, histories[l - 1])
            if pushed:
                B.gas_linear_push(z, model.weights[l - 1], y, ids, histories[l - 1], c_identity=1.0 - beta,
                                  c_weight=beta, relu=True)
            else:
                B.gas_linear(z, model.weights[l - 1], y, c_identity=1.0 - beta, c_weight=beta, relu=not last)
        saved.append((z, h, y))
        if last:
            break
        if do_push and not pushed:
            B.gas_push(y, ids, histories[l - 1])
        if nv > nb and not fused:
            B.gas_pull(histories[l - 1], bg.n_id[nb:], x_next[nb:])
        x = x_next
    # ---- backward
    wg = _WeightGrads()
    grads = {}
    g = grad_out(y) if callable(grad_out) else grad_out     # a loss: gradient at the output, from the output
    g_h0 = None
    ready = None                              # the gradient at the layer's aggregated rows, if the launch above formed it
    one_width = L >= 4 and model.op != "gin" and all(i == o for i, o in zip(ins, widths))
    dws = _matrices(widths[0], widths, torch.float32, dev) if one_width else [None] * L
    # gradient matrices that wait for their weight gradients are allocated together
    pooled = one_width and dt == torch.float32 and 4 * nb * widths[0] <= wg.LARGEST
    gxs, spare, total = [], [], None
    joint = ()                                # widths of the layers whose input gradient shares the adjoint's launch
    if fused and (model.op == "gcnii" or (model.op == "gcn" and L > 2)):      # (GCN's first layer has none)
        joint = {(i, o) for i, o in set(zip(ins, widths))
                 if B.spmm_linear_supported(zs[ins.index(i)], o) and _back_in_one_launch(o, nb, bg.nnz_t, bg.max_col)}
    by_layers = together and pooled and joint == {(widths[0], widths[0])} and all(w.data_ptr() % 16 == 0 for w in model.weights)
    if by_layers:
        # the launches of as many layers in one call as wait for their weight gradients together
        f = widths[0]
        g_h0 = torch.zeros((nv, f), dtype=dt, device=dev)
        gzs = [torch.empty((nb, f), dtype=dt, device=dev) for _ in range(2)]      # in turn, layer L's first
        B.gas_linear_bwd_input_add(g, model.weights[L - 1], gzs[0], c_identity=1.0 - betas[L - 1], c_weight=betas[L - 1],
                                   total=g_h0[:nb], c_total=model.alpha)
        grads[L - 1] = wg.add(zs[L - 1], g, dws[L - 1], betas[L - 1])
        top = L - 1
        while top > 0:
            down = range(top - 1, max(-1, top - 1 - wg.TOGETHER), -1)
            gxs = _matrices(nb, [f] * len(down), dt, dev)
            for some in _layer_groups(len(down)):
                some, part = down[some.start:some.stop], gxs[some.start:some.stop]
                B.gas_spmm_t_relu_linear_layers(bg.colptr, bg.row, bg.val_t, gzs[(L - 2 - some[0]) % 2], [ys[l] for l in some], part,
                                                [model.weights[l] for l in some], [gzs[(L - 1 - l) % 2] for l in some],
                                                s_agg=1.0 - model.alpha, c_identity=[1.0 - betas[l] for l in some],
                                                c_weight=[betas[l] for l in some], total=g_h0[:nb], c_total=model.alpha)
            for l, gx in zip(down, gxs):
                grads[l] = wg.add(zs[l], gx, dws[l], betas[l])
            top = down[-1]
        gx = torch.empty((nv, f), dtype=dt, device=dev)
        B.gas_spmm_t(bg.plan_t_all, bg.colptr, bg.row, bg.val_t, gzs[(L - 1) % 2], gx, s_agg=1.0 - model.alpha)
        B.gas_axpy(g_h0, gx, g_h0, 1.0)
    for l in range(L, 0, -1) if not by_layers else ():
        z, h, _ = saved[l - 1]                # g: the gradient before this layer's activation
        gz, ready = ready, None
        if model.op == "gcn":
            grads[l - 1] = wg.add(z, g, dws[l - 1])
            if l > 1 and gz is None:          # below the first layer there is nothing to train
                gz = torch.empty_like(z)
                B.gas_linear_bwd_input(g, model.weights[l - 1], gz)
        elif model.op == "gin":
            gz = torch.empty_like(z)
            w1, w2 = model.weights[l - 1]
            dw2 = wg.add(h, g)
            gh = torch.empty_like(h)
            B.gas_linear_bwd_input(g, w2, gh, mask=h)
            grads[l - 1] = (wg.add(z, gh), dw2)
            B.gas_linear_bwd_input(gh, w1, gz)
            # gradient of this layer's eps: sum over the in-batch nodes of <dL/dZ_v, h_v> (h = the layer's input)
            if "eps" not in grads:
                grads["eps"] = torch.zeros(L, dtype=torch.float32, device=dev)
            x_in = x0 if l == 1 else saved[l - 2][2]
            B.gas_row_dot(gz, x_in[:nb], torch.empty(nb, dtype=torch.float32, device=dev), grads["eps"][l - 1:l])
        else:
            beta = betas[l - 1]
            grads[l - 1] = wg.add(z, g, dws[l - 1], beta)
            if g_h0 is None:
                g_h0 = torch.zeros((nv, z.shape[1]), dtype=dt, device=dev)
                total = g_h0[:nb]
            if gz is None:
                # the initial residual's share on the way: g_h0 += alpha * gz
                gz = torch.empty_like(z)
                B.gas_linear_bwd_input_add(g, model.weights[l - 1], gz, c_identity=1.0 - beta, c_weight=beta,
                                           total=total, c_total=model.alpha)
        if l == 1:
            if model.op == "gcnii":
                gx = torch.empty((nv, gz.shape[1]), dtype=dt, device=dev)
                B.gas_spmm_t(bg.plan_t_all, bg.colptr, bg.row, bg.val_t, gz, gx, s_agg=1.0 - model.alpha)
                B.gas_axpy(g_h0, gx, g_h0, 1.0)
            break
        # the adjoint of the aggregation and of the layer below's ReLU in one pass
        y_below = saved[l - 2][2]
        if pooled and not gxs:                # as many as wait together
            gxs = _matrices(nb, widths[max(0, l - 1 - wg.TOGETHER):l - 1], dt, dev)
        gx = gxs.pop() if gxs else torch.empty((nb, gz.shape[1]), dtype=dt, device=dev)
        s_agg = 1.0 - model.alpha if model.op == "gcnii" else 1.0
        w_below = model.weights[l - 2]
        if joint and (l > 2 or model.op == "gcnii") and (ins[l - 2], widths[l - 2]) in joint and w_below.data_ptr() % 16 == 0:
            # narrow layers: the layer below's input gradient in the same launch
            beta = betas[l - 2]
            ready = spare.pop() if spare and spare[-1].shape[1] == w_below.shape[0] else torch.empty(
                (nb, w_below.shape[0]), dtype=dt, device=dev)
            B.gas_spmm_t_relu_linear(bg.colptr, bg.row, bg.val_t, gz, y_below, gx, w_below, ready, s_agg=s_agg,
                                     c_identity=1.0 - beta, c_weight=beta,
                                     total=total, c_total=model.alpha)
            spare.append(gz)                  # read by this launch; the next one may write it
        elif model.op == "gin":
            B.gas_spmm_t_relu(bg.plan_t, bg.colptr, bg.row, None, gz, y_below, gx, diag=1.0 + model.gin_eps)
        else:
            B.gas_spmm_t_relu(bg.plan_t, bg.colptr, bg.row, bg.val_t, gz, y_below, gx, s_agg=s_agg)
        g = gx
    if model.op == "gcnii":
        gp = torch.empty_like(g_h0)
        B.gas_relu_bwd(g_h0, h0, gp)
        grads["w_in"] = wg.add(x0, gp)
    wg.done()
    return y, grads, {"x0": x0, "h0": h0, "layers": saved}


def _sgd(pairs, lr, weight_decay):
    """The plain update of every (w, dw), matrices of one dtype sharing launches."""
    if all(w.dtype == pairs[0][0].dtype for w, _ in pairs):
        B.gas_sgd_steps(pairs, lr, weight_decay)
        return
    for w, dw in pairs:
        B.gas_sgd_step(w, dw, lr, weight_decay)


def apply_sgd(model: Model, grads, lr, weight_decay=0.0, max_norm=None):
    """One gradient-descent update of every weight matrix, in place (gas_sgd_steps).  max_norm: the
    gradients are first clipped by their global L2 norm (paper, Section 3): one gas_sq_norm per gradient, then
    gas_sgd_step_clipped, which forms the common factor on the device."""
    pairs = []
    for l in range(model.n_layers):
        if model.op == "gin":
            pairs += list(zip(model.weights[l], grads[l]))
        else:
            pairs.append((model.weights[l], grads[l]))
    if model.op == "gcnii":
        pairs.append((model.w_in, grads["w_in"]))
    if max_norm is None:
        _sgd(pairs, lr, weight_decay)
        return
    sq = torch.empty(len(pairs), dtype=torch.float32, device=pairs[0][0].device)
    for k, (_, dw) in enumerate(pairs):
        B.gas_sq_norm(dw, sq[k:k + 1])
    for w, dw in pairs:
        B.gas_sgd_step_clipped(w, dw, lr, sq, max_norm, weight_decay)


def layer_input(model: Model, l, bg: BatchGraph, kept, histories):
    """The mini-batch tensor [nv, F] layer l read in a pass whose activations were kept (train_batch, not fused):
    the features (GCNII: the projected features) for l = 1, else layer l-1's output for the in-batch rows and the
    halo rows as they stand in history table l-1 (this batch's pushes do not touch them)."""
    if l == 1:
        return kept["h0"] if model.op == "gcnii" else kept["x0"]
    y = kept["layers"][l - 2][2]
    x = torch.empty((bg.nv, y.shape[1]), dtype=y.dtype, device=y.device)
    B.gas_pull(y, None, x[:bg.nb], base=0, n=bg.nb)
    if bg.nv > bg.nb:
        B.gas_pull(histories[l - 2], bg.n_id[bg.nb:], x[bg.nb:])
    return x


def train_step(model: Model, bg: BatchGraph, x_feat, histories, labels_batch, lr, weight_decay=0.0, n_labelled=None,
               fused=False, max_norm=None, reg_weight=0.0, reg_eps=None):
    """One optimisation step of Algorithm 1's loop body on one mini-batch: forward with Push/Pull per layer,
    softmax cross-entropy averaged over the labelled in-batch nodes, backward with the histories held constant,
    gradient-descent update of the weights (in place).  labels_batch: int32 [nb], the labels of the in-batch
    nodes in batch order, < 0 = unlabelled; n_labelled: their count if the caller knows it (saves a device
    read-back).  reg_weight: the local Lipschitz regulariser of Eq. (3) is added for every layer (lipschitz_reg_grad
    on the layer's kept input).  Returns (loss_sum as a 1-element float32 device tensor, n_labelled, logits, grads)."""
    if n_labelled is None:
        n_labelled = int((labels_batch >= 0).sum().item())
    dev = x_feat.device
    loss_rows = torch.empty(bg.nb, dtype=torch.float32, device=dev)
    loss_sum = torch.empty(1, dtype=torch.float32, device=dev)

    def loss_grad(y):
        g = torch.empty_like(y)
        B.gas_softmax_xent(y, labels_batch, g, loss_rows, loss_sum, scale=1.0 / max(1, n_labelled))
        return g
    y, grads, kept = _train_batch(model, bg, x_feat, histories, loss_grad, True, fused, keep_input=False)
    if reg_weight != 0.0:
        # loss + reg_weight * sum over the layers of Eq. (3), each differentiated with respect to its layer's
        # weights; reg_eps[l-1]: layer l's drawn perturbations [nv, F_in]
        if fused:
            raise ValueError("the regulariser perturbs the whole mini-batch tensor of every layer: fused=False")
        for l in range(1, model.n_layers + 1):
            _, _, dw = lipschitz_reg_grad(model, l, bg, layer_input(model, l, bg, kept, histories), reg_eps[l - 1],
                                          kept["h0"])
            for a, b in zip(grads[l - 1] if model.op == "gin" else (grads[l - 1],), dw if model.op == "gin" else (dw,)):
                B.gas_axpy(a, b, a, reg_weight)
    apply_sgd(model, grads, lr, weight_decay, max_norm)
    return loss_sum, n_labelled, y, grads


def appnp_forward_batch(w1, w2, alpha, n_steps, bg: BatchGraph, x_feat, histories, do_push=True, fused=False):
    """APPNP (paper, operator appendix) on one mini-batch: h0 = relu(x W1) W2 for every row of the mini-batch
    tensor (graph-agnostic, so exact for halo rows), then n_steps propagation steps
    h <- alpha h0 + (1 - alpha) A_hat h, each one aggregation call with the residual in its epilogue; steps
    1..K-1 are pushed to histories[l-1] and their halo rows pulled back.  fused: from step 2 on the aggregation
    reads the halo rows from the history table in place (no pull).  Returns h^(K) of the in-batch rows."""
    dev, dt = x_feat.device, x_feat.dtype
    nb, nv = bg.nb, bg.nv
    x0 = torch.empty((nv, x_feat.shape[1]), dtype=dt, device=dev)
    B.gas_pull(x_feat, bg.n_id, x0)
    h0 = torch.empty((nv, w2.shape[1]), dtype=dt, device=dev)
    B.gas_mlp2(x0, w1, w2, h0, relu_out=False)
    x, y = h0, None
    for l in range(1, n_steps + 1):
        last = l == n_steps
        x_next = torch.empty((nb if (last or fused) else nv, h0.shape[1]), dtype=dt, device=dev)
        y = x_next[:nb]
        if fused and l > 1:
            B.gas_spmm_hist(bg.plan, bg.rowptr, bg.src, bg.val, x, histories[l - 2], y, s_agg=1.0 - alpha, r=h0,
                            s_res=alpha)
        else:
            B.gas_spmm(bg.plan, bg.rowptr, bg.col, bg.val, x, y, s_agg=1.0 - alpha, r=h0, s_res=alpha)
        if last:
            break
        if do_push:
            B.gas_push(y, bg.n_id[:nb], histories[l - 1])
        if not fused and nv > nb:
            B.gas_pull(histories[l - 1], bg.n_id[nb:], x_next[nb:])
        x = x_next
    return y


# Rows from which on PNA's transforms go by degree, and their products' terms (rows x columns x outputs).
PNA_GROUPED_ROWS, PNA_GROUPED_TERMS = 24_576, 2_000_000_000


def _by_degree(bg: BatchGraph, x, w2, groups=None):
    """The batch's rows by degree if a PNA layer's transforms take them so (gas_pna_linear), else None: fp32, degrees up to
    PNA_MAX_DEGREE, and enough work that fewer columns outweigh the tiles that a degree fills in part, the degrees' matrices
    and two launches more.  Passes of three layers, us without -> with: 50,000 rows of 256 -> 256 forward 906 -> 758, training
    2,790 -> 2,471, 128 -> 128 414 -> 398 and 1,536 -> 1,415; but 100 -> 64 313 -> 311 and 1,083 -> 1,177, 16,000 rows of
    256 -> 256 359 -> 357 and 1,110 -> 1,090, 8,000 238 -> 264 and 722 -> 755.  The first pass over a batch builds the groups too: 50,000
    rows of 256 -> 256 951 -> 818 and 2,859 -> 2,544, 128 -> 128 454 -> 456 and 1,573 -> 1,459."""
    if x.dtype != torch.float32 or bg.max_row > B.PNA_MAX_DEGREE or bg.nb < PNA_GROUPED_ROWS or \
            bg.nb * w2.shape[0] * w2.shape[1] < PNA_GROUPED_TERMS or bg.nb < 512 * (bg.max_row + 1):
        return None
    return bg.groups if groups is None else groups


def _second_round(bg: BatchGraph, w2) -> bool:
    """Whether the tiles that degrees fill in part (half a tile for a degree) take the forward product by degree, 128 x 128 a
    workgroup, two on a compute unit, into a second round that the plain product does not need.  Forward passes of three layers,
    us without -> with: 30,500 rows of up to 25 entries, 256 -> 256 (502 tiles for 512 places), 536 -> 475, 31,500 (518)
    542 -> 579, 32,500 (532) 566 -> 590, 33,000, where the plain product has its second round too, 726 -> 598; 128 -> 128 at
    63,000 of up to 28 (506) 469 -> 449, 65,000 (521) 498 -> 517, 66,000 579 -> 534.  Outputs of 64 columns a tile, three
    workgroups on a compute unit, 32,000 rows of 192 -> 192 472 -> 466."""
    n = w2.shape[1]
    tiles, columns = -(-bg.nb // 128), -(-n // 128)
    return -(-n // 64) * 64 == columns * 128 and tiles * columns <= 512 < (bg.nb / 128 + (bg.max_row + 1) / 2) * columns


def _groups_of_layers(bg: BatchGraph, x, weights, gradients=True):
    """_by_degree of every layer of a pass, for its gradients and for its forward product; a pass under capture, which may have
    to record their building, records it once."""
    out, groups = [], None
    for _, w2 in weights:
        second = _second_round(bg, w2)
        got = _by_degree(bg, x, w2, groups) if gradients or not second else None
        groups = groups if got is None else got
        out.append((got, None if second else got))
    return out


def pna_layer(x, nb, rowptr, col, w1, w2, delta, relu, y=None, longest=B.ANY_LENGTH, idx=None, hist=None):
    """One PNA layer (paper, operator appendix) for the in-batch rows: h'_v = W2 [h_v, (+)_w W1 [h_v, h_w]].
    x: mini-batch tensor [nv, F]; w1 [2F, F1] (rows 0..F-1 multiply the receiving node, rows F.. the neighbour),
    w2 [F + 9 F1, F_out].  The neighbour part of a message is computed once per node (gas_linear over all of
    V_b), aggregated by mean, min and max in one pass with the degree scalers (gas_pna_aggregate), the
    receiving-node part is added inside that call, and the concatenation with h_v is laid out in one buffer
    that the second gas_linear reads."""
    dev, dt = x.device, x.dtype
    f, f1 = x.shape[1], w1.shape[1]
    p = torch.empty((x.shape[0], f1), dtype=dt, device=dev)
    B.gas_linear(x, w1[f:], p)
    q = torch.empty((nb, f1), dtype=dt, device=dev)
    B.gas_linear(x[:nb], w1[:f], q)
    cat = torch.empty((nb, f + 9 * f1), dtype=dt, device=dev)
    B.gas_pna_aggregate(rowptr, col, p, cat[:, f:], delta, add=q, longest=longest, own=x, own_to=cat[:, :f])   # h_v into the first F columns
    if y is None:
        y = torch.empty((nb, w2.shape[1]), dtype=dt, device=dev)
    if idx is not None:
        B.gas_linear_push(cat, w2, y, idx, hist, relu=relu)
    else:
        B.gas_linear(cat, w2, y, relu=relu)
    return y


def _pna_messages(bg: BatchGraph, x, w1, delta, blocks):
    """The neighbour part of the messages of every row of x and [h | aggregates]: the aggregators' `blocks` (9, or 3 without the
    scaled ones)."""
    dev, dt, nb = x.device, x.dtype, bg.nb
    f, f1 = x.shape[1], w1.shape[1]
    p = torch.empty((x.shape[0], f1), dtype=dt, device=dev)
    B.gas_linear(x, w1[f:], p)
    q = torch.empty((nb, f1), dtype=dt, device=dev)
    B.gas_linear(x[:nb], w1[:f], q)
    cat = torch.empty((nb, f + blocks * f1), dtype=dt, device=dev)
    # h_v goes into the first F columns
    B.gas_pna_aggregate(bg.rowptr, bg.col, p, cat[:, f:], delta, add=q, blocks=blocks, longest=bg.max_row, own=x, own_to=cat[:, :f])
    return p, cat


def pna_forward_batch(weights, delta, bg: BatchGraph, x_feat, histories, do_push=True):
    """All layers of a PNA model for one mini-batch in the order of Algorithm 1; weights[l] = (W1, W2)."""
    dev, dt = x_feat.device, x_feat.dtype
    nb, nv = bg.nb, bg.nv
    x = torch.empty((nv, x_feat.shape[1]), dtype=dt, device=dev)
    B.gas_pull(x_feat, bg.n_id, x)
    L = len(weights)
    y = None
    by_degree = _groups_of_layers(bg, x, weights, gradients=False)
    for l in range(1, L + 1):
        w1, w2 = weights[l - 1]
        last = l == L
        x_next = torch.empty((nb if last else nv, w2.shape[1]), dtype=dt, device=dev)
        groups = by_degree[l - 1][1]
        ids, hist = (bg.n_id[:nb], histories[l - 1]) if not last and _pushes(do_push, histories[l - 1]) else (None, None)
        if groups is None:
            y = pna_layer(x, nb, bg.rowptr, bg.col, w1, w2, delta, relu=not last, y=x_next[:nb], longest=bg.max_row, idx=ids, hist=hist)
        else:
            y, f, f1 = x_next[:nb], x.shape[1], w1.shape[1]
            cat = _pna_messages(bg, x, w1, delta, 3)[1]
            B.gas_pna_linear(groups, bg.max_row, cat, w2, f1, delta, y, relu=not last, idx=ids, hist=hist)
        if last:
            break
        _next_input(x_next, bg, histories[l - 1], do_push and hist is None)
        x = x_next
    return y


def gat_forward_batch(weights, bg: BatchGraph, x_feat, histories, negative_slope=0.2, do_push=True, heads=1):
    """All layers of a GAT (paper, operator appendix) for one mini-batch in the order of Algorithm 1;
    weights[l] = (W, a_dst, a_src); bg: the batch subgraph with self-loops.  Per layer: P = X W for every row of
    the mini-batch tensor (gas_linear_in_order), then scores, softmax and weighted sum in one pass (gas_gat_aggregate,
    ReLU in its epilogue on all layers but the last), push, pull.  heads > 1: the columns of W, a_dst and a_src are
    `heads` equal blocks, all taken by one gas_gat_aggregate call."""
    dev, dt = x_feat.device, x_feat.dtype
    nb, nv = bg.nb, bg.nv
    x = torch.empty((nv, x_feat.shape[1]), dtype=dt, device=dev)
    B.gas_pull(x_feat, bg.n_id, x)
    L = len(weights)
    y = None
    for l in range(1, L + 1):
        w, a_dst, a_src = weights[l - 1]
        last = l == L
        p = torch.empty((nv, w.shape[1]), dtype=dt, device=dev)
        B.gas_linear_in_order(x, w, p)                                # as in training: the same weights push the same rows
        x_next = torch.empty((nb if last else nv, w.shape[1]), dtype=dt, device=dev)
        y = x_next[:nb]
        if w.shape[1] % heads:
            raise ValueError("gat_forward_batch: the layer width is not a multiple of the number of heads")
        ids, hist = (bg.n_id[:nb], histories[l - 1]) if not last and _pushes(do_push, histories[l - 1]) else (None, None)
        B.gas_gat_aggregate(bg.rowptr, bg.col, p, a_dst, a_src, y, negative_slope, relu=not last, heads=heads, longest=bg.max_row,
                            idx=ids, hist=hist)
        if last:
            break
        _next_input(x_next, bg, histories[l - 1], do_push and hist is None)
        x = x_next
    return y


def _next_input(y_rows, bg: BatchGraph, history, do_push):
    """Push the in-batch rows (already in rows 0..nb-1 of the next mini-batch tensor) and pull its halo rows."""
    if do_push:
        B.gas_push(y_rows[:bg.nb], bg.n_id[:bg.nb], history)
    if bg.nv > bg.nb:
        B.gas_pull(history, bg.n_id[bg.nb:], y_rows[bg.nb:])


def pna_train_batch(weights, delta, bg: BatchGraph, x_feat, histories, grad_out, do_push=True):
    """pna_forward_batch with the activations kept, then the backward pass (operator appendix, PNA; histories are
    constants, so only in-batch rows pass gradient to the layer below, while the neighbour half of W1 takes gradient
    through every row of V_b).  bg needs the CSC copy with csc_pos.  grad_out: dLoss/dY_L [nb, F_L] or a function of
    Y_L.  Returns (Y_L, grads, kept) with grads[l] = (dW1 [2F, F1], dW2), float32, and kept[l] = the stored
    activations (X, P, [X[:nb] | A9], Y) the backward pass read.  Every step is a gas_* call."""
    dev, dt = x_feat.device, x_feat.dtype
    nb, nv = bg.nb, bg.nv
    x = torch.empty((nv, x_feat.shape[1]), dtype=dt, device=dev)
    B.gas_pull(x_feat, bg.n_id, x)
    L = len(weights)
    kept = []
    y = None
    by_degree = _groups_of_layers(bg, x, weights)
    for l in range(1, L + 1):
        w1, w2 = weights[l - 1]
        last = l == L
        groups = by_degree[l - 1][1]
        p, cat = _pna_messages(bg, x, w1, delta, 9)
        x_next = torch.empty((nb if last else nv, w2.shape[1]), dtype=dt, device=dev)
        y = x_next[:nb]
        pushed = not last and _pushes(do_push, histories[l - 1])
        if groups is not None:
            B.gas_pna_linear(groups, bg.max_row, cat, w2, w1.shape[1], delta, y, relu=not last, idx=bg.n_id[:nb] if pushed else None,
                             hist=histories[l - 1] if pushed else None)
        elif pushed:
            B.gas_linear_push(cat, w2, y, bg.n_id[:nb], histories[l - 1], relu=True)
        else:
            B.gas_linear(cat, w2, y, relu=not last)
        kept.append((x, p, cat, y))
        if last:
            break
        _next_input(x_next, bg, histories[l - 1], do_push and not pushed)
        x = x_next
    grads, wg = {}, _WeightGrads()
    g = grad_out(y) if callable(grad_out) else grad_out
    for l in range(L, 0, -1):
        w1, w2 = weights[l - 1]
        x, p, cat, _ = kept[l - 1]            # g: the gradient before this layer's activation
        f, f1 = x.shape[1], w1.shape[1]
        groups = by_degree[l - 1][0]
        if groups is not None:
            dw2 = torch.empty(w2.shape, dtype=torch.float32, device=dev)
            B.gas_pna_linear_bwd_weight(groups, bg.max_row, cat, g, f1, delta, dw2)
            gcat = torch.empty((nb, f + 3 * f1), dtype=dt, device=dev)       # the nine blocks folded with their scalers
            B.gas_pna_linear_bwd_input(groups, bg.max_row, g, w2, f1, delta, gcat)
        else:
            dw2 = wg.add(cat, g)
            gcat = torch.empty_like(cat)
            B.gas_linear_bwd_input(g, w2, gcat)
        gp = torch.empty((nv, f1), dtype=dt, device=dev)
        gq = torch.empty((nb, f1), dtype=dt, device=dev)
        B.gas_pna_aggregate_bwd(bg.rowptr, bg.col, bg.colptr, bg.row, bg.csc_pos, p, gcat[:, f:], gp, delta, gadd=gq,
                                plan_t=bg.plan_t_all, blocks=9 if groups is None else 3, longest=bg.max_row)
        dw1 = torch.empty((2 * f, f1), dtype=torch.float32, device=dev)
        wg.add(x[:nb], gq, dw1[:f])
        wg.add(x, gp, dw1[f:])
        grads[l - 1] = (dw1, dw2)
        if l == 1:
            break
        # dL/dX[:nb] = the copy of h_v in the concatenation + the neighbour part + the receiving-node part, then the
        # layer below's ReLU
        part = torch.empty((nb, f), dtype=dt, device=dev)
        B.gas_linear_bwd_input_add(gp[:nb], w1[f:], part, add=gcat[:, :f])
        g = torch.empty((nb, f), dtype=dt, device=dev)
        B.gas_linear_bwd_input_add(gq, w1[:f], g, add=part, mask=kept[l - 2][3])
    wg.done()
    return y, grads, kept


def gat_train_batch(weights, bg: BatchGraph, x_feat, histories, grad_out, negative_slope=0.2, do_push=True, heads=1):
    """gat_forward_batch with the activations kept, then the backward pass (operator appendix, GAT).  P = X W is
    computed for every node of V_b, so W takes gradient through all nv rows of P's gradient; only in-batch rows pass
    gradient to the layer below.  bg: the batch subgraph with self-loops and the CSC copy with csc_pos.
    Returns (Y_L, grads, kept) with grads[l] = (dW, d a_dst, d a_src), float32, and kept[l] = (X, P, Y).  Every
    step is a gas_* call."""
    dev, dt = x_feat.device, x_feat.dtype
    nb, nv = bg.nb, bg.nv
    x = torch.empty((nv, x_feat.shape[1]), dtype=dt, device=dev)
    B.gas_pull(x_feat, bg.n_id, x)
    L = len(weights)
    kept = []
    y = None
    for l in range(1, L + 1):
        w, a_dst, a_src = weights[l - 1]
        last = l == L
        p = torch.empty((nv, w.shape[1]), dtype=dt, device=dev)
        # The gradients of the attention vectors are sums that cancel: another order of the sums in p moves them by 1e-2 of
        # their norm in bf16.  Odd widths keep the order of k, here and in inference.
        B.gas_linear_in_order(x, w, p)
        x_next = torch.empty((nb if last else nv, w.shape[1]), dtype=dt, device=dev)
        y = x_next[:nb]
        if w.shape[1] % heads:
            raise ValueError("gat_train_batch: the layer width is not a multiple of the number of heads")
        ids, hist = (bg.n_id[:nb], histories[l - 1]) if not last and _pushes(do_push, histories[l - 1]) else (None, None)
        B.gas_gat_aggregate(bg.rowptr, bg.col, p, a_dst, a_src, y, negative_slope, relu=not last, heads=heads, longest=bg.max_row,
                            idx=ids, hist=hist)
        kept.append((x, p, y))
        if last:
            break
        _next_input(x_next, bg, histories[l - 1], do_push and hist is None)
        x = x_next
    grads, wg = {}, _WeightGrads()
    g = grad_out(y) if callable(grad_out) else grad_out
    for l in range(L, 0, -1):
        w, a_dst, a_src = weights[l - 1]
        x, p, _ = kept[l - 1]                 # g: the gradient before this layer's activation
        gp = torch.empty_like(p)
        gd = torch.empty(w.shape[1], dtype=torch.float32, device=dev)
        gs = torch.empty(w.shape[1], dtype=torch.float32, device=dev)
        B.gas_gat_aggregate_bwd(bg.rowptr, bg.col, bg.colptr, bg.row, bg.csc_pos, p, a_dst, a_src, g, gp, gd, gs,
                                negative_slope, plan_t=bg.plan_t_all, heads=heads, longest=bg.max_row, longest_col=bg.max_col_all)
        grads[l - 1] = (wg.add(x, gp), gd, gs)
        if l == 1:
            break
        g = torch.empty((nb, w.shape[0]), dtype=dt, device=dev)
        B.gas_linear_bwd_input(gp[:nb], w, g, mask=kept[l - 2][2])
    wg.done()
    return y, grads, kept


def sgd_update(weights, grads, lr, weight_decay=0.0):
    """gas_sgd_step on every tensor of a list of per-layer weight tuples (PNA, GAT) with the matching gradients."""
    _sgd([pair for l, ws in enumerate(weights) for pair in zip(ws, grads[l])], lr, weight_decay)


def layer_forward(model: Model, l, bg: BatchGraph, x, h0=None, y=None):
    """Layer l (1-based) of the model applied to a mini-batch tensor x [nv, F]: output for the in-batch rows."""
    dev, dt = x.device, x.dtype
    nb = bg.nb
    last = l == model.n_layers
    z = torch.empty((nb, x.shape[1]), dtype=dt, device=dev)
    if y is None:
        y = torch.empty((nb, model.out_width(l - 1)), dtype=dt, device=dev)
    if model.op == "gcn":
        B.gas_spmm(bg.plan, bg.rowptr, bg.col, bg.val, x, z)
        B.gas_linear(z, model.weights[l - 1], y, relu=not last)
    elif model.op == "gin":
        B.gas_spmm(bg.plan, bg.rowptr, bg.col, None, x, z, diag=1.0 + model.gin_eps)
        w1, w2 = model.weights[l - 1]
        B.gas_mlp2(z, w1, w2, y, relu_out=not last)
    elif model.op == "gcnii":
        B.gas_spmm(bg.plan, bg.rowptr, bg.col, bg.val, x, z, s_agg=1.0 - model.alpha, r=h0, s_res=model.alpha)
        beta = gcnii_beta(l)
        B.gas_linear(z, model.weights[l - 1], y, c_identity=1.0 - beta, c_weight=beta, relu=not last)
    else:
        raise ValueError(model.op)
    return y


def lipschitz_reg(model: Model, l, bg: BatchGraph, x, eps, h0=None):
    """Eq. (3) for layer l on one mini-batch: the layer applied to the mini-batch tensor x and to x + eps (one
    drawn perturbation per row, in-batch and halo rows alike), and the mean over the in-batch nodes of the
    distance between the two output rows.  Returns (sum of distances as a 1-element device tensor, nb)."""
    dev = x.device
    y = layer_forward(model, l, bg, x, h0)
    xp = torch.empty_like(x)
    B.gas_axpy(x, eps, xp, 1.0)
    y2 = layer_forward(model, l, bg, xp, h0)
    dist = torch.empty(bg.nb, dtype=torch.float32, device=dev)
    total = torch.empty(1, dtype=torch.float32, device=dev)
    B.gas_row_distance(y, y2, dist, total)
    return total, bg.nb


def lipschitz_reg_grad(model: Model, l, bg: BatchGraph, x, eps, h0=None):
    """Eq. (3) for layer l and its gradient with respect to that layer's weights (the layer's input held fixed).
    Both evaluations of the layer are differentiated: with u_v = (y_v - y'_v) / (nb ||y_v - y'_v||)
    (gas_row_distance_bwd) the output gradients are u and -u; each goes back through its own evaluation's stored
    activations (gas_relu_bwd, gas_linear_bwd_input for GIN's hidden layer, gas_linear_bwd_weight), and the two
    weight gradients are added.  Returns (sum of distances as a 1-element device tensor, nb, dW) with dW float32
    (a pair for GIN), scaled for the MEAN over the in-batch nodes."""
    dev, dt = x.device, x.dtype
    nb = bg.nb
    last = l == model.n_layers
    xp = torch.empty_like(x)
    B.gas_axpy(x, eps, xp, 1.0)
    outs = []
    for xx in (x, xp):
        z = torch.empty((nb, x.shape[1]), dtype=dt, device=dev)
        y = torch.empty((nb, model.out_width(l - 1)), dtype=dt, device=dev)
        h = None
        if model.op == "gcn":
            B.gas_spmm(bg.plan, bg.rowptr, bg.col, bg.val, xx, z)
            B.gas_linear(z, model.weights[l - 1], y, relu=not last)
        elif model.op == "gin":
            w1, w2 = model.weights[l - 1]
            B.gas_spmm(bg.plan, bg.rowptr, bg.col, None, xx, z, diag=1.0 + model.gin_eps)
            h = torch.empty((nb, w1.shape[1]), dtype=dt, device=dev)
            B.gas_linear(z, w1, h, relu=True)            # stored: the backward pass reads the hidden activation
            B.gas_linear(h, w2, y, relu=not last)
        else:
            beta = gcnii_beta(l)
            B.gas_spmm(bg.plan, bg.rowptr, bg.col, bg.val, xx, z, s_agg=1.0 - model.alpha, r=h0, s_res=model.alpha)
            B.gas_linear(z, model.weights[l - 1], y, c_identity=1.0 - beta, c_weight=beta, relu=not last)
        outs.append((z, h, y))
    y, y2 = outs[0][2], outs[1][2]
    dist = torch.empty(nb, dtype=torch.float32, device=dev)
    total = torch.empty(1, dtype=torch.float32, device=dev)
    B.gas_row_distance(y, y2, dist, total)
    u = torch.empty_like(y)
    B.gas_row_distance_bwd(y, y2, u, 1.0 / max(1, nb))

    def weight_grad(zz, gg, c):
        dw = torch.empty((zz.shape[1], gg.shape[1]), dtype=torch.float32, device=dev)
        ws = torch.empty(max(1, B.gas_linear_bwd_weight_workspace(zz.shape[0], zz.shape[1], gg.shape[1])),
                         dtype=torch.uint8, device=dev)
        B.gas_linear_bwd_weight(zz, gg, dw, ws, c_weight=c)
        return dw

    def add(a, b):
        B.gas_axpy(a, b, a, 1.0)                         # float32 matrices, in place
        return a

    grads = None
    for sign, (z, h, yy) in zip((1.0, -1.0), outs):
        g = u
        if not last:
            g = torch.empty_like(u)
            B.gas_relu_bwd(u, yy, g)
        if model.op == "gin":
            w1, w2 = model.weights[l - 1]
            dw2 = weight_grad(h, g, sign)
            gh = torch.empty_like(h)
            B.gas_linear_bwd_input(g, w2, gh, mask=h)
            part = (weight_grad(z, gh, sign), dw2)
            grads = part if grads is None else tuple(add(a, b) for a, b in zip(grads, part))
        else:
            c = gcnii_beta(l) if model.op == "gcnii" else 1.0
            part = weight_grad(z, g, sign * c)
            grads = part if grads is None else add(grads, part)
    return total, nb, grads
