"""The work a user has this library do, as cases that can be timed and checked.

A pass of a case goes through the public binding only (paper_2309_03523_amd.binding): a forward
of a recurrent layer over a fused batch of chunks, a training step of the EvolveGCN-O or of the
attention layer, an inference of the attention layer, or two epochs of the stale filter.  The graphs are
Chung-Lu snapshots (power-law degrees, dense next to sparse snapshots), the features N(0,1), the
cache the features plus a small drift, weights Xavier-uniform: the recipes of the repository's
configurations, drawn on the device from the seed alone.

Offline work that a training job does once (packing at create, labels, chunk generation, chunk
assignment) is preparation here.
"""
import math

import numpy as np
import torch

from paper_2309_03523_amd import binding

EVOLVE = ["W_init", "U_z", "V_z", "B_z", "U_r", "V_r", "B_r", "U_h", "V_h", "B_h"]


# ------------------------------------------------------------------------------------ the cases


def _recurrent(**kw):
    c = dict(kind="recurrent", T=8, N=1000, F=32, S=32, H=32, cell="gru", gcn_layers=1, concat=False, time_layers=1,
             edges=4000, spread=0.0, alpha=0.0, window=8, ranges=4, inside=0.0, chunks="ranges", presence=False)
    c.update(kw)
    return c


def _evolve(**kw):
    c = dict(kind="evolve", T=16, N=3000, F=64, edges=24000, spread=0.0, alpha=2.2, window=16, ranges=8, inside=0.0, dx=True)
    c.update(kw)
    return c


def _attention(**kw):
    c = dict(kind="attention", T=12, N=5001, F=128, edges=30000, spread=0.0, alpha=2.1, window=16, ranges=16, inside=0.0,
             train=False, dx=False)
    c.update(kw)
    return c


def listed():
    return [
        # The smallest fused batch: a GCN + GRU layer over a thousand vertices; launches and the serial steps count.
        _recurrent(name="gru_tiny", T=8, N=1000, edges=4000, ranges=4),
        # A middle-sized graph with odd sizes: vertex count, feature width, windows and ranges divide nothing.
        _recurrent(name="gru_ragged", T=10, N=12345, F=50, S=64, H=64, edges=60000, spread=0.5, alpha=2.1, window=4, ranges=13),
        # The benchmark's default configuration: 32 uneven power-law snapshots of 100 000 vertices, 64 chunks.
        _recurrent(name="gru_powerlaw", T=32, N=100000, F=128, S=128, H=128, edges=1000000, spread=1.0, alpha=2.1, window=8,
                   ranges=16),
        # MPNN-LSTM: two GCN layers, both outputs into the first of two LSTM layers, one long window.
        _recurrent(name="mpnn_lstm", T=32, N=40000, F=172, S=128, H=128, cell="lstm", gcn_layers=2, concat=True, time_layers=2,
                   edges=400000, spread=0.5, alpha=2.0, window=32, ranges=64, inside=0.85),
        # Vertices that come and go: sequences of different lengths concatenated into lanes.
        _recurrent(name="gru_presence", T=32, N=50000, F=128, S=128, H=128, edges=500000, spread=1.0, alpha=2.1, window=8, ranges=16,
                   presence=True),
        # Chunks as a label propagation generates them: label classes, states from a cache at every change of label.
        _recurrent(name="lstm_labels", T=24, N=30001, F=128, S=128, H=128, cell="lstm", edges=300000, spread=0.5, alpha=2.1,
                   chunks="labels", window=24, ranges=1),
        # Wide features and a wide hidden state.
        _recurrent(name="gru_wide", T=8, N=20000, F=300, S=256, H=256, edges=160000, alpha=2.2, window=8, ranges=8),
        # EvolveGCN-O training step on a small graph: the recurrence of the weights counts.
        _evolve(name="evolve_small"),
        # EvolveGCN-O training step with the input gradient on a large one (an eighth of the benchmark's vertices).
        _evolve(name="evolve_large", T=64, N=62500, F=256, edges=500000, alpha=2.2, window=16, ranges=8),
        # Inference of the graph attention + temporal attention layer on a small graph.
        _attention(name="attention_small"),
        # Its training step with the input gradient on a large one (a quarter of the benchmark's vertices).
        _attention(name="attention_large", T=16, N=250000, edges=1500000, alpha=2.1, ranges=128, train=True, dx=True),
        # The stale filter over an embedding table, two epochs.
        dict(name="stale_filter", kind="stale", R=3200000, F=128, dtype="f32", factor=0.4, listed_rows=False),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["recurrent"] * 6 + ["evolve"] * 2 + ["attention"] * 2 + ["stale"])
    if kind == "stale":
        return dict(kind="stale", R=_log_int(rng, 5000, 3000000), F=rng.choice([32, 64, 100, 128, 172, 256][:4 + rng.randrange(3)]),
                    dtype=rng.choice(["f32", "bf16"]), factor=round(rng.uniform(0.2, 0.7), 3), listed_rows=rng.random() < 0.4)
    if kind == "attention":
        T = rng.randint(4, 24)
        N = max(500, _log_int(rng, 20000, 3000000) // T)
        train = rng.random() < 0.7
        return _attention(T=T, N=N, edges=int(N * rng.uniform(2, 6)), spread=round(rng.uniform(0, 0.8), 2),
                          alpha=round(rng.uniform(2.1, 2.6), 2), window=rng.choice([T, max(2, T // 2)]),
                          ranges=rng.randint(1, min(64, N // 100)), inside=rng.choice([0.0, 0.85]), train=train,
                          dx=train and rng.random() < 0.5)
    if kind == "evolve":
        T = rng.randint(6, 64)
        F = rng.choice([32, 64, 128, 256])
        N = max(500, _log_int(rng, 30000, 400000000 // F) // T)
        return _evolve(T=T, N=N, F=F, edges=int(N * rng.uniform(3, 8)), alpha=round(rng.uniform(2.1, 2.6), 2),
                       window=rng.choice([T, max(2, T // 3)]), ranges=rng.randint(1, 16), inside=rng.choice([0.0, 0.85]),
                       dx=rng.random() < 0.5)
    T = rng.randint(4, 40)
    H = rng.choice([32, 64, 64, 128, 128, 128, 96, 256])
    N = max(300, _log_int(rng, 8000, 100000000 // H) // T)
    F = rng.choice([H, 16 + rng.randrange(180)])
    cell = rng.choice(["gru", "gru", "lstm", "lstm", "none"])
    two = rng.random() < 0.3
    built = H in (32, 64, 128) and cell != "none"      # widths the stacked time encoder and the concatenated input take
    c = _recurrent(T=T, N=N, F=F, S=H, H=H, cell=cell, gcn_layers=2 if two else 1,
                   concat=two and built and cell == "lstm" and rng.random() < 0.5,
                   time_layers=2 if built and rng.random() < 0.25 else 1,
                   edges=int(N * rng.uniform(2, 10)), spread=round(rng.uniform(0, 1), 2),
                   alpha=round(rng.uniform(2.0, 2.6), 2), window=rng.choice([T, max(2, T // 2), max(2, T // 4)]),
                   ranges=rng.randint(1, min(32, N // 64)), inside=rng.choice([0.0, 0.85]))
    option = rng.randrange(6)
    if option in (3, 5):
        c["presence"] = cell != "none"
    if option in (4, 5):
        c.update(chunks="labels", window=T, ranges=1)
    return c


# ------------------------------------------------------------------------------------ inputs


def _stream(seed, name):
    return np.random.default_rng([int(seed), *name.encode()])


def _gen(seed, name):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(_stream(seed, name).integers(1 << 62)))
    return g


def _weights(N, alpha):
    rank = np.arange(1, N + 1, dtype=np.float64)
    w = np.ones(N) if alpha == 0 else rank ** (-1.0 / (alpha - 1.0))
    return w / w.sum()


def _bounds(case, seed):
    """Uneven vertex ranges, each at least a quarter of the mean."""
    N, n = case["N"], case["ranges"]
    width = np.full(n, N // n // 4)
    extra = np.floor(_stream(seed, "ranges").dirichlet(np.ones(n)) * (N - width.sum())).astype(np.int64)
    extra[0] += N - width.sum() - extra.sum()
    return np.concatenate([[0], np.cumsum(width + extra)]).astype(np.int64)


def _graph(case, seed):
    """Per snapshot (rowptr int64 [N+1], col int32): symmetric, self-loops stored, columns ascending."""
    N, T = case["N"], case["T"]
    w = _weights(N, case["alpha"])[_stream(seed, "order").permutation(N)]
    cdf = torch.from_numpy(np.cumsum(w)).cuda()
    cdf0 = torch.cat([cdf.new_zeros(1), cdf])
    bounds = torch.from_numpy(_bounds(case, seed)).cuda()
    z = _stream(seed, "counts").standard_normal(T)
    s = case["spread"]
    counts = np.clip(np.exp(s * z - s * s / 2), 0.1, 6.0) * case["edges"]
    g = _gen(seed, "graph")
    loops = torch.arange(N, device="cuda")
    rowptr, cols = [], []
    for m in counts.astype(np.int64).tolist():
        u = torch.searchsorted(cdf, torch.rand(m, generator=g, device="cuda", dtype=torch.float64) * cdf[-1]).clamp_(max=N - 1)
        v = torch.searchsorted(cdf, torch.rand(m, generator=g, device="cuda", dtype=torch.float64) * cdf[-1]).clamp_(max=N - 1)
        if case["inside"] > 0:    # this share of the edges stays inside the first endpoint's range
            b = torch.searchsorted(bounds, u, right=True) - 1
            lo, hi = bounds[b], bounds[b + 1]
            r = cdf0[lo] + torch.rand(m, generator=g, device="cuda", dtype=torch.float64) * (cdf0[hi] - cdf0[lo])
            near = torch.minimum(torch.maximum(torch.searchsorted(cdf, r), lo), hi - 1)
            v = torch.where(torch.rand(m, generator=g, device="cuda") < case["inside"], near, v)
        key = torch.unique(torch.cat([u * N + v, v * N + u, loops * N + loops]))
        row = torch.div(key, N, rounding_mode="floor")
        cols.append((key - row * N).to(torch.int32))
        rp = torch.zeros(N + 1, dtype=torch.int64, device="cuda")
        rp[1:] = torch.cumsum(torch.bincount(row, minlength=N), 0)
        rowptr.append(rp)
    return rowptr, cols


def _chunks(case, seed):
    b = _bounds(case, seed).tolist()
    T, w = case["T"], case["window"]
    return [(b[i], b[i + 1], t, min(T, t + w)) for t in range(0, T, w) for i in range(len(b) - 1)]


def _xavier(rng, n_out, n_in):
    a = math.sqrt(6.0 / (n_in + n_out))
    return rng.uniform(-a, a, size=(n_out, n_in)).astype(np.float32)


def _round_bf16(a):
    return torch.from_numpy(np.asarray(a, np.float32)).to(torch.bfloat16).to(torch.float32).numpy()


def _params(case, seed):
    rng = _stream(seed, "parameters")
    p = {}
    if case["kind"] == "evolve":
        F = case["F"]
        for n in EVOLVE:
            p["evolve." + n] = (rng.uniform(-0.2, 0.2, (F, F)).astype(np.float32) if n[0] == "B" else _xavier(rng, F, F))
        return p
    if case["kind"] == "attention":
        S = case["F"]
        p = {"gat.weight": _xavier(rng, S, S), "gat.att_src": _xavier(rng, 8, S // 8), "gat.att_dst": _xavier(rng, 8, S // 8),
             "attn.pos": 0.1 * rng.standard_normal((case["T"], S))}
        p.update({"attn.weight_" + x: _xavier(rng, S, S) for x in "qkv"})
        return {k: _round_bf16(v) for k, v in p.items()}
    F, S, H = case["F"], case["S"], case["H"]
    for layer in range(case["gcn_layers"]):
        p["gcn%d.weight" % layer] = _xavier(rng, S, S if layer else F)
        p["gcn%d.bias" % layer] = rng.uniform(-0.1, 0.1, S).astype(np.float32)
    g = {"gru": 3, "lstm": 4, "none": 0}[case["cell"]] * H
    for layer in range(case["time_layers"] if g else 0):
        name = "rnn1" if layer else "rnn"
        p[name + ".weight_ih"] = _xavier(rng, g, H if layer else S * (2 if case["concat"] else 1))
        p[name + ".weight_hh"] = _xavier(rng, g, H)
        p[name + ".bias_ih"] = rng.uniform(-0.1, 0.1, g).astype(np.float32)
        p[name + ".bias_hh"] = rng.uniform(-0.1, 0.1, g).astype(np.float32)
    return p


def _normal(case, seed, name, width, base=None, dtype=torch.float32):
    """[T, N, width] of N(0,1) (or base + 0.1 N(0,1)), rows at a pitch of a multiple of 8 values."""
    T, N = case["T"], case["N"]
    g = _gen(seed, name)
    buf = torch.zeros((T, N, (width + 7) // 8 * 8), device="cuda", dtype=dtype)
    for t in range(T):
        z = torch.randn((N, width), generator=g, device="cuda")
        buf[t, :, :width] = z if base is None else base[t] + 0.1 * z
    return buf[:, :, :width]


def _labels(case, seed):
    """Communities of very different sizes (the largest hold a few per cent of the vertices), each of which is
    cut in time here and there: int32 [T, N]."""
    T, N = case["T"], case["N"]
    n = max(1, N // 16)
    rng = _stream(seed, "labels")
    community = np.minimum(n - 1, np.floor(n * rng.random(N) ** 4)).astype(np.int64)
    cut = rng.random((T, n)) < np.minimum(0.9, 0.1 + np.arange(n) / n)
    cut[0] = True
    since = np.maximum.accumulate(np.where(cut, np.arange(T)[:, None], 0), axis=0)
    return torch.from_numpy(np.ascontiguousarray(since[:, community] * n + community[None, :], dtype=np.int32)).cuda()


def _presence(case, seed):
    rng = _stream(seed, "presence")
    p = rng.uniform(0.15, 1.0, case["N"])
    return torch.from_numpy((rng.random((case["T"], case["N"])) < p).astype(np.uint8)).cuda()


def _inputs(case, seed):
    """Everything but the layer: tensors on the device by name."""
    case = dict(case)
    if case["kind"] == "stale":
        return _stale_inputs(case, seed)
    d = {"params": _params(case, seed), "chunks": _chunks(case, seed)}
    d["rowptr"], d["col"] = _graph(case, seed)
    dtype = torch.bfloat16 if case["kind"] == "attention" else torch.float32
    d["X"] = _normal(case, seed, "features", case["F"], dtype=dtype)
    d["C"] = _normal(case, seed, "cache", case["F"], d["X"], dtype=dtype)
    if case["kind"] != "recurrent":
        if case["kind"] == "evolve" or case["train"]:
            d["target"] = _normal(case, seed, "target", case["F"], dtype=dtype)
        return d
    d["C1"] = _normal(case, seed, "cache1", case["S"]) if case["gcn_layers"] == 2 else None
    d["labels"] = _labels(case, seed) if case["chunks"] == "labels" else None
    d["presence"] = _presence(case, seed) if case["presence"] else None
    if case["cell"] == "none":
        d["H0"] = None
    else:
        rows = case["T"] * case["N"] if d["labels"] is not None else len(range(0, case["T"], case["window"])) * case["N"]
        n = (2 if case["cell"] == "lstm" else 1) * case["time_layers"]
        d["H0"] = 0.1 * torch.randn((n * rows, case["H"]), generator=_gen(seed, "states"), device="cuda")
    return d


def _stale_inputs(case, seed):
    """Embeddings of two epochs, A and B, [R, F].  A tenth of the rows has not moved; the others moved by a
    Gaussian vector of a length between 0 and 2, many short ones and few long ones; exactly one by 2.  No length
    lies within a thousandth of the threshold, where the rounding of a distance would decide."""
    R, F = case["R"], case["F"]
    dtype = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    g = _gen(seed, "drift")
    length = 2.0 * (1.0 - torch.sqrt(torch.rand(R, generator=g, device="cuda")))
    length[torch.rand(R, generator=g, device="cuda") < 0.1] = 0.0
    A = torch.randn((R, F), generator=g, device="cuda")
    ld = (F + 7) // 8 * 8
    near = (length / 2.0 - case["factor"]).abs() < (1e-3 if case["dtype"] == "f32" else 2e-2)
    length[near | (length > 1.9)] = 0.0
    length[R // 2] = 2.0
    if case["dtype"] == "bf16":     # a step that bfloat16 keeps: one coordinate moves, from a value that it holds exactly
        at = torch.randint(0, F, (R,), generator=g, device="cuda")
        A = A.to(dtype).to(torch.float32)
        B = A.clone()
        B[torch.arange(R, device="cuda"), at] = 0.0
        A[torch.arange(R, device="cuda"), at] = length.to(dtype).to(torch.float32)
    else:
        d = torch.randn((R, F), generator=g, device="cuda")
        B = A + d * (length / d.norm(dim=1))[:, None]
        del d
    out = {}
    for name, E in (("A", A), ("B", B)):
        buf = torch.zeros((R, ld), device="cuda", dtype=dtype)
        buf[:, :F] = E.to(dtype)
        out[name] = buf[:, :F]
    out["rows"] = None
    if case["listed_rows"]:         # three rows in ten are read by another chunk
        out["rows"] = torch.sort(torch.randperm(R, generator=g, device="cuda")[:max(1, 3 * R // 10)])[0]
    return out


def prepare(case, seed):
    d = _inputs(case, seed)
    kind = case["kind"]
    if kind == "stale":
        R = case["R"]
        n = R if d["rows"] is None else int(d["rows"].numel())
        s = dict(case=case, A=d["A"], B=d["B"], rows=d["rows"], L=torch.empty_strided(d["B"].shape, d["B"].stride(),
                 dtype=d["B"].dtype, device="cuda").copy_(d["B"]))
        s["workspace"] = torch.empty(binding.stale_workspace_bytes(n), dtype=torch.uint8, device="cuda")
        for e in "AB":
            s["dist" + e] = torch.zeros(n, device="cuda")
            s["idx" + e] = torch.full((n,), -1, dtype=torch.int64, device="cuda")
            s["message" + e] = torch.zeros((n, d["A"].stride(0)), dtype=d["A"].dtype, device="cuda")
            s["result" + e] = torch.zeros(24, dtype=torch.uint8, device="cuda")
        return s
    F, T, N = case["F"], case["T"], case["N"]
    if kind == "recurrent":
        layer = binding.DgcLayer(d["rowptr"], d["col"], N, d["chunks"], F=F, S=case["S"], H=case["H"], time_kind=case["cell"],
                                 n_struct_layers=case["gcn_layers"], lstm_input_concat=case["concat"],
                                 n_time_layers=case["time_layers"])
    elif kind == "evolve":
        layer = binding.DgcLayer(d["rowptr"], d["col"], N, d["chunks"], F=F, S=F, H=F, time_kind="none",
                                 struct_kind="evolve_gcn_o", act_out="relu")
    else:
        layer = binding.DgcLayer(d["rowptr"], d["col"], N, d["chunks"], F=F, S=F, H=F, time_kind="self_attn", struct_kind="gat",
                                 dtype="bf16", heads=8)
    layer.set_params(d["params"])
    out_dim = layer.out_dim
    s = dict(case=case, layer=layer, shapes={k: v.shape for k, v in d["params"].items()}, X=d["X"], C=d["C"],
             Y=torch.zeros((T, N, out_dim), device="cuda", dtype=d["X"].dtype))
    if kind == "recurrent":
        if d["labels"] is not None:
            layer.set_labels(d["labels"])
        if d["presence"] is not None:
            layer.set_presence(d["presence"])
        s.update(C1=d["C1"], H0=d["H0"], HN=None if d["H0"] is None else torch.zeros_like(d["H0"]))
    else:
        s["target"] = d.get("target")
        s["loss"] = torch.zeros(1, device="cuda")
        s["dX"] = torch.zeros((T, N, F), device="cuda", dtype=d["X"].dtype) if case["dx"] else None
    return s


def run(s):
    case = s["case"]
    if case["kind"] == "stale":
        # Two epochs.  The copies hold B at the start; epoch A sends the rows that moved far, epoch B sends the same
        # rows back, so the copies end as they began.
        out = {}
        for e in "AB":
            binding.stale_filter(s[e], s["L"], F=case["F"], rows=s["rows"], factor=case["factor"], dist=s["dist" + e],
                                 send_idx=s["idx" + e], send_buf=s["message" + e], result=s["result" + e], workspace=s["workspace"])
            out[e] = {"dist": s["dist" + e], "send": s["idx" + e], "message": s["message" + e][:, :case["F"]],
                      "counts": s["result" + e].view(torch.int64)[::2], "scalars": s["result" + e].view(torch.float32)[2:4]}
        out["copies"] = s["L"]
        return out
    layer = s["layer"]
    if case["kind"] == "recurrent":
        layer.forward(s["X"], s["C"], s["Y"], C1=s["C1"], H0=s["H0"], HN=s["HN"])
        return {"Y": s["Y"], "HN": s["HN"]}
    layer.forward(s["X"], s["C"], s["Y"])
    if s["target"] is None:
        return {"Y": s["Y"]}
    layer.backward(s["Y"], target=s["target"], loss_out=s["loss"], dX=s["dX"])
    grads = {k: layer.get_param(k + ".grad", shape) for k, shape in s["shapes"].items()}
    return {"Y": s["Y"], "loss": s["loss"], "dX": s["dX"], "grads": grads}


# ------------------------------------------------------------------------------------ work


def _expected_nnz(case):
    """Stored non-zeros of all snapshots: of 2 m directed pairs drawn, the duplicates of a power-law graph fall away."""
    N = case["N"]
    w = _weights(N, case["alpha"])
    edge = np.unique(np.round(np.geomspace(1, N + 1, 200)).astype(np.int64))
    count = np.diff(edge).astype(np.float64)
    mean = np.add.reduceat(w, edge[:-1] - 1) / count
    pairs = count[:, None] * count[None, :]
    s, r, near = case["spread"], case["ranges"], case["inside"]
    nnz = 0.0
    for z in (-1.645, -1.036, -0.674, -0.385, -0.126, 0.126, 0.385, 0.674, 1.036, 1.645):
        m = case["edges"] * min(6.0, max(0.1, math.exp(s * z - s * s / 2)))
        for share, rate in ((1 / r, near * r + 1 - near), (1 - 1 / r, 1 - near)):     # pairs of one range, of two
            nnz += 0.1 * share * float((pairs * -np.expm1(-2.0 * m * rate * mean[:, None] * mean[None, :])).sum())
    return case["T"] * (nnz + N)


def work(case):
    if case["kind"] == "stale":
        F, size = case["F"], 4 if case["dtype"] == "f32" else 2
        n = case["R"] * (0.3 if case["listed_rows"] else 1.0)
        sent = 0.9 * n * (1.0 - case["factor"]) ** 2
        # both tables read, distances written; of the rows sent the copy and the message written, and their numbers
        return {"bytes": 2 * (n * (2 * F * size + 4) + sent * (2 * F * size + 8)), "flops": 2 * 3.0 * n * F}
    T, N, F = case["T"], case["N"], case["F"]
    rows, nnz = T * N, _expected_nnz(case)
    csr = 4 * nnz + 8 * T * (N + 1)
    if case["kind"] == "evolve":
        # X, cache, target read and Y written, per snapshot the aggregation, X W and its gradient; the weight recurrence
        n_b, n_f = 4, 2 * nnz * F + 4 * rows * F * F + 3 * T * 12 * F ** 3
        if case["dx"]:
            n_b, n_f = 5, n_f + 2 * nnz * F + 2 * rows * F * F
        return {"bytes": n_b * 4.0 * rows * F + csr, "flops": float(n_f)}
    if case["kind"] == "attention":
        # four projections, 2 x 8 heads x 16 features a neighbour, and the causal scores of the window
        f = rows * 8 * F * F + 4 * nnz * F + 2 * rows * F * min(case["window"], T)
        n_b = 3 + (1 if case["train"] else 0) + (1 if case["dx"] else 0)
        return {"bytes": n_b * 2.0 * rows * F + csr, "flops": float(f * (3 if case["train"] else 1))}
    S, H = case["S"], case["H"]
    part = 0.575 if case["presence"] else 1.0    # of the rows exist
    g = {"gru": 3, "lstm": 4, "none": 0}[case["cell"]] * H
    n_state = {"gru": 1, "lstm": 2, "none": 0}[case["cell"]] * case["time_layers"]
    flops = 2 * nnz * F * (part if case["gcn_layers"] == 1 else 1) + 2 * rows * F * S * (part if case["gcn_layers"] == 1 else 1)
    nbytes = 8.0 * rows * F + csr + 4 * rows * part * (H if g else S)
    if case["gcn_layers"] == 2:
        flops += part * (2 * nnz * S + 2 * rows * S * S)
        nbytes += 4 * rows * S
    flops += part * rows * g * (2 * S * (2 if case["concat"] else 1) + 2 * H + (4 * H if case["time_layers"] == 2 else 0))
    nbytes += 8 * n_state * H * (0.6 * rows if case["chunks"] == "labels" else len(range(0, T, case["window"])) * N)
    return {"bytes": nbytes, "flops": float(flops)}


def tolerance(case):
    # About four times what the start is off 64 bits by.  Gradients of the input carry single large differences: where an
    # output lies within rounding of zero the ReLU's gate opens or not (evolve), and a row's gradient is one sum of bfloat16
    # roundings beside much larger rows (attention).
    if case["kind"] == "attention":
        return {"rel": 1e-2, "max": 0.9}
    if case["kind"] == "stale":
        return {"rel": 1e-5, "max": 1e-4}
    if case["kind"] == "evolve":
        return {"rel": 1e-4, "max": 0.15}
    return {"rel": 1e-5, "max": 1e-4}


# ------------------------------------------------------------------------------------ 64 bits


def _sparse(rowptr, col, val, N):
    return torch.sparse_csr_tensor(rowptr, col.to(torch.int64), val, size=(N, N))


def _rows_of(rowptr):
    return torch.repeat_interleave(torch.arange(rowptr.numel() - 1, device=rowptr.device), rowptr[1:] - rowptr[:-1])


class _Normalised:
    """One snapshot's normalised adjacency, split into neighbours of the row's own chunk and the others."""

    def __init__(self, rowptr, col, group):
        N = rowptr.numel() - 1
        d = (rowptr[1:] - rowptr[:-1]).double().rsqrt()
        row = _rows_of(rowptr)
        val = d[row] * d[col.long()]
        own = (group[row] == group[col.long()]).double()
        self.own = _sparse(rowptr, col, val * own, N)
        self.others = _sparse(rowptr, col, val * (1 - own), N)

    def __call__(self, fresh, stale):
        return self.own @ fresh.double() + self.others @ stale.double()


def _groups(case, d):
    """Per snapshot, the chunk that each vertex belongs to."""
    if d.get("labels") is not None:
        return list(d["labels"])
    g = [torch.zeros(case["N"], dtype=torch.int64, device="cuda") for _ in range(case["T"])]
    for k, (lo, hi, t0, t1) in enumerate(d["chunks"]):
        for t in range(t0, t1):
            g[t][lo:hi] = k
    return g


def _cell(kind, x, h, c, p, name):
    gi = x @ p[name + ".weight_ih"].T + p[name + ".bias_ih"]
    gh = h @ p[name + ".weight_hh"].T + p[name + ".bias_hh"]
    if kind == "gru":
        ir, iz, i_n = gi.chunk(3, 1)
        hr, hz, hn = gh.chunk(3, 1)
        r, z = torch.sigmoid(ir + hr), torch.sigmoid(iz + hz)
        n = torch.tanh(i_n + r * hn)
        return (1 - z) * n + z * h, c
    i, f, g, o = (gi + gh).chunk(4, 1)
    c = torch.sigmoid(f) * c + torch.sigmoid(i) * torch.tanh(g)
    return torch.sigmoid(o) * torch.tanh(c), c


def _exact_recurrent(case, d):
    T, N, H, cell = case["T"], case["N"], case["H"], case["cell"]
    p = {k: torch.from_numpy(v).double().cuda() for k, v in d["params"].items()}
    groups = _groups(case, d)
    Y = torch.zeros((T, N, case["S"] if cell == "none" else H), dtype=torch.float64, device="cuda")
    lstm = cell == "lstm"
    n_state = 2 if lstm else 1
    if cell != "none":
        V = d["H0"].shape[0] // (n_state * case["time_layers"])
        H0 = d["H0"].double().view(case["time_layers"], n_state, V, H)
        HN = torch.zeros_like(H0)
        state = [[None, None] for _ in range(case["time_layers"])]
    for t in range(T):
        A = _Normalised(d["rowptr"][t], d["col"][t], groups[t])
        z = A(d["X"][t], d["C"][t]) @ p["gcn0.weight"].T + p["gcn0.bias"]
        if case["gcn_layers"] == 2:
            first = torch.relu(z)
            z = A(first, d["C1"][t]) @ p["gcn1.weight"].T + p["gcn1.bias"]
            if case["concat"]:
                z = torch.cat([first, z], 1)
        if cell == "none":
            Y[t] = z
            continue
        here = torch.ones(N, dtype=torch.bool, device="cuda") if d["presence"] is None else d["presence"][t].bool()
        if d["labels"] is None:
            rows = torch.arange(N, device="cuda") + (t // case["window"]) * N
            enters = torch.full((N,), t % case["window"] == 0, device="cuda")
            leaves = torch.full((N,), (t + 1) % case["window"] == 0 or t + 1 == T, device="cuda")
        elif d["presence"] is None:
            rows = torch.arange(N, device="cuda") + t * N
            enters = torch.ones_like(here) if t == 0 else groups[t] != groups[t - 1]
            leaves = torch.ones_like(here) if t + 1 == T else groups[t] != groups[t + 1]
        else:           # runs of present instances with one label
            rows = torch.arange(N, device="cuda") + t * N
            before = torch.full((N,), -1, dtype=torch.int64, device="cuda")
            after = before.clone()
            for u in range(t):
                before = torch.where(d["presence"][u].bool(), groups[u].long(), before)
            for u in range(T - 1, t, -1):
                after = torch.where(d["presence"][u].bool(), groups[u].long(), after)
            enters = here & (before != groups[t])
            leaves = here & (after != groups[t])
        x = z
        for layer in range(case["time_layers"]):
            h, c = state[layer]
            if h is None:
                h = torch.zeros((N, H), dtype=torch.float64, device="cuda")
                c = h
            h = torch.where(enters[:, None], H0[layer, 0][rows], h)
            c = torch.where(enters[:, None], H0[layer, n_state - 1][rows], c)
            nh, nc = _cell(cell, x, h, c, p, "rnn1" if layer else "rnn")
            h, c = torch.where(here[:, None], nh, h), torch.where(here[:, None], nc, c)
            state[layer] = [h, c]
            at = rows[leaves]
            HN[layer, 0][at] = h[leaves]
            if lstm:
                HN[layer, 1][at] = c[leaves]
            x = h
        Y[t] = torch.where(here[:, None], x, Y[t])
    return {"Y": Y, "HN": None if cell == "none" else HN.reshape(d["H0"].shape)}


def _evolved(P, T):
    W, out = P["W_init"], []
    for _ in range(T):
        z = torch.sigmoid(P["U_z"] @ W + P["V_z"] @ W + P["B_z"])
        r = torch.sigmoid(P["U_r"] @ W + P["V_r"] @ W + P["B_r"])
        c = torch.tanh(P["U_h"] @ W + P["V_h"] @ (r * W) + P["B_h"])
        W = (1 - z) * W + z * c
        out.append(W)
    return out


def _exact_evolve(case, d):
    T, N, F = case["T"], case["N"], case["F"]
    groups = _groups(case, d)
    P = {n: torch.from_numpy(d["params"]["evolve." + n]).double().cuda().requires_grad_() for n in EVOLVE}
    Ws = _evolved(P, T)
    Y = torch.zeros((T, N, F), dtype=torch.float64, device="cuda")
    dX = torch.zeros_like(Y) if case["dx"] else None
    loss, dWs = 0.0, []
    for t in range(T):
        A = _Normalised(d["rowptr"][t], d["col"][t], groups[t])
        W = Ws[t].detach()
        M = A(d["X"][t], d["C"][t])
        Y[t] = torch.relu(M @ W)
        off = Y[t] - d["target"][t].double()
        loss = loss + (off ** 2).sum() / (T * N * F)
        dP = 2.0 / (T * N * F) * off * (Y[t] > 0)
        dWs.append(M.T @ dP)
        if case["dx"]:
            dX[t] = A.own @ (dP @ W.T)           # symmetric
    torch.autograd.backward(Ws, dWs)
    return {"Y": Y, "loss": loss.reshape(1), "dX": dX, "grads": {"evolve." + n: P[n].grad for n in EVOLVE}}


def _segment(x, rowptr, how):
    return torch.segment_reduce(x, how, offsets=rowptr, axis=0, unsafe=True)


def _attend(rowptr, col, own, row, x, c, W, a_src, a_dst):
    """Graph attention of one snapshot before the ELU, [N, S]; rows are cut into pieces to bound the memory."""
    N = rowptr.numel() - 1
    zx, zc = (x @ W.T).view(N, 8, -1), (c @ W.T).view(N, 8, -1)
    sx, sc = (zx * a_src).sum(-1), (zc * a_src).sum(-1)
    e = (zx * a_dst).sum(-1)[row] + torch.where(own[:, None], sx[col], sc[col])
    e = torch.nn.functional.leaky_relu(e, 0.2)
    top = _segment(e.detach(), rowptr, "max")
    e = torch.exp(e - top[row])
    total = torch.zeros((N, 8), dtype=e.dtype, device=e.device).index_add(0, row, e)
    e = e / total[row]
    parts = []
    for h in range(8):
        parts.append(_Weighted.apply(rowptr, col, row, e[:, h] * own, zx[:, h]) +
                     _Weighted.apply(rowptr, col, row, e[:, h] * ~own, zc[:, h]))
    return torch.cat(parts, 1)


class _Weighted(torch.autograd.Function):
    """out[i] = sum of val over the stored row times z[col]; the adjacency's pattern is symmetric."""

    @staticmethod
    def forward(ctx, rowptr, col, row, val, z):
        ctx.save_for_backward(rowptr, col, row, val, z)
        return _sparse(rowptr, col, val, z.shape[0]) @ z.contiguous()

    @staticmethod
    def backward(ctx, g):
        rowptr, col, row, val, z = ctx.saved_tensors
        order = torch.sort(col, stable=True)[1]             # the transpose: same pattern, rows and columns exchanged
        gz = _sparse(rowptr, row[order], val[order], z.shape[0]) @ g.contiguous()
        return None, None, None, (g[row] * z[col]).sum(1), gz


def _temporal(g, pos, Wq, Wk, Wv):
    """g [w, n, S] -> [w, n, S]: causal attention of every vertex over the window, 8 heads."""
    w, n, S = g.shape
    p = g + pos[:, None, :]
    q, k, v = ((p @ M.T).view(w, n, 8, S // 8).permute(1, 2, 0, 3).contiguous() for M in (Wq, Wk, Wv))
    s = (q @ k.transpose(2, 3).contiguous()) / math.sqrt(S // 8)
    s = s.masked_fill(torch.ones((w, w), dtype=torch.bool, device=g.device).triu(1), -math.inf)
    return (torch.softmax(s, -1) @ v).permute(2, 0, 1, 3).reshape(w, n, S)


def _exact_attention(case, d):
    T, N, S = case["T"], case["N"], case["F"]
    P = {k: torch.from_numpy(v).double().cuda().requires_grad_() for k, v in d["params"].items()}
    groups = _groups(case, d)
    X, C = d["X"], d["C"]

    def snapshot(t, x):
        col, row = d["col"][t].long(), _rows_of(d["rowptr"][t])
        own = groups[t][row] == groups[t][col]
        u = _attend(d["rowptr"][t], col, own, row, x, C[t].double(), P["gat.weight"], P["gat.att_src"], P["gat.att_dst"])
        return torch.nn.functional.elu(u)

    G = torch.zeros((T, N, S), dtype=torch.float64, device="cuda")
    with torch.no_grad():
        for t in range(T):
            G[t] = snapshot(t, X[t].double())
    Y = torch.zeros_like(G)
    dG = torch.zeros_like(G) if case["train"] else None
    loss = 0.0
    for t0 in range(0, T, case["window"]):
        t1 = min(T, t0 + case["window"])
        for lo in range(0, N, 32768):
            hi = min(N, lo + 32768)
            g = G[t0:t1, lo:hi].clone().requires_grad_(case["train"])
            with torch.set_grad_enabled(case["train"]):
                y = _temporal(g, P["attn.pos"][t0:t1], P["attn.weight_q"], P["attn.weight_k"], P["attn.weight_v"])
            Y[t0:t1, lo:hi] = y.detach()
            if case["train"]:
                part = ((y - d["target"][t0:t1, lo:hi].double()) ** 2).sum() / (T * N * S)
                part.backward()
                loss = loss + part.detach()
                dG[t0:t1, lo:hi] = g.grad
    if not case["train"]:
        return {"Y": Y}
    dX = torch.zeros_like(G) if case["dx"] else None
    for t in range(T):
        x = X[t].double().requires_grad_()
        snapshot(t, x).backward(dG[t])
        if case["dx"]:
            dX[t] = x.grad
    return {"Y": Y, "loss": loss.reshape(1), "dX": dX, "grads": {k: v.grad for k, v in P.items()}}


def _exact_stale(case, d):
    out = {}
    A, B = d["A"], d["B"]
    rows = torch.arange(case["R"], device="cuda") if d["rows"] is None else d["rows"]
    dist = torch.cat([(a.double() - b.double()).norm(dim=1) for a, b in zip(A[rows].split(1 << 19), B[rows].split(1 << 19))])
    D = dist.max()
    sent = rows[dist > case["factor"] * D]
    for e, E, far in (("A", A, dist), ("B", B, torch.where(dist > case["factor"] * D, dist, torch.zeros_like(dist)))):
        message = torch.zeros((rows.numel(), case["F"]), dtype=torch.float64, device="cuda")
        message[:sent.numel()] = E[sent].double()
        out[e] = {"dist": far, "send": None, "message": message, "counts": None,
                  "scalars": torch.stack([D, case["factor"] * D])}
    out["copies"] = B.double()
    return out


def exact(case, seed):
    if case["kind"] == "attention" and _expected_nnz(case) > 8e6:
        return None         # minutes: the softmax over the longest rows
    d = _inputs(case, seed)
    return {"recurrent": _exact_recurrent, "evolve": _exact_evolve, "attention": _exact_attention,
            "stale": _exact_stale}[case["kind"]](case, d)
