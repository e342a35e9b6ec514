"""The edge-table kernels of the aggregation against the column-walking ones, over the forms that both take, and the input
gradient's table of the neighbours of a row's own chunk: split rows in it, rows with no other neighbour, other labels afterwards.
Bound of an fp32 sum of n products in any order: n + 3 roundings of 2^-24 of the sum of the products' sizes; two such sums
of normalised rows of N(0,1) are within 1e-6 of each other, root mean square, with rows of up to 2000 neighbours."""
import numpy as np
import pytest

import oracle
from oracle import labelled
from refs import rel_err
from workloads import synth

pytestmark = pytest.mark.gpu


def _graph(rng, N, hubs, degree):
    deg = rng.integers(0, degree, N)
    src = np.repeat(np.arange(N), deg)
    dst = rng.integers(0, N, src.size)
    for h in hubs:
        n = int(rng.integers(N // 40, N // 8))
        src, dst = np.append(src, np.full(n, h)), np.append(dst, rng.integers(0, N, n))
    key = np.unique(np.concatenate([src * N + dst, dst * N + src, np.arange(N) * N + np.arange(N)]))
    rowptr = np.zeros(N + 1, np.int64)
    rowptr[1:] = np.cumsum(np.bincount(key // N, minlength=N))
    return rowptr, (key % N).astype(np.int32)


@pytest.mark.parametrize("N,T,F,pitch,rows,long_nnz,part_nnz", [
    (900, 3, 1, 4, 0, 0, 0), (900, 3, 31, 32, 0, 0, 0), (901, 2, 32, 40, 3, 100, 32), (2500, 2, 33, 36, 0, 64, 17),
    (2500, 2, 64, 64, 16, 200, 64), (2500, 2, 130, 144, 5, 0, 0), (20000, 3, 300, 304, 0, 0, 0), (20000, 3, 260, 260, 0, 500, 100),
    (30000, 4, 128, 128, 0, 300, 512)])
def test_table_and_walk(N, T, F, pitch, rows, long_nnz, part_nnz):
    import torch
    from paper_2309_03523_amd import binding
    rng = synth.stream(N + F, "inside")
    snaps = [_graph(rng, N, rng.integers(0, N, 3), 12) for _ in range(T)]
    rowptr, col = ([torch.from_numpy(s[k]).cuda() for s in snaps] for k in (0, 1))
    cut = N // 3
    chunks = [(0, cut, 0, T), (cut, N, 0, T - 1)]
    X, C = (torch.zeros((T, N, pitch), device="cuda")[:, :, :F].copy_(torch.randn((T, N, F), device="cuda")) for _ in range(2))
    out = []
    for kernel in ("walk", "table"):
        layer = binding.DgcLayer(rowptr, col, N, chunks, F=F, S=32, H=32, time_kind="none", rows_per_group=rows, long_nnz=long_nnz,
                                 part_nnz=part_nnz, agg_kernel=kernel)
        M = torch.full((cut * T + (N - cut) * (T - 1), (F + 7) // 8 * 8), float("nan"), device="cuda")
        layer.aggregate(X, C, M)
        torch.cuda.synchronize()
        out.append(M.double())
        layer.destroy()
    assert torch.isfinite(out[1]).all() and bool((out[1][:, F:] == 0).all())
    off = float((out[1] - out[0]).norm() / out[0].norm())
    most = float((out[1] - out[0]).abs().max() / out[0].pow(2).mean().sqrt())
    print(f"N={N} F={F}: {off:.2e}, most {most:.2e}", flush=True)
    assert off < 1e-6 and most < 1e-4


def _ring(N, reach):
    """Every vertex with the `reach` before and behind it."""
    import torch
    i = torch.arange(N, device="cuda")
    col = torch.sort((i[:, None] + torch.arange(-reach, reach + 1, device="cuda")) % N, 1)[0]
    return torch.arange(N + 1, device="cuda") * (2 * reach + 1), col.reshape(-1).to(torch.int32)


@pytest.mark.parametrize("N,T,F,pitch,reach,long_nnz,part_nnz", [
    (90001, 3, 193, 200, 2, 0, 0), (90001, 3, 224, 224, 3, 4, 3), (90001, 3, 225, 232, 3, 0, 0),       # two slices of 128 columns; four of 64
    ((1 << 20) + 3, 1, 132, 132, 8, 0, 0), ((1 << 20) + 3, 1, 176, 176, 8, 0, 0),
    (3000, 4, 72, 72, 6, 0, 0), (3000, 4, 20, 24, 8, 0, 0)])                                           # a row for each lane group
def test_wide_slices_and_short_groups(N, T, F, pitch, reach, long_nnz, part_nnz):
    import torch
    from paper_2309_03523_amd import binding
    rowptr, col = _ring(N, reach)
    gen = torch.Generator(device="cuda").manual_seed(F)
    X, C = (torch.zeros((T, N, pitch), device="cuda")[:, :, :F].copy_(torch.randn((T, N, F), device="cuda", generator=gen)) for _ in range(2))
    out = []
    for kernel in ("walk", "table"):
        layer = binding.DgcLayer([rowptr] * T, [col] * T, N, [(0, N // 3, 0, T), (N // 3, N, 0, T)], F=F, S=32, H=32, time_kind="none",
                                 long_nnz=long_nnz, part_nnz=part_nnz, agg_kernel=kernel)
        M = torch.full((N * T, (F + 7) // 8 * 8), float("nan"), device="cuda")
        layer.aggregate(X, C, M)
        torch.cuda.synchronize()
        out.append(M)
        layer.destroy()
    assert bool(torch.isfinite(out[1]).all()) and bool((out[1][:, F:] == 0).all())
    assert float((out[1] - out[0]).double().norm() / out[0].double().norm()) < 1e-6


def test_missing_numbers_stay_where_they_are():
    """NaN in the rows of other chunks' fresh features and in cache rows of the own chunk, which no sum depends on."""
    import torch
    from paper_2309_03523_amd import binding
    N, F = 1000, 70
    rowptr, col = _graph(synth.stream(3, "nan"), N, [5], 6)
    X, C = (torch.randn((1, N, 72), device="cuda")[:, :, :F] for _ in range(2))
    layer = binding.DgcLayer([torch.from_numpy(rowptr).cuda()], [torch.from_numpy(col).cuda()], N, [(200, 600, 0, 1)], F=F, S=32, H=32,
                             time_kind="none")
    M = torch.zeros((400, 72), device="cuda")
    layer.aggregate(X, C, M)
    want = M.clone()
    X[0, :200] = float("nan")
    X[0, 600:] = float("inf")
    C[0, 200:600] = float("nan")
    layer.aggregate(X, C, M)
    torch.cuda.synchronize()
    assert torch.equal(M, want)
    layer.destroy()


@pytest.mark.parametrize("F,rows,long_nnz,part_nnz", [(32, 0, 0, 0), (64, 4, 20, 7), (128, 16, 40, 16), (256, 0, 60, 200)])
def test_input_gradient_of_split_rows(F, rows, long_nnz, part_nnz):
    """Where an output lies within rounding of zero its ReLU may open on one side only, and its row's gradient is another one: such
    elements of Y (at most a few in 1e5) and the rows that they hand a gradient to are left out."""
    import torch
    from paper_2309_03523_amd.runner import DeviceWorkload
    T, N = 3, 410
    chunks = [[0, 1, 0, 3], [1, 180, 0, 3], [180, 410, 1, 3]]          # (the first row: no neighbour of its chunk but itself)
    wl = synth.random_small(300 + F, T, N, F, F, F, 6.0, chunks, "none", hub=True)
    wl.params = synth.evolve_params(300 + F, F, F, random_bias=True)
    target = synth.stream(F, "target").standard_normal((T, N, F)).astype(np.float32)
    dw = DeviceWorkload(wl, struct_kind="evolve_gcn_o", act_out="relu", rows_per_group=rows, long_nnz=long_nnz, part_nnz=part_nnz)
    Y = dw.forward()
    dX = torch.full((T, N, F), np.nan, device="cuda")
    dw.layer.backward(Y, target=torch.from_numpy(target).cuda(), dX=dX)
    torch.cuda.synchronize()
    got = Y.cpu().numpy()
    want = oracle.evolve(wl.graph, wl.chunks, wl.params, wl.X, wl.C, target, want_grads=True, want_dx=True)
    m = ~np.isnan(want["dX"]).any(axis=2) & ~np.isnan(want["Y"]).any(axis=2)
    assert m.sum() == 3 + 3 * 179 + 2 * 230
    flipped = ((got > 0) != (want["Y"] > 0)) & m[..., None]
    assert flipped.sum() <= 3 and np.abs(got[flipped]).max(initial=0) < 1e-6 and np.abs(want["Y"][flipped]).max(initial=0) < 1e-6
    for t, i in zip(*np.nonzero(flipped.any(axis=2))):
        s = wl.graph.snaps[t]
        m[t, s.col[s.rowptr[i]:s.rowptr[i + 1]]] = False
    print(f"F={F}: {int(flipped.sum())} gates on one side only, {int(m.sum())} rows compared", flush=True)
    assert m.sum() > 600
    assert rel_err(got[m], want["Y"][m]) < 1e-4 and rel_err(dX.cpu().numpy()[m], want["dX"][m]) < 1e-4
    dw.layer.destroy()


def test_input_gradient_after_other_labels():
    """Two input gradients of one layer, other labels in between: the table follows them."""
    import torch
    from paper_2309_03523_amd.runner import DeviceWorkload
    T, N, F = 3, 200, 64
    wl = synth.random_small(12, T, N, F, F, F, 6.0, [[0, N, 0, T]], "none", hub=True)
    wl.params = synth.evolve_params(12, F, F, random_bias=True)
    target = synth.stream(F, "target").standard_normal((T, N, F)).astype(np.float32)
    dw = DeviceWorkload(wl, struct_kind="evolve_gcn_o", act_out="relu")
    rng = np.random.default_rng(4)
    for classes in (2, 9, 1):
        lab = rng.integers(0, classes, (T, N))
        dw.layer.set_labels(torch.from_numpy(lab.astype(np.int32).reshape(-1)).cuda())
        Y = dw.forward()
        dX = torch.full((T, N, F), np.nan, device="cuda")
        dw.layer.backward(Y, target=torch.from_numpy(target).cuda(), dX=dX)
        torch.cuda.synchronize()
        want = labelled.evolve(wl.graph, lab, wl.params, wl.X, wl.C, target, want_dx=True)
        assert rel_err(Y.cpu().numpy(), want["Y"]) < 1e-4 and rel_err(dX.cpu().numpy(), want["dX"]) < 1e-4, classes
    dw.layer.destroy()


@pytest.mark.parametrize("first,recorded", [(None, None), (None, 9), (4, 2), (4, None)])
def test_recorded_training_step_after_other_labels(first, recorded):
    """A step with input gradient that is recorded into a graph (classes of labels before the first eager step and before the recording), and replayed with labels that have more
    and fewer neighbours in a chunk: every replay against an eager step of the same labels, and both against the oracle."""
    import torch
    from paper_2309_03523_amd.runner import DeviceWorkload
    T, N, F = 3, 300, 64
    wl = synth.random_small(13, T, N, F, F, F, 6.0, [[0, N, 0, T]], "none", hub=True)
    wl.params = synth.evolve_params(13, F, F, random_bias=True)
    target = synth.stream(F, "target").standard_normal((T, N, F)).astype(np.float32)
    dw = DeviceWorkload(wl, struct_kind="evolve_gcn_o", act_out="relu", long_nnz=30, part_nnz=11)
    on_device, dX = torch.from_numpy(target).cuda(), torch.zeros((T, N, F), device="cuda")
    rng = np.random.default_rng(7)

    def labels(classes):
        lab = rng.integers(0, classes, (T, N))
        dw.layer.set_labels(torch.from_numpy(lab.astype(np.int32).reshape(-1)).cuda())
        return lab

    def step():
        dw.layer.forward(dw.X, dw.C, dw.Y)
        dw.layer.backward(dw.Y, target=on_device, dX=dX)

    def results():
        torch.cuda.synchronize()
        grads = {n: dw.layer.get_param(n + ".grad", wl.params[n].shape) for n in oracle.EVOLVE_PARAMS}
        return dict(grads, Y=dw.Y.cpu().numpy(), dX=dX.cpu().numpy())

    side = torch.cuda.Stream()
    if first:
        labels(first)
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        step()
    torch.cuda.synchronize()
    if recorded:
        labels(recorded)                       # no eager step between the labels and the recording
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        step()
    for classes, eager_first in ((5, False), (1, False), (30, True), (2, True)):
        lab = labels(classes)
        if eager_first:
            step()
            eager = results()
        for t in (dw.Y, dX):
            t.fill_(float("nan"))
        graph.replay()
        got = results()
        if not eager_first:
            step()
            eager = results()
        for k in eager:
            if k == "dX" and not (first or recorded):      # recorded without labels: the same products, added in another order
                assert np.linalg.norm(got[k] - eager[k]) < 1e-6 * np.linalg.norm(eager[k]), classes
            else:
                np.testing.assert_array_equal(got[k], eager[k], err_msg=f"{classes} classes: {k}")
        want = labelled.evolve(wl.graph, lab, wl.params, wl.X, wl.C, target, want_dx=True)
        assert rel_err(got["Y"], want["Y"]) < 1e-4 and rel_err(got["dX"], want["dX"]) < 1e-4, classes
    dw.layer.destroy()


@pytest.mark.parametrize("F", [20, 64, 200])
def test_infinities_stay_infinities(F):
    """Sums with one infinite term are infinite, not NaN, whatever the length of their row and of those beside it."""
    import torch
    from paper_2309_03523_amd import binding
    N = 700
    rowptr, col = _graph(synth.stream(9, "inf"), N, [5, 300], 9)
    X = torch.randn((1, N, F), device="cuda")
    X[0, ::13] = float("inf")
    row = np.repeat(np.arange(N), np.diff(rowptr))
    hit = np.zeros(N, bool)
    hit[row[col % 13 == 0]] = True
    assert 50 < hit.sum() < N - 50
    layer = binding.DgcLayer([torch.from_numpy(rowptr).cuda()], [torch.from_numpy(col).cuda()], N, [(0, N, 0, 1)], F=F, S=32, H=32,
                             time_kind="none")
    M = torch.zeros((N, (F + 7) // 8 * 8), device="cuda")
    layer.aggregate(X, X, M)
    torch.cuda.synchronize()
    got = M.cpu().numpy()[:, :F]
    assert np.isposinf(got[hit]).all() and np.isfinite(got[~hit]).all()
    layer.destroy()


def _pairs(N):
    """Vertices 2k and 2k + 1 are neighbours; the last one of an odd number has none."""
    import torch
    i = torch.arange(N, device="cuda")
    other = torch.where((i ^ 1) < N, i ^ 1, i)
    n = 1 + (other != i).long()
    rowptr = torch.zeros(N + 1, dtype=torch.int64, device="cuda")
    rowptr[1:] = torch.cumsum(n, 0)
    col = torch.stack([torch.minimum(i, other), torch.maximum(i, other)], 1).reshape(-1)
    keep = torch.ones(2 * N, dtype=torch.bool, device="cuda")
    keep[1::2] = n == 2
    return rowptr, col[keep].to(torch.int32)


def test_more_rows_than_a_launch_has_waves():
    """Groups of one row: the second GCN layer's four slices of each are more waves than a launch can hold."""
    import torch
    from paper_2309_03523_amd import binding
    N, F, S = (1 << 24) + 77, 16, 256
    rowptr, col = _pairs(N)
    gen = torch.Generator(device="cuda").manual_seed(3)
    X = torch.randn((1, N, F), device="cuda", generator=gen)
    C1 = torch.zeros((1, N, S), device="cuda")
    layer = binding.DgcLayer([rowptr], [col], N, [(0, N, 0, 1)], F=F, S=S, H=S, time_kind="none", n_struct_layers=2, rows_per_group=1)
    rng = synth.stream(3, "large")
    p = {"gcn0.weight": rng.standard_normal((S, F)) / 4, "gcn0.bias": rng.standard_normal(S),
         "gcn1.weight": rng.standard_normal((S, S)) / 16, "gcn1.bias": rng.standard_normal(S)}
    p = {k: v.astype(np.float32) for k, v in p.items()}
    layer.set_params(p)
    Y = torch.full((1, N, S), float("nan"), device="cuda")
    layer.forward(X, X, Y, C1=C1)
    torch.cuda.synchronize()
    layer.destroy()
    assert all(bool(torch.isfinite(y).all()) for y in Y[0].split(1 << 20))
    at = torch.cat([torch.arange(1000), N - 1 - torch.arange(1000), (1 << 23) - 500 + torch.arange(1000), torch.randint(0, N, (4000,))]).cuda()
    w = {k: torch.from_numpy(v).double().cuda() for k, v in p.items()}

    def first(i):
        return torch.relu(mean(lambda j: X[0, j].double(), i) @ w["gcn0.weight"].T + w["gcn0.bias"])

    def mean(f, i):
        other = torch.where((i ^ 1) < N, i ^ 1, i)
        return 0.5 * (f(i) + f(other))

    want = mean(first, at) @ w["gcn1.weight"].T + w["gcn1.bias"]
    assert float((Y[0, at].double() - want).norm() / want.norm()) < 1e-6


def test_more_rows_than_a_launch_counts_neighbours_of():
    """The input gradient's table over more groups than one launch counts and fills, against the kernels that walk the columns.
    Of 1e9 outputs some lie so near zero that their ReLU opens in one forward only: both gradients are those of one Y."""
    import torch
    from paper_2309_03523_amd import binding
    N, F = (1 << 25) + 1001, 32
    rowptr, col = _pairs(N)
    gen = torch.Generator(device="cuda").manual_seed(4)
    X, target = (torch.randn((1, N, F), device="cuda", generator=gen) for _ in range(2))
    p = synth.evolve_params(4, F, F, random_bias=True)
    cut = (1 << 24) + 1
    out = []
    for kernel in ("walk", "table"):
        layer = binding.DgcLayer([rowptr], [col], N, [(0, cut, 0, 1), (cut, N, 0, 1)], F=F, S=F, H=F, time_kind="none",
                                 struct_kind="evolve_gcn_o", act_out="relu", rows_per_group=1, agg_kernel=kernel)
        layer.set_params(p)
        Y, dX = torch.zeros((1, N, F), device="cuda"), torch.full((1, N, F), float("nan"), device="cuda")
        layer.forward(X, X, Y)
        Y = out[0][1] if out else Y
        layer.backward(Y, target=target, dX=dX)
        torch.cuda.synchronize()
        layer.destroy()
        out.append((dX.double(), Y))
    assert bool(torch.isfinite(out[1][0]).all())
    assert float((out[0][0] - out[1][0]).norm() / out[0][0].norm()) < 1e-6


@pytest.mark.parametrize("labelled_layer", [False, True])
def test_last_row_without_a_neighbour_of_its_chunk(labelled_layer):
    """Only a graph without the row's self-loop, which validate_level = 1 refuses, has one; nothing hands a gradient to it.  Its lanes read the
    entry behind the table's last."""
    import torch
    from paper_2309_03523_amd import binding
    N, F = 64, 32
    i = torch.arange(N - 1, device="cuda")
    rowptr = torch.arange(N + 1, device="cuda")
    rowptr[1:] += 1                                               # vertex 0: itself and the last one
    col = torch.cat([i[:1], i.new_tensor([N - 1]), i[1:], i[:1]]).to(torch.int32)
    chunks = [(0, N, 0, 1)] if labelled_layer else [(0, N // 2, 0, 1), (N // 2, N, 0, 1)]
    gen = torch.Generator(device="cuda").manual_seed(5)
    X, target = (torch.randn((1, N, F), device="cuda", generator=gen) for _ in range(2))
    layer = binding.DgcLayer([rowptr], [col], N, chunks, F=F, S=F, H=F, time_kind="none", struct_kind="evolve_gcn_o", act_out="relu",
                             validate_level=0)
    layer.set_params(synth.evolve_params(5, F, F, random_bias=True))
    if labelled_layer:
        layer.set_labels((torch.arange(N, device="cuda") >= N // 2).to(torch.int32))
    Y, dX = torch.zeros((1, N, F), device="cuda"), torch.full((1, N, F), float("nan"), device="cuda")
    left = [torch.full((k,), float("nan"), device="cuda") for k in (1 << 12, 1 << 16, 1 << 19)]      # for the layer's workspace to find
    torch.cuda.synchronize()
    del left
    torch.cuda.empty_cache()
    layer.forward(X, X, Y)
    layer.backward(Y, target=target, dX=dX)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(dX).all()) and bool((dX[0, N - 1] == 0).all()) and bool((dX[0, N - 2] != 0).any())
    layer.destroy()


@pytest.mark.parametrize("N,rows,degree", [(40, 0, 1), (700, 1, 9), (9001, 16, 12), (9001, 5, 40), (30000, 0, 6)])
def test_table_of_long_and_short_rows(N, rows, degree):
    """Items of a few entries and of several reads of 512 (rows of up to 3750), against the kernels that walk the columns."""
    import torch
    from paper_2309_03523_amd import binding
    F, T = 32, 2
    rng = synth.stream(N + rows, "long and short")
    snaps = [_graph(rng, N, rng.integers(0, N, 5), degree) for _ in range(T)]
    rowptr, col = ([torch.from_numpy(s[k]).cuda() for s in snaps] for k in (0, 1))
    gen = torch.Generator(device="cuda").manual_seed(6)
    X, target = (torch.randn((T, N, F), device="cuda", generator=gen) for _ in range(2))
    p = synth.evolve_params(4, F, F, random_bias=True)
    out = []
    for kernel in ("walk", "table"):
        layer = binding.DgcLayer(rowptr, col, N, [(0, N // 3, 0, T), (N // 3, N, 0, T)], F=F, S=F, H=F, time_kind="none",
                                 struct_kind="evolve_gcn_o", act_out="relu", rows_per_group=rows, agg_kernel=kernel)
        layer.set_params(p)
        Y, dX = torch.zeros((T, N, F), device="cuda"), torch.full((T, N, F), float("nan"), device="cuda")
        layer.forward(X, X, Y)
        Y = out[0][1] if out else Y            # (the same gates for both)
        layer.backward(Y, target=target, dX=dX)
        torch.cuda.synchronize()
        layer.destroy()
        out.append((dX.double(), Y))
    assert bool(torch.isfinite(out[1][0]).all())
    assert float((out[0][0] - out[1][0]).norm() / out[0][0].norm()) < 1e-6
