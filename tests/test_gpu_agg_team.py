"""Rows that the four waves of a workgroup share in the aggregation: lengths around every threshold (a row per lane group, a
row per wave, four batches of a wave, split rows), groups of one row up to 32, a workgroup whose last groups are missing, and short
parts, few (shared) and more than the chip holds workgroups (one a wave).
Bound of an fp32 sum of n products in any order: n + 3 roundings of 2^-24 of the sum of the products' sizes."""
import numpy as np
import pytest

import oracle
from refs import rel_err
from workloads import synth

pytestmark = pytest.mark.gpu

LENGTHS = [1, 2, 8, 9, 16, 17, 31, 32, 33, 34, 63, 64, 65, 96, 127, 128, 129, 131, 255, 256, 257, 400, 511, 640]


@pytest.mark.parametrize("F", [5, 64, 66, 128, 200, 300])
@pytest.mark.parametrize("rows_per_group,long_nnz,part_nnz", [(0, 0, 0), (16, 256, 100), (32, 500, 130), (5, 40, 33), (16, 130, 16)])
def test_shared_rows(F, rows_per_group, long_nnz, part_nnz):
    import torch
    from paper_2309_03523_amd import binding
    N, T = 659, 2
    rng = synth.stream(F + rows_per_group, "rows")
    rowptr, col = [], []
    for t in range(T):
        n = rng.choice(LENGTHS, N) if t else np.concatenate([rng.integers(1, 20, N - 50), rng.choice(LENGTHS, 50)])
        cj = [np.sort(np.append(rng.permutation(np.delete(np.arange(N), i))[:n[i] - 1], i)) for i in range(N)]
        rowptr.append(np.concatenate([[0], np.cumsum(n)]).astype(np.int64))
        col.append(np.concatenate(cj).astype(np.int32))
    X, C = (rng.standard_normal((T, N, F)).astype(np.float32) for _ in range(2))
    lo, hi = 200, 659
    layer = binding.DgcLayer([torch.from_numpy(r).cuda() for r in rowptr], [torch.from_numpy(c).cuda() for c in col], N,
                             [(lo, hi, 0, T)], F=F, S=32, H=32, time_kind="none", rows_per_group=rows_per_group, long_nnz=long_nnz,
                             part_nnz=part_nnz)
    ld = (F + 3) // 4 * 4
    dX, dC = (torch.zeros((T, N, ld), device="cuda")[:, :, :F].copy_(torch.from_numpy(a)) for a in (X, C))
    M = torch.full((T * (hi - lo), (F + 7) // 8 * 8), np.nan, device="cuda")
    layer.aggregate(dX, dC, M)
    torch.cuda.synchronize()
    got = M.cpu().numpy().reshape(T, hi - lo, -1)[:, :, :F]
    for t in range(T):
        n = np.diff(rowptr[t])
        d = 1.0 / np.sqrt(n.astype(np.float64))
        for i in range(lo, hi):
            j = col[t][rowptr[t][i]:rowptr[t][i + 1]]
            src = np.where(((j >= lo) & (j < hi))[:, None], X[t, j], C[t, j]).astype(np.float64)
            terms = d[i] * d[j][:, None] * src
            bound = (n[i] + 3) * 2.0 ** -24 * np.abs(terms).sum(0)
            assert (np.abs(got[t, i - lo] - terms.sum(0)) <= bound).all(), (t, i, n[i])
    layer.destroy()


@pytest.mark.parametrize("F", [64, 128, 256])
def test_shared_rows_of_an_input_gradient(F):
    """Neighbours outside the chunk left out, rows written through a row map."""
    import torch
    from paper_2309_03523_amd.runner import DeviceWorkload
    T, N = 2, 420
    wl = synth.random_small(70 + F, T, N, F, F, F, 5.0, [[0, 180, 0, 2], [180, 420, 0, 2]], "none", hub=True)
    assert max(int(np.diff(s.rowptr).max()) for s in wl.graph.snaps) > 128
    wl.params = synth.evolve_params(70 + F, F, F, random_bias=True)
    target = synth.stream(F, "target").standard_normal((T, N, F)).astype(np.float32)
    dw = DeviceWorkload(wl, struct_kind="evolve_gcn_o", act_out="relu")
    Y = dw.forward()
    dX = torch.full((T, N, F), np.nan, device="cuda")
    dw.layer.backward(Y, target=torch.from_numpy(target).cuda(), dX=dX)
    torch.cuda.synchronize()
    want = oracle.evolve(wl.graph, wl.chunks, wl.params, wl.X, wl.C, target, want_grads=True, want_dx=True)
    assert rel_err(Y.cpu().numpy(), want["Y"]) < 1e-4 and rel_err(dX.cpu().numpy(), want["dX"]) < 1e-4
    dw.layer.destroy()


@pytest.mark.parametrize("F", [40, 128, 190])
def test_shared_rows_of_absent_vertices(F):
    """Rows that nobody wants are skipped, the others go to their lanes."""
    import torch
    from oracle import tfusion
    from paper_2309_03523_amd.runner import DeviceWorkload
    T, N = 3, 300
    wl = synth.random_small(90 + F, T, N, F, 64, 64, 5.0, [[0, 300, 0, 3]], "gru", hub=True)
    assert max(int(np.diff(s.rowptr).max()) for s in wl.graph.snaps) > 128
    present = (synth.stream(F, "presence").random((T, N)) < 0.6).astype(np.uint8)
    hub = int(np.argmax(np.diff(wl.graph.snaps[0].rowptr)))
    present[:, hub] = [1, 0, 1]
    dw = DeviceWorkload(wl)
    dw.layer.set_presence(torch.from_numpy(present).cuda())
    Y = dw.forward(use_h0=False).cpu().numpy()
    Z = oracle.forward(wl.graph, wl.chunks, wl.params, wl.X, wl.C, time_kind="none").astype(np.float64)
    want = tfusion.run_separate(np.nan_to_num(Z), present, wl.chunks, wl.params, "gru")
    assert rel_err(Y[present != 0], want[present != 0]) < 1e-4
    dw.layer.destroy()
