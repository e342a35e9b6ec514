"""Rows of the graph attention that the four waves of a workgroup share: lengths around the threshold (128) and where a quarter
ends inside a batch or is shorter than the others, whole and as parts of split rows, several in one group and in one workgroup; short parts, few (shared)
and more than the chip holds workgroups (one a wave).
Rows of more than 128 neighbours average as many projections, so the bar is the layer's bf16 one relative to the root mean
square of the row looked at."""
import numpy as np
import pytest

from oracle import dysat
from refs import rel_err
from workloads import synth

pytestmark = pytest.mark.gpu

TOL = 2e-2
LENGTHS = [128, 129, 130, 131, 132, 133, 160, 191, 192, 193, 255, 256, 257, 258, 319, 320, 321, 400, 511, 512, 513, 600]


@pytest.mark.parametrize("T,N,cut,kw", [
    (2, 700, 11, {}), (1, 701, 350, dict(rows_per_group=32)), (1, 689, 5, dict(rows_per_group=1)),
    (1, 700, 20, dict(long_nnz=300, part_nnz=131, rows_per_group=8)), (2, 693, 400, dict(long_nnz=130, part_nnz=3)),
    (1, 693, 400, dict(long_nnz=130, part_nnz=40)),
])
def test_shared_rows(T, N, cut, kw):
    from paper_2309_03523_amd.runner import DysatDevice
    wl = synth.dysat_small(N, T, N, 128, 8, 3.0, [[0, cut, 0, T], [cut, N, 0, T]])
    k = len(LENGTHS)
    for t in range(T):
        rng = synth.stream(N + t, "rows")
        leaves = [rng.choice(N - k, size=n - 1, replace=False) + k for n in LENGTHS]
        u = np.concatenate([np.full(len(x), i) for i, x in enumerate(leaves)])
        wl.graph.snaps[t] = synth.csr_from_undirected(N, u, np.concatenate(leaves))
        assert np.diff(wl.graph.snaps[t].rowptr)[:k].tolist() == LENGTHS
    dd = DysatDevice(wl, validate_level=1, **kw)
    got = dd.forward().float().cpu().numpy()
    want = dysat.gradients(wl.graph, wl.chunks, wl.params, wl.X, wl.C, 8, dY=np.zeros_like(wl.X))["Y"]
    for i in range(k):
        assert rel_err(got[:, i], want[:, i], floor=1.0) < TOL, LENGTHS[i]
    assert rel_err(got, want, floor=1.0) < TOL
    dd.layer.destroy()


@pytest.mark.parametrize("first", [16, 64, 120, 180])
@pytest.mark.parametrize("kw", [{}, dict(long_nnz=130, part_nnz=50)])
def test_neighbours_of_weight_zero(first, kw):
    """A run of neighbours whose logits are below every float (their projections are finite) has weight zero wherever it lies in a
    shared or split row, also where it fills the first of a wave's batches; a row of nothing but such neighbours is NaN."""
    from paper_2309_03523_amd.runner import DysatDevice
    T, N, n = 2, 300, 240
    wl = synth.dysat_small(4, T, N, 128, 8, 3.0, [[0, N, 0, T]])
    for t in range(T):                                   # vertex 0: neighbours 0 .. n; the others see it and themselves
        wl.graph.snaps[t] = synth.csr_from_undirected(N, np.zeros(n, np.int64), np.arange(1, n + 1))
    wl.params["gat.weight"] = np.eye(128, dtype=np.float32)
    wl.params["gat.att_src"] = np.full((8, 16), -1e35, np.float32)
    wl.params["gat.att_dst"] = np.zeros((8, 16), np.float32)
    wl.X[:, first:first + 50] = 1e4                      # logits beyond the largest float
    wl.X[:, n + 2:] = 1e4                                # see only themselves (and n + 1 shares a tile with one of them)
    dd = DysatDevice(wl, **kw)
    got = dd.forward().float().cpu().numpy()
    dd.layer.destroy()
    assert np.isnan(got[:, n + 2:]).all() and np.isfinite(got[:, :n + 1]).all()
    want = dysat.gradients(wl.graph, wl.chunks, wl.params, wl.X, wl.C, 8, dY=np.zeros_like(wl.X))["Y"]
    assert rel_err(got[:, 0], want[:, 0], floor=1.0) < TOL
