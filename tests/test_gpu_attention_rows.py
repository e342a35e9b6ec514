"""The passes of the graph attention over a row's non-zeros (forward, row pass, reverse-edge pass) at the row lengths
where they can go wrong: around a batch of neighbours, two batches, the 64 column ids that a wave loads at once, and
the parts of split rows; and the projections and the input gradient at vertex counts around a tile.  The bar is the
layer's bf16 one, taken relative to the root mean square of the rows looked at, so that a neighbour left out or taken
twice shows (one of 130 changes a row by about a tenth of it)."""
import numpy as np
import pytest

from oracle import dysat
from refs import rel_err
from workloads import synth

pytestmark = pytest.mark.gpu

TOL = 2e-2
LENGTHS = [1, 2, 4, 8, 9, 15, 16, 17, 31, 32, 33, 48, 63, 64, 65, 79, 80, 127, 128, 129, 130]


def _graph(T, N, seed):
    """Vertex i < len(LENGTHS) has a row of LENGTHS[i] non-zeros, the self-loop counted; the rest are their leaves."""
    snaps, k = [], len(LENGTHS)
    for t in range(T):
        rng = synth.stream(seed + t, "rows")
        leaves = [rng.choice(N - k, size=n - 1, replace=False) + k for n in LENGTHS]
        u = np.concatenate([np.full(len(x), i) for i, x in enumerate(leaves)])
        snaps.append(synth.csr_from_undirected(N, u, np.concatenate(leaves)))
        assert np.diff(snaps[-1].rowptr)[:k].tolist() == LENGTHS
    return snaps


@pytest.mark.parametrize("T,N,cut,kw", [
    (2, 160, 80, {}), (2, 161, 97, {}), (1, 191, 30, {}),
    (2, 192, 64, dict(long_nnz=16, part_nnz=16)), (2, 193, 100, dict(long_nnz=32, part_nnz=17)),
    (1, 160, 33, dict(long_nnz=64, part_nnz=65)), (2, 160, 21, dict(rows_per_group=32)),
])
def test_row_lengths(T, N, cut, kw):
    import torch
    from paper_2309_03523_amd.runner import DysatDevice
    wl = synth.dysat_small(N, T, N, 128, 8, 3.0, [[0, cut, 0, T], [cut, N, 0, T]])
    wl.graph.snaps[:] = _graph(T, N, N)
    up = synth.round_bf16(synth.stream(N, "up").standard_normal(wl.X.shape).astype(np.float32))
    dd = DysatDevice(wl, validate_level=1, **kw)
    got = dd.forward().float().cpu().numpy()
    want = dysat.gradients(wl.graph, wl.chunks, wl.params, wl.X, wl.C, 8, dY=up, want_dx=True)
    for i in range(len(LENGTHS)):
        assert rel_err(got[:, i], want["Y"][:, i], floor=1.0) < TOL, LENGTHS[i]
    assert rel_err(got, want["Y"], floor=1.0) < TOL
    dX = torch.empty((T, N, 128), device="cuda", dtype=torch.bfloat16)
    grads, _ = dd.backward(dY=torch.from_numpy(up).cuda().to(torch.bfloat16), dX=dX)
    for name in dysat.PARAMS:
        assert rel_err(grads[name], want["grads"][name], floor=1.0) < TOL, name
    # a row's gradient against its own norm: the rows differ by more than 10x (a leaf of one hub, a hub of 130 leaves),
    # and each of the stored intermediates (dQ, dK, dV, dU, dz, dX) adds a bf16 rounding of 1.1e-3 RMS to it
    g, w = dX.float().cpu().numpy().astype(np.float64), want["dX"]
    e = np.sqrt(((g - w) ** 2).mean(axis=2) / (w * w).mean(axis=2))
    print(f"dX max row error {e.max():.3e}", flush=True)
    assert e.max() < 1e-2
    dd.layer.destroy()
