"""Graph attention rows that a wave takes four at a time (groups of four rows and more), beside rows that it takes alone, that a
workgroup shares and that are split: the row lengths and the bar of the other row tests, groups that end inside four."""
import pytest

from test_gpu_attention_rows import test_row_lengths as _row_lengths

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,N,cut,kw", [
    (2, 160, 80, dict(rows_per_group=4)), (2, 161, 97, dict(rows_per_group=5)), (1, 191, 30, dict(rows_per_group=7)),
    (2, 192, 64, dict(rows_per_group=16, long_nnz=16, part_nnz=16)), (2, 193, 100, dict(rows_per_group=6, long_nnz=40, part_nnz=17)),
    (1, 160, 33, dict(rows_per_group=32, long_nnz=64, part_nnz=65)), (2, 163, 3, dict(rows_per_group=3)),
])
def test_slots(T, N, cut, kw):
    _row_lengths(T, N, cut, kw)


@pytest.mark.parametrize("N", [700, 2500, 6000])
def test_default_groups(N):
    """The work list is what the header says: groups of 16 rows, halved while there are fewer than 8192 of them."""
    import oracle
    from paper_2309_03523_amd.runner import DysatDevice
    from workloads import synth
    T = 6
    wl = synth.dysat_small(5, T, N, 128, 8, 3.0, [[0, N // 3, 0, T], [N // 3, N, 0, T]])
    rows = 16
    while rows > 1 and T * N // rows < 8192:
        rows //= 2
    dd = DysatDevice(wl)
    want = oracle.worklist(wl.graph, wl.chunks, rows, 1024, 512)["work_short"]
    assert dd.layer.packing("work_short").tolist() == [list(x) for x in want]
    dd.layer.destroy()


@pytest.mark.parametrize("rows", [1, 3, 4, 8])
def test_rows_that_store_nothing(rows):
    """A vertex without so much as a self-loop, which only validate_level = 1 refuses: its row is zero whatever group it is in."""
    import numpy as np
    from paper_2309_03523_amd.runner import DysatDevice
    from workloads import synth
    T, N = 2, 160
    wl = synth.dysat_small(8, T, N, 128, 8, 3.0, [[0, 60, 0, T], [60, N, 0, T]])
    out = []
    for empty in (False, True):
        if empty:
            for s in wl.graph.snaps:          # of a vertex that is its own only neighbour
                alone = int(np.nonzero(np.diff(s.rowptr) == 1)[0][0])
                s.col = np.delete(s.col, s.rowptr[alone])
                s.rowptr[alone + 1:] -= 1
        dd = DysatDevice(wl, rows_per_group=rows)
        out.append(dd.forward().float().cpu().numpy())
        dd.layer.destroy()
        if not empty:
            lone = [int(np.nonzero(np.diff(s.rowptr) == 1)[0][0]) for s in wl.graph.snaps]
    assert np.isfinite(out[1]).all()
    others = [i for i in range(N) if i not in lone]
    np.testing.assert_array_equal(out[0][:, others], out[1][:, others])
