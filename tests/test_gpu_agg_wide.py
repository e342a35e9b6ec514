"""The edge-table aggregation of rows wider than the 256 floats that a wave spans (two stretches of columns), with
split rows, against the oracle and against the column-walking kernels.  fp32 sums in another order: the
repository's fp32 bar."""
import numpy as np
import pytest

import oracle
from refs import rel_err
from workloads import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("F", [256, 257, 300, 320, 384, 512])
@pytest.mark.parametrize("long_nnz", [0, 12])
def test_wide_rows(F, long_nnz):
    from paper_2309_03523_amd.runner import run_forward
    chunks = synth.grid_chunks(3, 2, [np.asarray([0, 21, 70])] * 2)
    wl = synth.random_small(F, 3, 70, F, 64, 64, 6.0, chunks, "none", hub=True)
    want = oracle.forward(wl.graph, wl.chunks, wl.params, wl.X, wl.C, time_kind="none")
    got = {k: run_forward(wl, agg_kernel=k, long_nnz=long_nnz, part_nnz=5 if long_nnz else 0) for k in ("table", "walk")}
    for k in got:
        assert rel_err(got[k], want) < 1e-4, k
    assert rel_err(got["table"], got["walk"]) < 1e-4
