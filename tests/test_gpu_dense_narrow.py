"""The narrow time encoder (S = H of 32 and 64) where it can go wrong: input widths around 16, 32 and the k-blocks that a wave
requests ahead, chunks that leave part of a 16-vertex tile or its second half empty, windows of one step, several tiles a
workgroup with windows of different lengths, masks, sequences, and rows of infinities.  Against the oracle in double; the bar for
the root mean square distance is what the fp32 instruction's kernel is off by at these sizes (3e-7: rounded sums of the products
and the gates' fast exponentials), for the largest element the repository's fp32 one."""
import numpy as np
import pytest

import oracle
from refs import rel_err
from workloads import synth

pytestmark = pytest.mark.gpu

WIDTHS = [1, 4, 15, 16, 17, 31, 32, 33, 48, 50, 64, 65, 96, 128, 129, 200, 256, 257]


def _check(wl, kind, H, windows, seed, mask=None):
    import torch
    from paper_2309_03523_amd.runner import DeviceWorkload
    V = int(sum(c[1] - c[0] for c in wl.chunks))
    n = 2 if kind == "lstm" else 1
    H0 = (0.5 * synth.stream(seed, "h0").standard_normal((n * V, H))).astype(np.float32)
    dw = DeviceWorkload(wl)
    dw.H0 = torch.from_numpy(H0).cuda()
    kw = {} if mask is None else dict(reset_mask=torch.from_numpy(mask).cuda())
    dw.Y.fill_(float("nan"))
    HN = torch.full_like(dw.H0, float("nan"))
    dw.layer.forward(dw.X, dw.C, dw.Y, C1=dw.C1, H0=dw.H0, HN=HN, **kw)
    torch.cuda.synchronize()
    want = oracle.forward(wl.graph, wl.chunks, wl.params, wl.X, wl.C, time_kind=kind, H0=H0, reset_mask=mask)
    want = np.asarray(want, np.float64)
    got = dw.Y.cpu().numpy()
    here = ~np.isnan(want)
    assert np.array_equal(np.isnan(got), ~here)
    off = np.linalg.norm((got - want)[here]) / np.linalg.norm(want[here])
    assert off < 3e-7 and rel_err(got[here], want[here]) < 1e-4, off
    row = 0
    hn = HN.cpu().numpy()
    for lo, hi, t0, t1 in wl.chunks:        # the state after the window is the last output
        np.testing.assert_array_equal(hn[row:row + hi - lo], got[t1 - 1, lo:hi])
        row += hi - lo
    dw.layer.destroy()


@pytest.mark.parametrize("F", WIDTHS)
@pytest.mark.parametrize("H", [32, 64])
@pytest.mark.parametrize("kind", ["gru", "lstm"])
def test_input_widths(F, H, kind):
    chunks = [[0, 15, 0, 4], [15, 31, 0, 1], [15, 31, 1, 4], [31, 48, 0, 4], [48, 81, 0, 2], [48, 81, 2, 4], [81, 82, 0, 3]]
    wl = synth.random_small(F + H, 4, 82, F, H, H, 4.0, chunks, kind)
    _check(wl, kind, H, chunks, F + H)


@pytest.mark.parametrize("H", [32, 64])
@pytest.mark.parametrize("kind", ["gru", "lstm"])
def test_many_tiles_and_masks(H, kind):
    """More half tiles than workgroups; windows of 1, 2 and 3."""
    n, T = 48, 6
    rng = synth.stream(H, "bounds")
    N = 24000
    cut = np.concatenate([[0], np.sort(rng.choice(N - 1, n - 1, replace=False)) + 1, [N]])
    chunks = []
    for i in range(n):
        chunks += [[int(cut[i]), int(cut[i + 1]), t, t + w] for t, w in ([(0, 1), (1, 2), (3, 3)] if i % 2 else [(0, 3), (3, 2), (5, 1)])]
    chunks = [c for c in chunks if (c[2] + c[0]) % 7]         # some vertices are not covered there
    wl = synth.random_small(H, T, N, 20, H, H, 2.0, chunks, kind)
    mask = (rng.random((T, N)) < 0.3).astype(np.uint8)
    _check(wl, kind, H, chunks, H, mask)


@pytest.mark.parametrize("H", [32, 64])
def test_infinities(H):
    """A row with an infinity: the other rows of its tile and their states stay what they are.  The lanes beside it cut their
    numbers into parts where they round them otherwise, which leaves out up to 2^-21 of a product (the sums of products that feed a
    gate are below 4 here and a gate's slope is at most 1): 4 * 2^-21 in an output, and other snapshots' bits are the same."""
    import torch
    from paper_2309_03523_amd.runner import DeviceWorkload
    wl = synth.random_small(H, 3, 40, 24, H, H, 0.0, [[0, 40, 0, 3]], "gru")      # no edges: a row sees itself
    out = []
    for x in (1.0, np.inf):
        wl.X[1, 5, 7] = x
        dw = DeviceWorkload(wl)
        out.append(dw.forward(use_h0=False).cpu().numpy())
        dw.layer.destroy()
    other = np.arange(40) != 5
    assert np.abs(out[0][:, other] - out[1][:, other]).max() <= 2.0 ** -19
    np.testing.assert_array_equal(out[0][0], out[1][0])
    assert np.isnan(out[1][1:, 5]).any()
