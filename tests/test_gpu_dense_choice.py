"""Layers 32 and 64 wide on either side of the sizes where the narrow kernel gives way to the one on halves, and LSTMs 96 and 128
wide whose transform's folding saves few products; windows of equal length, resets, chunks that leave the last tile part empty.
The oracle and the bars are those of the narrow kernel's tests and of the folded transform's (4e-7, LSTMs of several steps)."""
import numpy as np
import pytest

from refs import narrow_takes
from test_gpu_dense_fold import _close, _oracle
from test_gpu_dense_narrow import _check
from workloads import synth

pytestmark = pytest.mark.gpu


def _most(kind, H, F, window):
    """The most tiles of 32 vertices, up to 2048, that the narrow kernel takes."""
    few, many = 2, 2049
    while many - few > 1:
        n = (few + many) // 2
        few, many = (n, many) if narrow_takes(kind, H, F, n, window) else (few, n)
    return few


@pytest.mark.parametrize("over", [0, 1])
@pytest.mark.parametrize("kind,H,F,window", [
    ("gru", 32, 30, 2), ("lstm", 32, 17, 4), ("gru", 32, 40, 2), ("lstm", 32, 48, 3),
    ("gru", 64, 200, 1), ("lstm", 64, 33, 3), ("gru", 64, 64, 6), ("lstm", 64, 70, 4),
    ("gru", 64, 100, 2), ("lstm", 64, 130, 3), ("gru", 64, 150, 2)])
def test_either_side(kind, H, F, window, over):
    most = _most(kind, H, F, window)
    print(f"{kind} {H} wide, {F} columns, windows of {window}: {most} tiles", flush=True)
    T = 2 * window                             # two windows with half of the tiles each
    first, N = (most + over) // 2, most + over - (most + over) // 2
    N = 32 * N - 9
    chunks = [[0, 32 * first - 9, 0, window], [0, N, window, T]]
    wl = synth.random_small(F + window, T, N, F, H, H, 2.0, chunks, kind)
    _check(wl, kind, H, chunks, F, (synth.stream(F, "mask").random((T, N)) < 0.2).astype(np.uint8))


@pytest.mark.parametrize("F,S", [(97, 96), (112, 96), (130, 128), (160, 128), (161, 128)])
def test_few_products_saved(F, S):
    from paper_2309_03523_amd.runner import run_forward
    wl = synth.random_small(F + S, 4, 140, F, S, S, 4.0, [[0, 33, 0, 4], [33, 140, 0, 1], [33, 140, 1, 4]], "lstm")
    _close(run_forward(wl), _oracle(wl, "lstm"))
