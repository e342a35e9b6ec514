"""The split dense kernels (fp32 products as sums of bf16 products) against the oracle, at the sizes where they can go
wrong: widths of one and of eight column blocks and those between, input widths that leave a part of the last
k-block (or of the second launch of a wide transform) empty, chunks that end inside a tile.  The oracle's products are
double; the bar is the repository's fp32 one."""
import numpy as np
import pytest

import oracle
from refs import rel_err
from workloads import synth

pytestmark = pytest.mark.gpu

CASES = [  # F, S, time encoder, GCN layers, chunk bounds over 70 vertices
    (1, 32, "gru", 1, (0, 1, 33, 70)),
    (17, 64, "lstm", 1, (0, 31, 63, 70)),
    (50, 96, "gru", 1, (0, 32, 70)),
    (96, 160, "lstm", 1, (0, 64, 70)),
    (128, 128, "gru", 2, (0, 33, 70)),
    (172, 128, "lstm", 2, (0, 70)),
    (250, 192, "gru", 1, (0, 7, 70)),
    (300, 256, "lstm", 1, (0, 70)),
    (500, 64, "gru", 1, (0, 70)),
    (3, 32, "none", 1, (0, 1, 33, 70)),
    (16, 96, "none", 2, (0, 31, 70)),
    (240, 256, "none", 1, (0, 65, 70)),
    (257, 128, "none", 1, (0, 70)),
    (500, 256, "none", 1, (0, 33, 70)),
]


@pytest.mark.parametrize("F,S,kind,layers,bounds", CASES)
def test_split_dense_shapes(F, S, kind, layers, bounds):
    from paper_2309_03523_amd.runner import run_forward
    chunks = synth.grid_chunks(5, 3, [np.asarray(bounds)] * 2)
    wl = synth.random_small(F + S, 5, 70, F, S, S, 4.0, chunks, kind, layers)
    Y = run_forward(wl)
    want = oracle.forward(wl.graph, wl.chunks, wl.params, wl.X, wl.C, time_kind=kind, C1=wl.C1, H0=wl.H0,
                          n_struct_layers=layers)
    assert rel_err(Y, want) < 1e-4


def test_split_dense_infinite_input():
    """An infinite input gives the infinities (and the NaN where opposite ones meet) that fp32 products give."""
    from paper_2309_03523_amd.runner import run_forward
    wl = synth.random_small(3, 2, 50, 40, 64, 64, 0.0, [[0, 50, 0, 2]], "none")     # no edges: a row sees itself
    wl.X[0, 5, 7] = np.inf
    wl.X[1, 33, 0] = -np.inf
    wl.X[1, 40, 39] = np.nan
    wl.X[0, 6, :2] = 3e38
    Y = run_forward(wl)
    with np.errstate(all="ignore"):
        want = (wl.X.astype(np.float64) @ wl.params["gcn0.weight"].astype(np.float64).T + wl.params["gcn0.bias"])
        want = want.astype(np.float32)
    assert np.array_equal(np.isnan(Y), np.isnan(want))
    assert np.array_equal(np.isposinf(Y), np.isposinf(want)) and np.array_equal(np.isneginf(Y), np.isneginf(want))
    keep = np.ones((2, 50), bool)
    keep[0, 5:7] = keep[1, 33] = keep[1, 40] = False
    assert rel_err(Y[keep], want[keep]) < 1e-4


def _same_specials(got, want):
    return (np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(np.isposinf(got), np.isposinf(want))
            and np.array_equal(np.isneginf(got), np.isneginf(want)))


def test_split_dense_infinite_weight():
    """Infinite weights against inputs whose lower parts are zero (1, 0, powers of two), against infinite inputs and
    against ordinary ones: the infinities of fp32 products, NaN only where they give it (infinity times zero,
    opposite infinities)."""
    from paper_2309_03523_amd.runner import run_forward
    wl = synth.random_small(4, 2, 50, 40, 64, 64, 0.0, [[0, 50, 0, 2]], "none")     # no edges: a row sees itself
    W = wl.params["gcn0.weight"]
    W[3, 7], W[40, 0], W[41, 0], W[41, 39] = np.inf, -np.inf, np.inf, np.inf
    wl.X[0, :, 7] = np.tile(np.float32([1.0, -1.0, 0.0, 2.0 ** -60, 0.3]), 10)
    wl.X[1, :, 0] = np.tile(np.float32([1.0, -2.0, np.inf, -np.inf, 3.0]), 10)
    wl.X[1, :5, 39] = np.float32([1.0, 1.0, 1.0, np.inf, -0.25])
    Y = run_forward(wl)
    with np.errstate(all="ignore"):
        want = (wl.X.astype(np.float64) @ W.astype(np.float64).T + wl.params["gcn0.bias"]).astype(np.float32)
    assert _same_specials(Y, want) and np.isnan(want).any() and np.isinf(want).any()
    finite = np.isfinite(want)
    assert rel_err(Y[finite], want[finite]) < 1e-4


@pytest.mark.parametrize("kind", ["gru", "lstm"])
def test_split_time_encoder_infinite_weight(kind):
    """An infinite gate weight saturates its gate whatever the bits of the state: no NaN that the oracle does not have."""
    from paper_2309_03523_amd.runner import run_forward
    wl = synth.random_small(5, 3, 40, 24, 32, 32, 0.0, [[0, 40, 0, 3]], kind)
    wl.H0[:, 4] = 1.0
    wl.H0[:, 9] = -0.5
    wl.params["rnn.weight_hh"][5, 4] = np.inf
    wl.params["rnn.weight_hh"][38, 9] = np.inf
    Y = run_forward(wl)
    with np.errstate(all="ignore"):
        want = oracle.forward(wl.graph, wl.chunks, wl.params, wl.X, wl.C, time_kind=kind, H0=wl.H0)
    assert np.isfinite(want).all()
    assert rel_err(Y, want) < 1e-4


@pytest.mark.parametrize("F,S", [(64, 64), (256, 256), (300, 96)])
def test_split_products_have_no_bias(F, S):
    """What the six bf16 products of an fp32 product leave out has either sign.  Parts that are cut off instead of rounded
    leave out 2^-24.5 of a term in the mean, always towards zero: 4e-8 of every sum.  Rounded ones leave the truncation of
    the matrix unit's additions (measured 6e-9) and noise of 1e-7 an element, over 1e5 elements less than 1e-9.  The bars:
    2e-8 for the mean, and for the root mean square 1.5e-7 (about one rounding of an fp32 sum; 1.2e-7 measured)."""
    from paper_2309_03523_amd.runner import run_forward
    N = 2000
    wl = synth.random_small(F, 1, N, F, S, S, 0.0, [[0, N, 0, 1]], "none")     # no edges: a row sees itself
    Y = run_forward(wl).astype(np.float64)
    want = wl.X.astype(np.float64) @ wl.params["gcn0.weight"].astype(np.float64).T + wl.params["gcn0.bias"].astype(np.float64)
    d = Y - want
    bias = float((d * np.sign(want)).sum() / np.abs(want).sum())
    rms = float(np.linalg.norm(d) / np.linalg.norm(want))
    print(f"F={F} S={S}: bias {bias:.2e}, rms {rms:.2e}", flush=True)
    assert abs(bias) < 2e-8 and rms < 1.5e-7


@pytest.mark.parametrize("F,S,kind,layers,bounds", CASES)
def test_split_dense_rounding(F, S, kind, layers, bounds):
    """Root mean square distance from the oracle's double products.  With all six part products a transform is up to 1.5e-7 off,
    a time encoder up to 3.3e-7 (its fast exponentials); a transform that leaves one of them out is 5e-6 off or more.  The
    bar between: 1e-6."""
    from paper_2309_03523_amd.runner import run_forward
    chunks = synth.grid_chunks(5, 3, [np.asarray(bounds)] * 2)
    wl = synth.random_small(F + S, 5, 70, F, S, S, 4.0, chunks, kind, layers)
    Y = run_forward(wl).astype(np.float64)
    want = oracle.forward(wl.graph, wl.chunks, wl.params, wl.X, wl.C, time_kind=kind, C1=wl.C1, H0=wl.H0,
                          n_struct_layers=layers).astype(np.float64)
    off = float(np.linalg.norm(Y - want) / np.linalg.norm(want))
    print(f"F={F} S={S} {kind} layers={layers}: {off:.2e}", flush=True)
    assert off < 1e-6
