"""The time encoders' products on two half-precision parts, and what leaves their range: an operand that is too large, a weight
matrix that is too large or too small, a bias that the scale of the sums does not hold.  From that step on (for such weights
and biases from the first) the tile runs on three bf16 parts; the oracle's results hold on either side, in the state, too.

The bar: root mean square distance over the output's root mean square.  With all part products a time encoder is within
3e-7 (its gates), with one of the three half products left out 1e-4, with a sum in the wrong scale 1; the bar is 1e-6."""
import numpy as np
import pytest

import oracle
from workloads import synth

pytestmark = pytest.mark.gpu

CHUNKS = [[0, 33, 0, 6], [33, 70, 0, 3], [33, 70, 3, 6], [70, 135, 1, 6]]
SHAPES = [  # F, S, cell, GCN layers, recurrent layers, concatenated input, activation after the transform
    (40, 64, "gru", 1, 1, False, "none"),
    (128, 128, "gru", 1, 1, False, "relu"),
    (300, 256, "gru", 1, 1, False, "none"),
    (128, 128, "gru", 1, 2, False, "none"),
    (70, 96, "lstm", 1, 1, False, "none"),
    (128, 128, "lstm", 2, 2, True, "none"),
    (250, 128, "lstm", 2, 1, True, "relu"),
]


def _large_rows(wl):
    wl.X[2:, 40:80:9] *= np.float32(3e3)
    wl.C[4:] *= np.float32(700.0)


ROWS = int(sum(c[1] - c[0] for c in CHUNKS))


def _large_state(wl):
    wl.H0[3:ROWS:7] *= np.float32(4e3)


def _large_weight(wl):
    wl.params["rnn.weight_hh"][5, 3] = 40.0


def _small_weights(wl):
    wl.params["rnn.weight_ih"] *= np.float32(1e-4)


def _large_bias(wl):
    wl.params["rnn.bias_ih"][7] = 1e31


CHANGES = {"none": lambda wl: None, "rows": _large_rows, "state": _large_state, "weight": _large_weight,
           "weights": _small_weights, "bias": _large_bias}


def _problem(shape, change):
    F, S, cell, gcn, rnn, concat, act = shape
    wl = synth.random_small(F + S + gcn, 6, 140, F, S, S, 4.0, CHUNKS, cell, gcn, input_concat=concat)
    wl.params = synth.layer_params(F + S + gcn, F, S, S, cell, gcn, random_bias=True, input_concat=concat, n_time_layers=rnn)
    n = rnn * (2 if cell == "lstm" else 1)
    wl.H0 = (0.5 * synth.stream(F, "halves").standard_normal((n * ROWS, S))).astype(np.float32)
    CHANGES[change](wl)
    return wl


@pytest.mark.parametrize("change", list(CHANGES))
@pytest.mark.parametrize("shape", SHAPES)
def test_halves_and_beyond(shape, change):
    import torch
    from paper_2309_03523_amd.runner import DeviceWorkload
    F, S, cell, gcn, rnn, concat, act = shape
    wl = _problem(shape, change)
    dw = DeviceWorkload(wl, n_time_layers=rnn, act_hidden="relu", act_out=act)
    dw.H0 = torch.from_numpy(wl.H0).cuda()
    Y, HN = (x.cpu().numpy() for x in dw.forward(want_state=True))
    dw.layer.destroy()
    want, want_HN = oracle.forward(wl.graph, wl.chunks, wl.params, wl.X, wl.C, time_kind=cell, n_struct_layers=gcn, C1=wl.C1,
                                   H0=wl.H0, return_state=True, n_time_layers=rnn, input_concat=concat, act_hidden="relu", act_out=act)
    m = ~np.isnan(want)
    assert np.array_equal(np.isnan(Y), ~m)
    if change == "state":       # gates of arguments of 2000 are 2000 times as far off in fp32: those rows are looked at by themselves
        changed, row = np.zeros(want.shape[:2], bool), 0
        for lo, hi, t0, t1 in CHUNKS:
            changed[t0:t1, lo:hi] = (np.arange(row, row + hi - lo) % 7 == 3)
            row += hi - lo
        state = np.tile(np.arange(ROWS) % 7 == 3, len(HN) // ROWS)
        parts = [("Y", Y[m[..., 0] & ~changed], want[m[..., 0] & ~changed], 1e-6), ("HN", HN[~state], want_HN[~state], 1e-6),
                 ("Y of such a state", Y[m[..., 0] & changed], want[m[..., 0] & changed], 2e-4),
                 ("HN of such a state", HN[state], want_HN[state], 2e-4)]
    else:
        bar = 5e-6 if change == "rows" else 1e-6       # (some rows' gates have arguments of 1000 and more, and their error)
        parts = [("Y", Y[m], want[m], bar), ("HN", HN, want_HN, bar)]
    for name, got, ref, bar in parts:
        off = float(np.linalg.norm(got.astype(np.float64) - ref) / np.linalg.norm(ref.astype(np.float64)))
        print(f"{shape} {change}: {name} {off:.2e}", flush=True)
        assert off < bar


@pytest.mark.parametrize("cell", ["gru", "lstm"])
def test_small_inputs_keep_their_place(cell):
    """Inputs of 1e-3 and states of 1e-5 beside each other, no bias: what the halves lose of a number (2^-31) is lost of sums of
    1e-4, over 128 columns of weights of 0.1: 4e-10 x 0.1 x 11 = 5e-10 in the mean, 1e-5 of an output at most."""
    from paper_2309_03523_amd.runner import DeviceWorkload
    wl = synth.random_small(5, 4, 70, 128, 128, 128, 4.0, [[0, 70, 0, 4]], cell)
    for k in wl.params:
        if "bias" in k:
            wl.params[k] = np.zeros_like(wl.params[k])
    wl.X *= np.float32(1e-3)
    wl.C *= np.float32(1e-3)
    wl.H0 = wl.H0 * np.float32(1e-5)
    dw = DeviceWorkload(wl, n_time_layers=1, act_out="relu")
    Y = dw.forward().cpu().numpy().astype(np.float64)
    dw.layer.destroy()
    want = oracle.forward(wl.graph, wl.chunks, wl.params, wl.X, wl.C, time_kind=cell, H0=wl.H0, act_out="relu").astype(np.float64)
    off = np.linalg.norm(Y - want) / np.linalg.norm(want)
    print(f"{cell}: {off:.2e}", flush=True)
    assert off < 1e-5
