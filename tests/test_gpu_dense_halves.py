"""The time encoders' products on two half-precision parts, and what leaves their range: an operand that is too large, a weight
matrix whose rows are too long (and one that is all small, which does not), a bias that the scale of the sums does not hold.  From that step on (for such weights
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


def _edge_of_the_range(wl):
    """The largest state that the halves hold, and the next number that they do not."""
    wl.H0[2, 5], wl.H0[40, 9], wl.H0[41, 9] = 31.98, 32.0, -31.98


def _large_weight(wl):
    wl.params["rnn.weight_hh"][5, 3] = 40.0


def _small_weights(wl):
    wl.params["rnn.weight_ih"] *= np.float32(1e-4)


def _large_bias(wl):
    wl.params["rnn.bias_ih"][7] = 1e31


CHANGES = {"none": lambda wl: None, "rows": _large_rows, "state": _large_state, "edge": _edge_of_the_range, "weight": _large_weight,
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


def _without_biases(cell, F, seed, scale):
    """A layer without biases over inputs of `scale` and states of a hundredth of that."""
    wl = synth.random_small(seed, 4, 70, F, 128, 128, 4.0, [[0, 70, 0, 4]], cell)
    for k in wl.params:
        if "bias" in k:
            wl.params[k] = np.zeros_like(wl.params[k])
    wl.X *= np.float32(scale)
    wl.C *= np.float32(scale)
    wl.H0 = wl.H0 * np.float32(0.01 * scale)
    return wl


def _distance(wl, cell):
    """Of the outputs from the layer in double, and what 1 - 2 / (1 + e^2x) in fp32 alone is off by: 2^-25 in the mean, of outputs
    that are a product of one such number and a gate of 1/2."""
    from paper_2309_03523_amd.runner import DeviceWorkload
    dw = DeviceWorkload(wl, n_time_layers=1)
    Y = dw.forward().cpu().numpy().astype(np.float64)
    dw.layer.destroy()
    want = _double(wl, cell)
    size = np.sqrt(np.mean(want ** 2))
    return np.linalg.norm(Y - want) / np.linalg.norm(want), 0.5 * 2.0 ** -25 / size


def _double(wl, cell):
    """A GCN layer and a recurrent one over one chunk of all vertices, in double (the oracle's gates are single)."""
    p = {k: v.astype(np.float64) for k, v in wl.params.items()}
    T, N, F = wl.X.shape
    h = wl.H0[:N].astype(np.float64)
    c = wl.H0[N:].astype(np.float64) if cell == "lstm" else None
    sig = lambda x: 1.0 / (1.0 + np.exp(-x))
    out = []
    for t, s in enumerate(wl.graph.snaps):
        n = np.diff(s.rowptr)
        row = np.repeat(np.arange(N), n)
        m = np.zeros((N, F))
        np.add.at(m, row, (1.0 / np.sqrt(n[row] * n[s.col]))[:, None] * wl.X[t].astype(np.float64)[s.col])
        z = m @ p["gcn0.weight"].T + p["gcn0.bias"]
        gi, gh = z @ p["rnn.weight_ih"].T + p["rnn.bias_ih"], h @ p["rnn.weight_hh"].T + p["rnn.bias_hh"]
        if cell == "gru":
            (ir, iz, i_n), (hr, hz, hn) = np.split(gi, 3, 1), np.split(gh, 3, 1)
            u = sig(iz + hz)
            h = (1.0 - u) * np.tanh(i_n + sig(ir + hr) * hn) + u * h
        else:
            i, f, g, o = np.split(gi + gh, 4, 1)
            c = sig(f) * c + sig(i) * np.tanh(g)
            h = sig(o) * np.tanh(c)
        out.append(h)
    return np.stack(out)


@pytest.mark.parametrize("scale", [1.0, 1e-3, 1e-5, 1e-7, 1e-10])
@pytest.mark.parametrize("F", [128, 300])                  # the transform folded, and not
@pytest.mark.parametrize("cell", ["gru", "lstm"])
def test_small_inputs(cell, F, scale):
    """What the halves lose of a small number (2^-37 of an input or a state, in sums over weights of 0.06 to 0.1) is less than a five-hundredth of
    what the plain formula for tanh loses of its value; besides that an output has the errors of any other."""
    off, plain = _distance(_without_biases(cell, F, F, scale), cell)
    print(f"{cell} {F}, inputs of {scale}: {off:.2e}, the formula alone {plain:.2e}", flush=True)
    assert off < 1e-6 + plain / 512


@pytest.mark.parametrize("scale", [1e-5, 1e-7])
@pytest.mark.parametrize("factor", [8.0, 30.0])
@pytest.mark.parametrize("F", [128, 300])
@pytest.mark.parametrize("cell", ["gru", "lstm"])
def test_large_weights_and_small_inputs(cell, F, factor, scale):
    """Weights of 0.5 to 0.8 and of 2 to 3 (whose rows are too long for the halves): what is lost of an input is multiplied twice where the
    transform is not folded, and still no more than what the formula alone loses."""
    wl = _without_biases(cell, F, F, scale)
    for k in ("gcn0.weight", "rnn.weight_ih", "rnn.weight_hh"):
        wl.params[k] = wl.params[k] * np.float32(factor)
    off, plain = _distance(wl, cell)
    print(f"{cell} {F}, weights times {factor}, inputs of {scale}: {off:.2e}, the formula alone {plain:.2e}", flush=True)
    assert off < 1e-6 + 2 * plain


@pytest.mark.parametrize("cell,rows", [("gru", slice(256, 384)), ("lstm", slice(256, 384))])
def test_rows_of_small_weights(cell, rows):
    """The gate that makes the output has weights a millionth of the others': 2^-38 of each is lost, over inputs of 1."""
    wl = _without_biases(cell, 300, 7, 1.0)
    for k in ("rnn.weight_ih", "rnn.weight_hh"):
        wl.params[k][rows] *= np.float32(1e-6)
    wl.H0 *= np.float32(0.0)
    off, plain = _distance(wl, cell)
    print(f"{cell}: {off:.2e}, the formula alone {plain:.2e}", flush=True)
    assert off < 1e-6 + plain / 16
