"""The transform folded into the time encoder's input side: input widths on both sides of where folding pays (and beyond one
staging buffer), one and two GCN layers, the concatenated input, an activation that forbids it, parameters that change or come in
another order, and weights and inputs that are not finite.  Against the oracle in double: the repository's fp32 bar for the
largest error, and 4e-7 for the root mean square distance (the fp32 instruction's kernel is at 3e-7 for GRUs and 4e-7 for LSTMs of
four steps: the gates' fast exponentials and the products' rounded sums)."""
import numpy as np
import pytest

import oracle
from refs import rel_err
from workloads import synth

pytestmark = pytest.mark.gpu

CHUNKS = [[0, 33, 0, 4], [33, 70, 0, 1], [33, 70, 1, 4]]


def _close(got, want):
    want = np.asarray(want, np.float64)
    assert np.array_equal(np.isnan(got), np.isnan(want))
    m = ~np.isnan(want)
    off = np.linalg.norm((got - want)[m]) / np.linalg.norm(want[m])
    assert off < 4e-7 and rel_err(got[m], want[m]) < 1e-4, off


def _oracle(wl, kind, layers=1, **kw):
    return oracle.forward(wl.graph, wl.chunks, wl.params, wl.X, wl.C, time_kind=kind, n_struct_layers=layers, C1=wl.C1, H0=wl.H0, **kw)


@pytest.mark.parametrize("F,S,kind,layers", [
    (1, 96, "gru", 1), (96, 96, "lstm", 1), (128, 96, "lstm", 1), (129, 96, "lstm", 1), (144, 96, "gru", 1), (145, 96, "gru", 1),
    (97, 128, "gru", 1), (192, 128, "gru", 1), (193, 128, "gru", 1), (40, 128, "lstm", 2), (300, 256, "gru", 1), (304, 256, "lstm", 1),
    (272, 192, "gru", 1), (273, 192, "gru", 1), (257, 224, "lstm", 1), (60, 160, "gru", 2), (97, 96, "lstm", 1), (128, 128, "lstm", 1),
    (129, 128, "lstm", 1), (288, 224, "lstm", 1), (208, 160, "lstm", 1),
])
def test_widths(F, S, kind, layers):
    from paper_2309_03523_amd.runner import run_forward
    wl = synth.random_small(F + S, 4, 70, F, S, S, 4.0, CHUNKS, kind, layers)
    _close(run_forward(wl), _oracle(wl, kind, layers))


@pytest.mark.parametrize("act_out", ["none", "relu"])
@pytest.mark.parametrize("concat", [False, True])
def test_concatenated_input_and_activation(act_out, concat):
    from paper_2309_03523_amd.runner import run_forward
    wl = synth.random_small(7, 4, 70, 50, 128, 128, 4.0, CHUNKS, "lstm", 2, input_concat=concat)
    wl.notes["input_concat"] = concat
    _close(run_forward(wl, act_out=act_out), _oracle(wl, "lstm", 2, act_out=act_out, input_concat=concat))


def test_parameters_change():
    """Each of the folded parameters by itself, after a forward; and before all of them are there."""
    from paper_2309_03523_amd.runner import DeviceWorkload
    wl = synth.random_small(9, 4, 70, 128, 128, 128, 4.0, CHUNKS, "gru")
    other = synth.random_small(10, 4, 70, 128, 128, 128, 4.0, CHUNKS, "gru").params
    dw = DeviceWorkload(wl)
    _close(dw.forward().cpu().numpy(), _oracle(wl, "gru"))
    for name in ("rnn.bias_ih", "gcn0.weight", "rnn.weight_ih", "gcn0.bias", "rnn.weight_hh"):
        wl.params[name] = other[name]
        dw.layer.set_param(name, other[name])
        _close(dw.forward().cpu().numpy(), _oracle(wl, "gru"))
    dw.layer.destroy()


def test_parameters_change_under_a_captured_forward():
    """A graph captured before the parameters change replays with the ones that are set."""
    import torch
    from paper_2309_03523_amd.runner import DeviceWorkload
    wl = synth.random_small(13, 4, 70, 96, 96, 96, 4.0, CHUNKS, "lstm")
    other = synth.random_small(14, 4, 70, 96, 96, 96, 4.0, CHUNKS, "lstm").params
    dw = DeviceWorkload(wl)
    dw.forward()
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        dw.layer.forward(dw.X, dw.C, dw.Y, C1=dw.C1, H0=dw.H0)
    for name in wl.params:
        wl.params[name] = other[name]
        dw.layer.set_param(name, other[name])
        eager = dw.forward().clone()
        dw.Y.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(torch.nan_to_num(dw.Y, nan=-7.0), torch.nan_to_num(eager, nan=-7.0)), name
    _close(dw.Y.cpu().numpy(), _oracle(wl, "lstm"))
    # then weights whose product overflows (the transformed rows do not), and the ones before again
    for scale, inputs in ((1e20, 1e-25), (1e-20, 1e25)):
        for name in ("gcn0.weight", "rnn.weight_ih"):
            wl.params[name] = wl.params[name] * np.float32(scale)
            dw.layer.set_param(name, wl.params[name])
        dw.X *= inputs
        dw.C *= inputs
        eager = dw.forward().clone()
        dw.Y.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        covered = ~torch.isnan(eager)
        assert covered.any() and torch.equal(dw.Y[covered], eager[covered]) and torch.equal(covered, ~torch.isnan(dw.Y))
    dw.layer.destroy()


def test_parameters_never_set():
    from paper_2309_03523_amd import binding
    from paper_2309_03523_amd.runner import DeviceWorkload
    wl = synth.random_small(11, 4, 70, 128, 128, 128, 4.0, CHUNKS, "gru")
    wl.params["gcn0.bias"][:] = 0.0
    names = [n for n in wl.params if n != "gcn0.bias"]       # the bias stays the zero it is
    set_params = binding.DgcLayer.set_params
    try:
        binding.DgcLayer.set_params = lambda self, params: [self.set_param(n, params[n]) for n in names[::-1]]
        dw = DeviceWorkload(wl)
    finally:
        binding.DgcLayer.set_params = set_params
    _close(dw.forward().cpu().numpy(), _oracle(wl, "gru"))
    dw.layer.destroy()


def test_not_finite():
    """An infinite or missing input makes NaN of its own rows' outputs from there on, as the transform's infinities of either sign
    do, and of no other's; weights whose product overflows are not folded."""
    from paper_2309_03523_amd.runner import DeviceWorkload, run_forward
    wl = synth.random_small(12, 3, 40, 128, 128, 128, 0.0, [[0, 40, 0, 3]], "gru")      # no edges: a row sees itself
    wl.X[1, 5, 7], wl.X[0, 6, 0], wl.X[2, 39, 127] = np.inf, np.nan, -np.inf
    Y = run_forward(wl)
    nan = np.zeros((3, 40), bool)
    nan[1:, 5] = nan[:, 6] = nan[2, 39] = True
    assert np.array_equal(np.isnan(Y).all(axis=2), nan) and np.array_equal(np.isnan(Y).any(axis=2), nan)
    keep = np.arange(40)[~nan.any(axis=0)]
    wl.X[~np.isfinite(wl.X)] = 1.0
    want = _oracle(wl, "gru")
    assert rel_err(Y[:, keep], want[:, keep]) < 1e-4
    # products of the weights above the largest float; the transformed rows themselves stay below it
    wl.params["gcn0.weight"] *= np.float32(1e20)
    wl.params["rnn.weight_ih"] *= np.float32(1e20)
    wl.X *= np.float32(1e-25)
    wl.C *= np.float32(1e-25)
    dw = DeviceWorkload(wl)
    Y = dw.forward().cpu().numpy()
    dw.layer.destroy()
    want = _oracle(wl, "gru")
    assert np.isfinite(Y).all() and np.abs(Y - want).mean() < 1e-4


@pytest.mark.parametrize("kind", ["gru", "lstm"])
@pytest.mark.parametrize("sign", [1, -1])
def test_infinite_inputs_of_weights_of_one_sign(kind, sign):
    """Weights whose products have one sign saturate the gates for an infinite input, and the outputs are finite: the oracle's."""
    from paper_2309_03523_amd.runner import run_forward
    wl = synth.random_small(15, 3, 40, 128, 128, 128, 0.0, [[0, 40, 0, 3]], kind)      # no edges: a row sees itself
    wl.params["gcn0.weight"] = np.maximum(np.abs(wl.params["gcn0.weight"]), np.float32(1e-3))
    wl.params["rnn.weight_ih"] = sign * np.maximum(np.abs(wl.params["rnn.weight_ih"]), np.float32(1e-3))
    wl.X[1, 5, 7], wl.X[2, 9, 0] = np.inf, -np.inf
    got = run_forward(wl)
    assert np.isfinite(got).all()
    assert rel_err(got, _oracle(wl, kind)) < 1e-4


def test_products_below_the_split_range():
    """Weights whose products are below 2^-110 are not folded: their parts would be lost, where the transformed rows keep them."""
    from paper_2309_03523_amd.runner import run_forward
    wl = synth.random_small(16, 4, 70, 128, 128, 128, 4.0, CHUNKS, "gru")
    for name in ("gcn0.weight", "rnn.weight_ih"):
        wl.params[name] = wl.params[name] * np.float32(2.0 ** -60)
    wl.params["gcn0.bias"] = wl.params["gcn0.bias"] * np.float32(2.0 ** 60)
    wl.X *= np.float32(2.0 ** 120)
    wl.C *= np.float32(2.0 ** 120)
    _close(run_forward(wl), _oracle(wl, "gru"))
