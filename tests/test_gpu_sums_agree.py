"""One window and a sequence table that says the same: labels that never change make every vertex one sequence of the
whole window, so the layer over labels and the layer over the one chunk do the same products.  They add them in the
same order, too: outputs and states have the same bits, in every variant of the split time encoder.  And how far a second
recurrent layer's sums are off double precision."""
import numpy as np
import pytest

from workloads import synth

pytestmark = pytest.mark.gpu

CASES = [  # F, S, time encoder, GCN layers, concatenated input, recurrent layers
    (40, 32, "gru", 1, False, 1),
    (16, 64, "lstm", 1, False, 1),
    (300, 160, "gru", 1, False, 1),
    (172, 128, "lstm", 2, True, 1),
    (40, 128, "gru", 2, False, 2),
    (33, 64, "lstm", 1, False, 2),
    (40, 128, "lstm", 2, True, 2),
]


@pytest.mark.parametrize("F,S,kind,layers,concat,recurrent", CASES)
def test_sequence_table_adds_like_the_window(F, S, kind, layers, concat, recurrent):
    import torch
    from paper_2309_03523_amd.runner import DeviceWorkload
    T, N = 6, 140
    wl = synth.random_small(F + S, T, N, F, S, S, 4.0, [[0, N, 0, T]], kind, layers, hub=True)
    wl.params = synth.layer_params(F + S, F, S, S, kind, layers, random_bias=True, input_concat=concat, n_time_layers=recurrent)
    wl.notes["input_concat"] = concat
    blocks = (2 if kind == "lstm" else 1) * recurrent
    H0 = (0.5 * synth.stream(S, "h0").standard_normal((blocks, N, S))).astype(np.float32)
    window = DeviceWorkload(wl, n_time_layers=recurrent)
    window.H0 = torch.from_numpy(H0.reshape(blocks * N, S)).cuda()
    Y, HN = window.forward(want_state=True)
    table = DeviceWorkload(wl, n_time_layers=recurrent)
    table.layer.set_labels(torch.zeros(T * N, dtype=torch.int32, device="cuda"))
    Hc = torch.zeros((blocks, T, N, S), device="cuda")
    Hc[:, 0] = torch.from_numpy(H0).cuda()
    HNt = torch.full_like(Hc, float("nan"))
    table.layer.forward(table.X, table.C, table.Y, C1=table.C1, H0=Hc.view(-1, S), HN=HNt.view(-1, S))
    torch.cuda.synchronize()
    assert torch.equal(table.Y, Y)
    assert torch.equal(HNt[:, T - 1], HN.view(blocks, N, S))
    window.layer.destroy()
    table.layer.destroy()


def _two_layers(wl, T, N, S):
    """The last layer's output [T, N, S] in double precision: no edges, no states."""
    p = {k: v.astype(np.float64) for k, v in wl.params.items()}
    z = wl.X.astype(np.float64) @ p["gcn0.weight"].T + p["gcn0.bias"]
    sigmoid = lambda x: 1.0 / (1.0 + np.exp(-x))
    state = [[np.zeros((N, S)), np.zeros((N, S))] for _ in range(2)]
    out = []
    for t in range(T):
        x = z[t]
        for layer, name in enumerate(("rnn", "rnn1")):
            h, c = state[layer]
            gi = x @ p[name + ".weight_ih"].T + p[name + ".bias_ih"]
            gh = h @ p[name + ".weight_hh"].T + p[name + ".bias_hh"]
            if wl.time_kind == "lstm":
                i, f, g, o = np.split(gi + gh, 4, axis=1)
                c = sigmoid(f) * c + sigmoid(i) * np.tanh(g)
                h = sigmoid(o) * np.tanh(c)
            else:
                (ir, iz, i_n), (hr, hz, hn) = np.split(gi, 3, axis=1), np.split(gh, 3, axis=1)
                u = sigmoid(iz + hz)
                h = (1 - u) * np.tanh(i_n + sigmoid(ir + hr) * hn) + u * h
            state[layer] = [h, c]
            x = h
        out.append(x)
    return np.stack(out)


@pytest.mark.parametrize("kind,bar", [("lstm", 2.3e-7), ("gru", 1.7e-7)])
def test_second_layer_rounding(kind, bar):
    """Root mean square distance from double precision over 8 x 512 rows, width 128.  On the fp32 instruction the layer was
    at 2.1e-7 (LSTM) and 1.9e-7 (GRU), most of it the gates' fast exponentials; with the small part products of the second
    layer's gates in one sum with the large ones it is at 2.5e-7 and 1.9e-7, with sums of their own at 2.1e-7 and 1.5e-7.
    The bars lie between."""
    from paper_2309_03523_amd.runner import DeviceWorkload
    T, N, S = 8, 512, 128
    wl = synth.random_small(3, T, N, S, S, S, 0.0, [[0, N, 0, T]], kind)     # no edges: a row sees itself
    wl.params = synth.layer_params(3, S, S, S, kind, 1, random_bias=True, n_time_layers=2)
    dw = DeviceWorkload(wl, n_time_layers=2)
    Y = dw.forward(use_h0=False).cpu().numpy()
    want = _two_layers(wl, T, N, S)
    off = float(np.linalg.norm(Y - want) / np.linalg.norm(want))
    print(f"{kind}: {off:.2e}", flush=True)
    assert off < bar
    dw.layer.destroy()
