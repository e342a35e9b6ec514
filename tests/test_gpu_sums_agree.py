"""One window and a sequence table that says the same: labels that never change make every vertex one sequence of the
whole window, so the layer over labels and the layer over the one chunk do the same products.  They add them in the
same order, too: outputs and states have the same bits, in every variant of the split time encoder."""
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
