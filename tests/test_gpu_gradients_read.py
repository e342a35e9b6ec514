"""Gradients are read right after the backward that makes them, without a synchronisation by the caller: every read waits for the
work on the default stream, also the first one and those of parameters that the backward writes last, and returns what a read after
a synchronisation returns."""
import numpy as np
import pytest

from workloads import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["evolve", "attention"])
def test_read_without_synchronising(kind):
    import torch
    from paper_2309_03523_amd.runner import DeviceWorkload, DysatDevice
    T, N = 8, 6000
    if kind == "evolve":
        wl = synth.random_small(5, T, N, 128, 128, 128, 4.0, [[0, N, 0, T]], "none", hub=True)
        wl.params = synth.evolve_params(5, 128, 128, random_bias=True)
        dw = DeviceWorkload(wl, struct_kind="evolve_gcn_o", act_out="relu")
    else:
        wl = synth.dysat_small(5, T, N, 128, 8, 4.0, [[0, N, 0, T]])
        dw = DysatDevice(wl)
    names = [n + ".grad" for n in wl.params]
    assert all((dw.layer.get_param(n, wl.params[n[:-5]].shape) == 0).all() for n in names)      # before any backward
    before = None
    for turn in range(3):
        dY = torch.randn((T, N, 128), device="cuda").to(dw.Y.dtype)
        dw.layer.forward(dw.X, dw.C, dw.Y)
        dw.layer.backward(dw.Y, dY=dY)
        first = {n: dw.layer.get_param(n, wl.params[n[:-5]].shape) for n in (names if turn % 2 else names[::-1])}
        torch.cuda.synchronize()
        for n in names:
            np.testing.assert_array_equal(first[n], dw.layer.get_param(n, wl.params[n[:-5]].shape))
            assert before is None or not np.array_equal(first[n], before[n])
        before = first
    dw.layer.destroy()
