"""Parameters that are set between an EvolveGCN-O forward and its backward: the gradients are those of the forward's parameters,
bit for bit, at widths whose matrices stay in registers and at those that are streamed; also of a forward that a graph replays."""
import numpy as np
import pytest

from workloads import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("F", [32, 64, 96, 128, 256])
@pytest.mark.parametrize("want_dx", [False, True])
def test_gradients_of_the_forwards_parameters(F, want_dx):
    import torch
    from paper_2309_03523_amd.runner import DeviceWorkload
    T, N = 3, 70
    wl = synth.random_small(F, T, N, F, F, F, 4.0, [[0, 33, 0, T], [33, N, 0, T]], "none")
    wl.params = synth.evolve_params(F, F, F, random_bias=True)
    other = synth.evolve_params(F + 1, F, F, random_bias=True)
    dw = DeviceWorkload(wl, struct_kind="evolve_gcn_o", act_out="relu")
    dY = torch.from_numpy(synth.stream(F, "upstream").standard_normal((T, N, F)).astype(np.float32)).cuda()

    def gradients():
        dX = torch.zeros((T, N, F), device="cuda") if want_dx else None
        dw.layer.backward(dw.Y, dY=dY, dX=dX)
        torch.cuda.synchronize()
        out = {k: dw.layer.get_param(k + ".grad", v.shape) for k, v in wl.params.items()}
        if want_dx:
            out["dX"] = dX.cpu().numpy()
        return out

    def same(a, b):
        for k in a:
            np.testing.assert_array_equal(a[k], b[k], err_msg=k)

    dw.forward()
    want = gradients()
    dw.layer.set_params(other)
    if not want_dx:                    # a second backward of that forward
        same(gradients(), want)
    dw.forward()
    want_other = gradients()
    assert not np.array_equal(want["evolve.U_r"], want_other["evolve.U_r"])
    dw.layer.set_params(wl.params)
    dw.forward()
    dw.layer.set_params(other)
    same(gradients(), want)

    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
        dw.layer.forward(dw.X, dw.C, dw.Y)
    replays = ((wl.params, other, want), (other, wl.params, want_other))
    for now, then, expected in replays[:1 if want_dx else 2]:      # (a backward with dX uses up what the forward left)
        dw.layer.set_params(now)
        graph.replay()
        torch.cuda.synchronize()
        dw.layer.set_params(then)
        same(gradients(), expected)
    dw.layer.destroy()
