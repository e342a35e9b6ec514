"""The input gradient of EvolveGCN-O where its transform takes two and three times as many runs of tiles as fit the chip, with a
last tile of one row: every vertex sees only itself, so a row of dX is the positive outputs' upstream row by the transpose of
that snapshot's weights.  Reference: float64, the weights' recurrence included.  Four times as many runs: the 64 x 62 500 case of
the full-size tests.  Bars: the fp32 products' 4e-7 in the root mean square distance, and for the largest error 2^-20 of the
largest value (256 products of fp32 accuracy, summed in fp32 in blocks of 16)."""
import numpy as np
import pytest

from workloads import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("F,T,N", [(256, 2, 131072), (256, 3, 131041), (128, 3, 174785)])
def test_runs_of_tiles(F, T, N):
    import torch
    from paper_2309_03523_amd.runner import DeviceWorkload
    wl = synth.random_small(F, T, N, F, F, F, 0.0, [[0, N, 0, T]], "none")
    wl.params = synth.evolve_params(F, F, F, random_bias=True)
    dw = DeviceWorkload(wl, struct_kind="evolve_gcn_o", act_out="relu")
    Y = dw.forward()
    dY = torch.randn(T, N, F, device="cuda", generator=torch.Generator("cuda").manual_seed(N))
    dX = torch.full_like(dY, float("nan"))
    dw.layer.backward(Y, dY=dY, dX=dX)
    torch.cuda.synchronize()
    p = {k.split(".")[1]: torch.from_numpy(np.asarray(v, np.float64)) for k, v in wl.params.items()}
    W = p["W_init"]
    for t in range(T):
        z = torch.sigmoid(p["U_z"] @ W + p["V_z"] @ W + p["B_z"])
        r = torch.sigmoid(p["U_r"] @ W + p["V_r"] @ W + p["B_r"])
        c = torch.tanh(p["U_h"] @ W + p["V_h"] @ (r * W) + p["B_h"])
        W = (1 - z) * W + z * c
        want = (dY[t] * (Y[t] > 0)).double() @ W.t().contiguous().cuda()
        off = dX[t].double() - want
        assert off.norm() <= 4e-7 * want.norm(), t
        assert off.abs().max() <= 2.0 ** -20 * want.abs().max(), t
    dw.layer.destroy()
