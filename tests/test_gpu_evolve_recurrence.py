"""The weight recurrence of the EvolveGCN-O path and its back-propagation at every width, seen by themselves: vertex i holds
the i-th unit vector and sees only itself, so row i of snapshot t is row i of relu(W_t) and the gradient of W_t is the
gradient of the positive outputs, both without a rounding but the one to fp32.  Reference: float64 autograd on the recurrence.
The kernels compute it in double, so an output is off by half a unit in the last place (2^-24 of itself) at most, and a gradient
by that in every element: the bars are twice that for the one, and 4e-8 in the root mean square for the other (uniform roundings
of normalised fp32 numbers give 2.5e-8 to 3.4e-8)."""
import numpy as np
import pytest

from workloads import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("F", [32, 64, 96, 128, 160, 192, 224, 256])
@pytest.mark.parametrize("T", [1, 2, 9])
def test_weight_recurrence(F, T):
    import torch
    from paper_2309_03523_amd.runner import DeviceWorkload
    wl = synth.random_small(F + T, T, F, F, F, F, 0.0, [[0, F, 0, T]], "none")
    wl.X[:] = np.eye(F, dtype=np.float32)
    wl.params = synth.evolve_params(F + T, F, F, random_bias=True)
    dY = synth.stream(F + T, "upstream").standard_normal((T, F, F)).astype(np.float32)
    dw = DeviceWorkload(wl, struct_kind="evolve_gcn_o", act_out="relu")
    Y = dw.forward()
    dw.layer.backward(Y, dY=torch.from_numpy(dY).cuda())
    torch.cuda.synchronize()
    P = {k: torch.from_numpy(np.asarray(v, np.float64)).requires_grad_() for k, v in wl.params.items()}
    p = {k.split(".")[1]: v for k, v in P.items()}
    W, loss = p["W_init"], 0.0
    got = Y.cpu().numpy()
    for t in range(T):
        z = torch.sigmoid(p["U_z"] @ W + p["V_z"] @ W + p["B_z"])
        r = torch.sigmoid(p["U_r"] @ W + p["V_r"] @ W + p["B_r"])
        c = torch.tanh(p["U_h"] @ W + p["V_h"] @ (r * W) + p["B_h"])
        W = (1 - z) * W + z * c
        want = torch.relu(W).detach().numpy()
        assert (np.abs(got[t] - want) <= 2.0 ** -23 * np.abs(want)).all(), t
        loss = loss + (W * torch.from_numpy(dY[t].astype(np.float64)) * torch.from_numpy(got[t] > 0)).sum()
    loss.backward()
    for k, v in P.items():
        g, w = dw.layer.get_param(k + ".grad", v.shape), v.grad.numpy()
        assert np.linalg.norm(g - w) <= 4e-8 * np.linalg.norm(w), k
    dw.layer.destroy()
