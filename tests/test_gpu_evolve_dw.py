"""The split weight-gradient kernel of the EvolveGCN-O path at the sizes where it can go wrong: every number of column
blocks, chunks of rows that leave part of a 16-row step or a whole one empty, a snapshot without rows, one workgroup
and many a snapshot; both upstream forms, with and without the input gradient.  The oracle's products are double; the
bar is the repository's fp32 one.  The parameter gradients do not depend on whether the input gradient is asked for:
the same bits."""
import numpy as np
import pytest

import oracle
from refs import rel_err
from workloads import synth

pytestmark = pytest.mark.gpu

CASES = [  # F, snapshots, vertices, chunks
    (32, 1, 1, [[0, 1, 0, 1]]),
    (32, 3, 300, [[0, 300, 0, 3]]),
    (64, 2, 80, [[0, 15, 0, 2], [15, 31, 0, 2], [31, 48, 0, 2], [48, 79, 0, 2]]),
    (96, 3, 66, [[0, 33, 0, 1], [33, 66, 0, 1], [0, 66, 2, 3]]),
    (128, 2, 100, [[0, 17, 0, 2], [17, 49, 0, 2], [49, 100, 1, 2]]),
    (160, 1, 40, [[0, 40, 0, 1]]),
    (192, 2, 33, [[0, 33, 0, 2]]),
    (224, 3, 20, [[0, 16, 0, 3], [16, 20, 0, 2]]),
    (256, 2, 400, [[0, 31, 0, 2], [31, 400, 0, 2]]),
]


@pytest.mark.parametrize("F,T,N,chunks", CASES)
@pytest.mark.parametrize("upstream", ["target", "dY"])
def test_weight_gradient_shapes(F, T, N, chunks, upstream):
    import torch
    from paper_2309_03523_amd.runner import DeviceWorkload
    wl = synth.random_small(40 + F, T, N, F, F, F, 4.0, chunks, "none", hub=True)
    wl.params = synth.evolve_params(40 + F, F, F, random_bias=True)
    target = synth.stream(F, "target").standard_normal((T, N, F)).astype(np.float32)
    dw = DeviceWorkload(wl, struct_kind="evolve_gcn_o", act_out="relu")
    Y = dw.forward()
    want = oracle.evolve(wl.graph, wl.chunks, wl.params, wl.X, wl.C, target, want_grads=True, want_dx=True)
    tgt = torch.from_numpy(target).cuda()
    up = dict(target=tgt) if upstream == "target" else dict(dY=(2.0 * (Y - tgt) / float(wl.rows * F)).contiguous())

    def grads():
        torch.cuda.synchronize()
        return {k: dw.layer.get_param(k + ".grad", wl.params[k].shape) for k in oracle.EVOLVE_PARAMS}

    dw.layer.backward(Y, **up)
    alone = grads()
    dX = torch.zeros((T, N, F), device="cuda")
    dw.layer.backward(Y, dX=dX, **up)
    beside = grads()
    covered = ~np.isnan(want["Y"]).any(axis=2)
    assert rel_err(dX.cpu().numpy()[covered], want["dX"][covered]) < 1e-4
    for k in oracle.EVOLVE_PARAMS:
        assert rel_err(alone[k], want["grads"][k]) < 1e-4, k
        assert np.array_equal(alone[k], beside[k]), k
    dw.layer.destroy()


def test_weight_gradient_infinite_rows():
    """An infinite row element against upstream gradients of 1 (whose lower parts are zero): the weight gradient has the
    infinities that fp32 products give, and NaN only where they do (infinity times a gradient that is zero).  One
    snapshot: the bias gradients are dL/dW times positive factors, element by element."""
    import torch
    from paper_2309_03523_amd.runner import DeviceWorkload
    F, N = 64, 40
    wl = synth.random_small(9, 1, N, F, F, F, 0.0, [[0, N, 0, 1]], "none")     # no edges: a row sees itself
    wl.params = synth.evolve_params(9, F, F, random_bias=True)
    wl.X[0, 3, 5], wl.X[0, 20, 7], wl.X[0, 21, 7] = np.inf, -np.inf, 2.0
    dw = DeviceWorkload(wl, struct_kind="evolve_gcn_o", act_out="relu")
    Y = dw.forward()
    dY = torch.ones((1, N, F), device="cuda")
    dw.layer.backward(Y, dY=dY)
    torch.cuda.synchronize()
    got = dw.layer.get_param("evolve.B_h.grad", (F, F))
    with np.errstate(all="ignore"):
        d = (Y.cpu().numpy()[0] > 0).astype(np.float64)
        want = wl.X[0].astype(np.float64).T @ d
    for special in (np.isnan, np.isposinf, np.isneginf):
        assert np.array_equal(special(got), special(want))
    assert np.isinf(want).any() and np.isnan(want).any()
    dw.layer.destroy()


def test_weight_gradient_rounding():
    """Distance of the ten gradients from double precision, root mean square.  The recurrence runs in double and the number
    of elements is a power of two, so what is left is the rounding of the gradient itself (3.4e-8 at most in the mean) and
    of the sums over 4096 rows a snapshot, which are kept below that.  The bar is 6e-8; sums that drop a part of the
    products, or add their small parts to the large ones, are at 8e-8 to 1.2e-7."""
    import torch
    from paper_2309_03523_amd.runner import DeviceWorkload
    T, N, F = 4, 4096, 64
    wl = synth.random_small(11, T, N, F, F, F, 4.0, [[0, N, 0, T]], "none")
    wl.params = synth.evolve_params(11, F, F, random_bias=True)
    target = synth.stream(F, "target").standard_normal((T, N, F)).astype(np.float32)
    dw = DeviceWorkload(wl, struct_kind="evolve_gcn_o", act_out="relu")
    Y = dw.forward()
    dw.layer.backward(Y, target=torch.from_numpy(target).cuda())
    torch.cuda.synchronize()
    want = oracle.evolve(wl.graph, wl.chunks, wl.params, wl.X, wl.C, target, want_grads=True)
    off = {}
    for k in oracle.EVOLVE_PARAMS:
        w = np.asarray(want["grads"][k], np.float64)
        off[k] = float(np.linalg.norm(dw.layer.get_param(k + ".grad", wl.params[k].shape) - w) / np.linalg.norm(w))
    print({k: f"{v:.2e}" for k, v in off.items()}, flush=True)
    assert max(off.values()) < 6e-8
    dw.layer.destroy()
