"""The network's fused kernels where their tiling can go wrong, against the FP64
oracle: fields of one pixel and of a few (the 22 x 14 widened tile wraps many
times), exactly one widened tile, one more pixel than a tile in each
direction, every channel padding (3, 4, 5, 16, 17, 32), more tiles than the
forward pass has blocks, and weights at a 2-byte aligned address (no 16-byte
loads).  Tolerances as in test_cnn_gpu.py (a few hundred float32 operations per
output: 1e-5 of each tensor's scale).

The surrogate's training step against the separate calls it fuses (normalise,
forward, backward, Adam): the same sums in the same order, so equal bit for
bit; the loss is a float64 sum over another partition, rounded once.
"""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

from oracle import cnn as ocnn  # noqa: E402
from test_cnn_gpu import rel, setup  # noqa: E402


@pytest.fixture(scope="module")
def L():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1902_00530_amd as lib
    return lib


def _stream():
    return torch.cuda.current_stream().cuda_stream


def _run(L, g, shape, params, ws):
    """Activations, output, gradients and loss of one pass."""
    n, h, w = shape.n, shape.h, shape.w
    a1 = torch.empty((n, 32, h, w), device="cuda")
    a2 = torch.empty_like(a1)
    y = torch.empty((n, 3, h, w), device="cuda")
    L.lbm_cnn_forward(shape, params, g["x"].data_ptr(), a1.data_ptr(), a2.data_ptr(), y.data_ptr(), ws.data_ptr(),
                      ws.numel(), _stream())
    gw = [torch.empty(a.shape, device="cuda") for a in g["w"]]
    gb = [torch.empty(a.shape, device="cuda") for a in g["b"]]
    grads = L.lbm_cnn_grads((ctypes.c_void_p * 3)(*[a.data_ptr() for a in gw]),
                            (ctypes.c_void_p * 3)(*[a.data_ptr() for a in gb]))
    loss = torch.empty(1, device="cuda")
    L.lbm_cnn_backward(shape, params, g["x"].data_ptr(), a1.data_ptr(), a2.data_ptr(), y.data_ptr(),
                       g["t"].data_ptr(), grads, loss.data_ptr(), ws.data_ptr(), ws.numel(), _stream())
    return (a1, a2, y), [gw[0], gb[0], gw[1], gb[1], gw[2], gb[2]], loss


@pytest.mark.parametrize("n,cin,h,w,odd", [(2, 4, 1, 1, 0), (1, 3, 2, 5, 0), (1, 4, 14, 22, 0), (2, 5, 9, 17, 0),
                                           (1, 16, 8, 16, 0), (2, 17, 13, 21, 0), (1, 32, 3, 40, 0),
                                           (67, 4, 16, 20, 0), (2, 4, 11, 19, 1), (1, 7, 10, 18, 1)])
def test_forward_and_backward(L, n, cin, h, w, odd):
    x, t, p, g, shape, params, ws = setup(L, n=n, cin=cin, h=h, w=w, seed=n + cin)
    if odd:  # the same weights one element past an aligned address
        for k in range(3):
            room = torch.empty(g["w"][k].numel() + 1, dtype=torch.bfloat16, device="cuda")
            room[1:].copy_(g["w"][k].reshape(-1))
            g["w"][k] = room[1:].view(g["w"][k].shape)
        params = L.lbm_cnn_params((ctypes.c_void_p * 3)(*[a.data_ptr() for a in g["w"]]), params.b)
    acts, grads, loss = _run(L, g, shape, params, ws)
    for got, ref in zip(acts, ocnn.forward(x, p)):
        assert rel(got.double().cpu().numpy(), ref) < 1e-5
    rl, rg = ocnn.backward(x, p, t)
    assert abs(loss.item() - rl) < 1e-5 * rl
    for k in range(6):
        assert rel(grads[k].double().cpu().numpy(), rg[k]) < 1e-5, k


@pytest.mark.parametrize("cin,h,w", [(4, 20, 24), (3, 9, 7), (4, 32, 32)])
def test_training_step_equals_the_separate_calls(L, cin, h, w):
    from paper_1902_00530_amd import surrogate as S
    total, n = 40, 36  # 32 x 32: 288 tiles
    net = S.Surrogate(h, w, 2, 4, max_batch=n, cin=cin, seed=5)
    rng = torch.Generator(device="cuda").manual_seed(11)
    X = torch.randn((total, cin, h, w), generator=rng, device="cuda") * 0.3 + 1.0
    T = X + 0.1 * torch.randn((total, cin, h, w), generator=rng, device="cuda")
    idx = torch.randperm(total, generator=rng, device="cuda")[:n].to(torch.int32)
    net.fit_normalisation(X)
    v = L.lbm_surrogate_view_of(net.handle)

    def at(ptr, count, dt):
        o = ptr - net.params.data_ptr()
        return net.params[o:o + count * torch.tensor([], dtype=dt).element_size()].view(dt)

    th = [at(v.theta[k], v.count[k], torch.float32).clone() for k in range(6)]
    m = [at(v.m[k], v.count[k], torch.float32).clone() for k in range(6)]
    vv = [at(v.v[k], v.count[k], torch.float32).clone() for k in range(6)]
    wb = [at(v.w_bf16[k], v.count[2 * k], torch.bfloat16).clone() for k in range(3)]
    norm = at(v.norm, 4 * cin, torch.float32)
    xn, tn = X[idx.long()].clone(), T[idx.long()].clone()
    for a in (xn, tn):
        L.lbm_channel_affine(a.data_ptr(), n, cin, cin, h * w, norm.data_ptr(), norm[cin:].data_ptr(), _stream())
    shape = L.lbm_cnn_shape(n, cin, 32, 3, h, w)
    params = L.lbm_cnn_params((ctypes.c_void_p * 3)(*[a.data_ptr() for a in wb]),
                              (ctypes.c_void_p * 3)(*[th[k].data_ptr() for k in (1, 3, 5)]))
    g = dict(x=xn, t=tn[:, :3].contiguous(), w=wb, b=[th[k] for k in (1, 3, 5)])
    ws = torch.empty(L.lbm_cnn_workspace_bytes(shape), dtype=torch.uint8, device="cuda")
    _, grads, ref_loss = _run(L, g, shape, params, ws)
    for k in range(6):
        L.lbm_cnn_adam(th[k].data_ptr(), m[k].data_ptr(), vv[k].data_ptr(), grads[k].data_ptr(), th[k].numel(), 1e-3,
                       0.9, 0.999, 1e-8, 1, wb[k // 2].data_ptr() if k % 2 == 0 else None, _stream())
    loss = net.train_step(X, T, idx, 1e-3)
    assert abs(loss.item() - ref_loss.item()) <= 2.0 ** -23 * abs(ref_loss.item())
    for k in range(6):
        for got, ref in ((v.theta[k], th[k]), (v.m[k], m[k]), (v.v[k], vv[k])):
            assert torch.equal(at(got, v.count[k], torch.float32), ref), k
    for k in range(3):
        assert torch.equal(at(v.w_bf16[k], v.count[2 * k], torch.bfloat16), wb[k]), k
    net.close()
