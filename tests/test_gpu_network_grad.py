"""GPU tests of the convolution weight gradient: every form of its tiling against FP64 sums."""

import ctypes as C

import numpy as np
import pytest
import torch

from oracle import net as onet
from paper_1708_01663_amd import _lib
from synth import complex_normal, mixed_2d

pytestmark = pytest.mark.gpu


def _p(t):
    return C.c_void_p(t.data_ptr())


# (B, H, W, Ci, Co, max_splits): one strip narrower than 16 pixels, a cut last
# strip, heights that are no multiple of a batch of rows or of a task, several
# channel pairs, one split and more splits than tasks
@pytest.mark.parametrize("B,H,W,Ci,Co,splits", [
    (1, 1, 1, 32, 32, 1), (2, 5, 8, 32, 64, 4), (1, 13, 12, 96, 32, 64), (3, 7, 33, 64, 32, 2),
    (2, 35, 16, 32, 32, 300), (1, 64, 48, 32, 96, 7)])
def test_weight_gradient_tiling(B, H, W, Ci, Co, splits):
    g = torch.Generator().manual_seed(B * 1000 + H * 10 + W)
    x = torch.randn(B, H, W, Ci, generator=g).bfloat16()
    dy = torch.randn(B, H, W, Co, generator=g).bfloat16()
    xd = torch.nn.functional.pad(x.double(), (0, 0, 1, 1, 1, 1))
    want = torch.stack([
        torch.tensordot(dy.double(), xd[:, t // 3:t // 3 + H, t % 3:t % 3 + W], dims=([0, 1, 2], [0, 1, 2]))
        for t in range(9)])                                     # [9][Co][Ci]
    dw = torch.full((9, Co, Ci), float("nan"), device="cuda")
    scratch = torch.full((splits * 9 * Co * Ci,), float("nan"), device="cuda")
    xg, dyg = x.cuda(), dy.cuda()
    print(f"wgrad {B} {H} {W} {Ci} {Co} {splits}", flush=True)
    rc = _lib.load().cisor_nn_conv3x3_wgrad(_p(xg), _p(dyg), _p(dw), _p(scratch), B, H, W, Ci, Co, splits,
                                            C.c_void_p(torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    assert rc == 0
    # exact products summed in FP32: N terms of order one, error about sqrt(N) ulp of the sum
    tol = 2.0 ** -23 * (B * H * W) ** 0.5 * 8 * max(1.0, (B * H * W) ** 0.5)
    assert float((dw.cpu().double() - want).abs().max()) <= tol


def test_weight_gradient_of_an_image_past_32_bit_offsets():
    """More than 2^32 elements an image; only its first and last rows are not zero, and whole numbers, so
    that every order of the sums gives the same."""
    H, W, C_ = 8196, 16400, 32
    assert H * W * C_ > 2 ** 32
    print(f"wgrad {H} {W} {C_}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(5)
    x = torch.zeros(1, H, W, C_, dtype=torch.bfloat16, device="cuda")
    dy = torch.zeros_like(x)
    for t in (x, dy):
        for rows in (slice(0, 3), slice(H - 3, H)):
            t[:, rows] = torch.randint(-1, 2, (1, 3, W, C_), generator=g, device="cuda").bfloat16()
    want = torch.zeros(9, C_, C_, dtype=torch.float64, device="cuda")
    for rows in (slice(0, 4), slice(H - 4, H)):           # the fourth row is zero
        xs, ds = x[0, rows].double(), dy[0, rows].double()
        xp = torch.nn.functional.pad(xs, (0, 0, 1, 1, 1, 1))
        for t in range(9):
            want[t] += ds.reshape(-1, C_).T @ xp[t // 3:t // 3 + 4, t % 3:t % 3 + W].reshape(-1, C_)
    dw = torch.full((9, C_, C_), float("nan"), device="cuda")
    scratch = torch.empty(256 * 9 * C_ * C_, device="cuda")
    rc = _lib.load().cisor_nn_conv3x3_wgrad(_p(x), _p(dy), _p(dw), _p(scratch), 1, H, W, C_, C_, 256,
                                            C.c_void_p(torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    assert rc == 0
    assert torch.equal(dw.double(), want)


# every layer's weights and biases by themselves, the concatenated inputs' among them, at a size whose
# deep levels are narrower than a strip too.  The bar is twice what rounding activations, gradients and
# weights to BF16 does to the FP64 reference (up to 0.05, in the middle layers)
@pytest.mark.parametrize("n,B,seed", [(64, 8, 0), (32, 8, 1)])
def test_every_layers_gradient_matches_fp64(n, B, seed):
    from paper_1708_01663_amd.warmstart import WarmStartNet
    net = WarmStartNet(n, n, 32, max_batch=B, seed=3)
    rng = np.random.default_rng(seed)
    p = net.params().cpu().numpy()
    off = 0
    for ci, co, _ in onet.layer_specs(32):
        off += 9 * ci * co
        p[off:off + co] = 0.05 * rng.standard_normal(co)
        off += co
    net.set_params(p)
    f = np.stack([mixed_2d(n, seed + i).ravel() for i in range(B)])
    ax = (np.arange(n) - (n - 1) / 2) * 0.1
    th = 2 * np.pi * rng.uniform(size=B)[:, None, None]
    uin = np.exp(2j * np.pi * (np.cos(th) * ax[:, None] + np.sin(th) * ax[None])).reshape(B, -1)
    u, ub = uin * (1 + 0.3 * f) + 0.2j * f, 0.3 * complex_normal(uin.shape, 9)
    dev = lambda a, t: torch.as_tensor(a).to(t).cuda()
    c64 = torch.complex64
    _, g = net.loss_grad(dev(f, torch.float32), dev(uin, c64), dev(u, c64), u_born=dev(ub, c64))
    _, want = onet.loss_and_grad(p, f, uin, u, n, n, u_born=ub)
    g, off = g.cpu().numpy(), 0
    for i, (ci, co, _) in enumerate(onet.layer_specs(32)):
        for k in (9 * ci * co, co):
            a, b = g[off:off + k], want[off:off + k]
            assert np.linalg.norm(a - b) <= 0.1 * np.linalg.norm(b), (i, k)
            off += k
