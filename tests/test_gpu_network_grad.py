"""GPU tests of the convolution weight gradient: every form of its tiling against FP64 sums."""

import ctypes as C

import pytest
import torch

from paper_1708_01663_amd import _lib

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
