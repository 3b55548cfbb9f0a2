"""GPU tests of the TV prox at the edges of its launches: image sides around the one-block limit
and tile multiples, iteration counts around a launch's share, outputs that overlap the input."""

import ctypes as C

import numpy as np
import pytest
import torch

from oracle import tv as otv
from paper_1708_01663_amd import _lib

pytestmark = pytest.mark.gpu

# FP32: each of the iterations rounds values of order one; FP64 likewise
BAR = {0: 1e-5, 1: 1e-10}


def prox(dim, n, prec, z, x, lam, iters):
    s = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    code = _lib.load().cisor_tv_prox_noalloc(dim, n, prec, C.c_void_p(z.data_ptr()), C.c_void_p(x.data_ptr()), lam,
                                             0.0, 1.5, iters, s)
    assert code == 0


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("dim,n,iters", [
    (2, 2, 5), (2, 16, 1), (2, 31, 119), (2, 32, 120), (2, 32, 121), (2, 32, 245), (2, 33, 1), (2, 33, 7), (2, 33, 8),
    (2, 40, 9), (2, 48, 16), (2, 49, 100), (3, 2, 1), (3, 3, 2), (3, 17, 9), (3, 33, 40)])
def test_prox_at_launch_edges(dim, n, iters, prec):
    print(f"tv {dim}D n {n} iterations {iters} precision {prec}", flush=True)
    rng = np.random.default_rng(n * 1000 + iters)
    dt = torch.float64 if prec else torch.float32
    z = torch.as_tensor(rng.uniform(-0.3, 1.8, (n,) * dim)).to(dt)
    ref = otv.prox_tv_box(z.double().numpy(), 0.07, 0.0, 1.5, iters)
    N = n ** dim
    zd = z.reshape(-1).cuda()
    x = torch.full_like(zd, float("nan"))
    prox(dim, n, prec, zd, x, 0.07, iters)
    assert np.linalg.norm(x.cpu().double().numpy() - ref.ravel()) <= BAR[prec] * np.linalg.norm(ref)
    buf = torch.zeros(N + 3, dtype=dt, device="cuda")   # output over the input, and shifted by three
    for shift in (0, 3):
        buf[:N] = zd
        prox(dim, n, prec, buf[:N], buf[shift:], 0.07, iters)
        assert torch.equal(buf[shift:shift + N], x)
