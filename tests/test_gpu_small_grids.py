"""GPU parity of the one-block-per-system path of small 2D grids against the oracle: the grid sides
at its edges (and just past them), every start mode, iteration caps and many systems."""

import numpy as np
import pytest
import torch

from gpu_common import make_pair, rel, say, to_dev, to_np
from oracle import cisor as ocisor, operators
from synth import disks_2d, random_field

pytestmark = pytest.mark.gpu
H = 0.1


def contrast(n):
    return disks_2d(n, n, count=2, radius_px=(max(1.0, n / 8), max(1.5, n / 4)), eps_range=(1.2, 1.6))


@pytest.mark.parametrize("prec", ["c64", "c128"])
@pytest.mark.parametrize("n", [2, 5, 31, 32, 33, 63, 64, 65])
def test_operator_and_solves_match_oracle(n, prec):
    from paper_1708_01663_amd.cisor import SolveOpts
    T, M = 3, 7
    say(f"small grid n={n} {prec}")
    prob, op = make_pair(n, H, T, M, precision=prec)
    f, x = contrast(n), random_field((T, n, n), n)
    fd, xd = to_dev(f.ravel(), op, real=True), to_dev(x.reshape(T, -1), op)
    tol_op = 2e-6 if prec == "c64" else 1e-12          # the operator's bar at every size
    for adj in (False, True):
        ref = (operators.apply_AH if adj else operators.apply_A)(prob.Ghat, f, x)
        assert rel(to_np(op.apply_A(fd, xd, adjoint=adj)).reshape(T, n, n), ref) < tol_op
    born = prob.u_in - operators.apply_A(prob.Ghat, f, prob.u_in)
    assert rel(to_np(op.born_field(fd)).reshape(T, n, n), born) < 10 * tol_op
    tol, bar = (1e-6, 1e-4) if prec == "c64" else (1e-10, 1e-8)
    u_ref, y_ref = ocisor.forward(prob, f, tol=1e-12)
    for start in (0, 1):
        u, y, its, code = op.forward(fd, SolveOpts(tol=tol, start=start))
        assert code == 0 and rel(to_np(u).reshape(T, n, n), u_ref) < bar and rel(to_np(y), y_ref) < bar
    # adjoint systems from a caller's guess (modes 2, 3 and 5), checked by their true residual
    for start in (2, 3, 5):
        v, its, code = op.solve(fd, xd, adjoint=True, opts=SolveOpts(tol=tol, start=start),
                                x0=(0.3 * xd).contiguous())
        res = operators.apply_AH(prob.Ghat, f, to_np(v).reshape(T, n, n)) - to_np(xd).reshape(T, n, n)
        for t in range(T):
            assert code == 0 and np.linalg.norm(res[t]) <= 1.05 * tol * np.linalg.norm(to_np(xd)[t])


@pytest.mark.parametrize("prec,n", [("c64", 32), ("c64", 50), ("c128", 30)])
def test_iteration_cap_and_zero_systems(prec, n):
    """maxit is a soft stop with every output written; a zero right-hand side gives zero at once."""
    from paper_1708_01663_amd.cisor import SolveOpts
    T = 3
    say(f"small grid cap n={n} {prec}")
    prob, op = make_pair(n, H, T, 5, precision=prec)
    f = contrast(n)
    fd = to_dev(f.ravel(), op, real=True)
    b = to_dev(random_field((T, n, n), 1).reshape(T, -1), op)
    b[1] = 0
    x, its, code = op.solve(fd, b, opts=SolveOpts(tol=1e-9 if prec == "c64" else 1e-14, maxit=2, start=0))
    assert code == 1 and list(its) == [2, 0, 2] and bool((x[1] == 0).all()) and bool(torch.isfinite(x.abs()).all())
    long, _, _ = op.solve(fd, b, opts=SolveOpts(tol=1e-6, start=0))
    r2 = rel(to_np(x), to_np(long))
    assert 0 < r2 < 0.5                               # two iterations on the way to the solution
    # frequent checks and replacements change nothing but the rounding
    often, _, code = op.solve(fd, b, opts=SolveOpts(tol=1e-6, start=0, check_every=1, replace_every=2))
    assert code == 0 and rel(to_np(often), to_np(long)) < 1e-4


def test_many_systems():
    """More systems than CUs, several blocks a CU: each gets the field it gets alone."""
    from paper_1708_01663_amd.cisor import Cisor, SolveOpts, ring
    n, M, T = 6, 4, 700
    f = torch.as_tensor(contrast(n).ravel()).float().cuda()
    a = 0.01 * np.arange(T)
    dirs = np.stack([np.cos(a), np.sin(a)], 1)
    say(f"small grid T={T}")
    u, _, its, code = Cisor(n, H, dirs, ring(M, n * H)).forward(f, SolveOpts(tol=1e-6, start=1))
    assert code == 0
    for t in (0, 255, 699):
        one, _, it1, _ = Cisor(n, H, dirs[t:t + 1], ring(M, n * H)).forward(f, SolveOpts(tol=1e-6, start=1))
        assert rel(to_np(u)[t], to_np(one)[0]) < 1e-6 and it1[0] == its[t]
