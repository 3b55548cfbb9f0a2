"""GPU tests of the row kernels of the BiCGSTAB iteration: solutions meet the tolerance in the oracle's
FP64 residual, forward and adjoint, with the vectors' loads of every batching."""

import numpy as np
import pytest

from gpu_common import make_pair, rel, say, to_dev, to_np
from oracle import operators
from synth import disks_2d, ellipses_2d, random_field

pytestmark = pytest.mark.gpu


# transform lengths 128 to 512 and two with a factor 3; n = P/2 (checks decided at compile time), an odd
# n and one with a partial last block of rows; a single system and several that stop at different steps
@pytest.mark.parametrize("prec", ["c64", "c128"])
@pytest.mark.parametrize("n,T", [(33, 1), (64, 3), (61, 5), (96, 2), (83, 3), (128, 2), (125, 3), (131, 2)])
@pytest.mark.parametrize("adjoint", [False, True])
def test_solutions_meet_the_fp64_residual(prec, n, T, adjoint):
    from paper_1708_01663_amd.cisor import SolveOpts
    say(f"solver rows {prec} {n} {T} {adjoint}")
    prob, op = make_pair(n, 1 / 10, T, 8, precision=prec)
    f = ellipses_2d(n, 3, inner=4, eps_range=(1.0, 1.3))
    rng = np.random.default_rng(n)
    scale = 10.0 ** np.arange(T)[:, None, None]   # tolerances are relative per system
    b = (rng.standard_normal((T, n, n)) + 1j * rng.standard_normal((T, n, n))) * scale
    bd = to_dev(b.reshape(T, -1), op)
    b = to_np(bd).reshape(T, n, n)
    tol = 1e-6 if prec == "c64" else 1e-10
    x, its, code = op.solve(to_dev(f.ravel(), op, real=True), bd, adjoint=adjoint, opts=SolveOpts(tol=tol, maxit=5000))
    assert code == 0 and min(its) > 0
    xn = to_np(x).reshape(T, n, n)
    apply = operators.apply_AH if adjoint else operators.apply_A
    for t in range(T):
        r = np.linalg.norm(b[t] - apply(prob.Ghat, f, xn[t])) / np.linalg.norm(b[t])
        # the stop test is on the FP64 residual; f and x are what the device holds, f rounded in c64
        assert r <= (1.05 * tol if prec == "c128" else 1.5 * tol), (t, its)


# the operator's own rows: every transform length that is no small grid, a side that leaves columns and
# rows over (the last one before the next length, and the first after the previous)
@pytest.mark.parametrize("prec", ["c64", "c128"])
@pytest.mark.parametrize("n", [33, 63, 65, 96, 97, 127, 129, 192, 193, 255, 257, 384, 385, 511])
def test_operator_rows_match_oracle(n, prec):
    T = 2
    say(f"operator rows n={n} {prec}")
    prob, op = make_pair(n, 0.1, T, 3, precision=prec)
    f, x = disks_2d(n, n, count=2, radius_px=(n / 8, n / 4), eps_range=(1.2, 1.6)), random_field((T, n, n), n)
    fd, xd = to_dev(f.ravel(), op, real=True), to_dev(x.reshape(T, -1), op)
    for adj in (False, True):
        ref = (operators.apply_AH if adj else operators.apply_A)(prob.Ghat, f, x)
        assert rel(to_np(op.apply_A(fd, xd, adjoint=adj)).reshape(T, n, n), ref) < (2e-6 if prec == "c64" else 1e-12)
