"""GPU checks of the register-tile steps (2-D Cartesian, FP64): sizes at the
edges of tiles and launches, every face combination they take, against the
oracle where it is quick and against the marching kernels (which an explicit
tiling selects) elsewhere.  Bars: rel-L2 <= 1e-12 per application, the stated
FP64 tolerance of either path against the oracle."""

import numpy as np
import pytest

from oracle import stepping as S
from oracle.operator import Operator
from oracle.problem import FREE, Problem
from oracle.twofield import TwoField

pytestmark = pytest.mark.gpu
TOL = 1e-12


@pytest.fixture(scope="module")
def E():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2205_12344_amd import elwh
    return elwh


def _media(shape, seed):
    rng = np.random.default_rng(seed)
    rho, mu = np.exp(0.25 * rng.standard_normal(shape)), np.exp(0.25 * rng.standard_normal(shape))
    return rho, mu * np.clip(2 * np.exp(0.25 * rng.standard_normal(shape)), 1, 3), mu


def _rel(a, b):
    return np.linalg.norm(np.asarray(a) - np.asarray(b)) / np.linalg.norm(np.asarray(b))


# nt at and beside multiples of the steps per launch (a last launch of one
# step, an even and an odd one), N_T = 3 the smallest
@pytest.mark.parametrize("n,bc,nt,periods", [
    ((2, 2), (0, 0, 1, 1), 8, 1), ((3, 40), (0, 0, 0, 1), 9, 1), ((41, 3), (0, 0, 1, 0), 12, 1),
    ((43, 27), (0, 0, 1, 1), 22, 1), ((51, 51), (0, 0, 0, 0), 23, 1), ((64, 64), (0, 0, 0, 1), 24, 1),
    ((105, 30), (0, 0, 1, 1), 45, 1), ((66, 131), (0, 0, 1, 0), 34, 3),
])
def test_filter_matches_oracle(E, n, bc, nt, periods):
    shape = (n[1] + 1, n[0] + 1)
    length = (1.0, 0.9)
    rho, lam, mu = _media(shape, sum(n))
    prob = Problem(2, n, length=length, bc=bc)
    op = Operator(prob, rho, lam, mu)
    omega = 2 * np.pi / (nt * 0.8 * 2 / np.sqrt(op.gershgorin())) * 1.001
    wh = S.WaveHoltz(op, omega, nt=nt, periods=periods)
    rng = np.random.default_rng(1)
    u0, f = rng.standard_normal((2,) + shape), rng.standard_normal((2,) + shape)
    ctx = E.Context(2, n, rho, lam, mu, omega, bc, length=length, nt=nt, periods=periods)
    x, g = prob.gather(u0), prob.gather(f)
    assert _rel(prob.gather(ctx.apply_filter(u0, f).cpu().numpy()), wh.apply_filter(x, g)) <= TOL
    y = ctx.apply_A(u0).cpu().numpy()
    assert _rel(prob.gather(y), x - wh.apply_filter(x)) <= TOL
    known = prob.scatter(np.ones(op.ndof)) == 0
    assert not np.any(y[known])          # Dirichlet nodes are written as zero


@pytest.mark.parametrize("n,bc", [((700, 260), (0, 0, 1, 1)), ((2300, 150), (0, 0, 0, 1)), ((333, 1040), (0, 0, 1, 0))])
def test_many_rounds_match_marching(E, n, bc):
    import torch
    shape = (n[1] + 1, n[0] + 1)
    rho, lam, mu = _media(shape, 5)
    g = torch.Generator(device="cuda").manual_seed(3)
    x, f = (torch.randn((2,) + shape, generator=g, device="cuda", dtype=torch.float64) for _ in range(2))
    kw = dict(length=(n[0] / 100, n[1] / 100), nt=41)
    a = E.Context(2, n, rho, lam, mu, 30.0, bc, **kw)
    b = E.Context(2, n, rho, lam, mu, 30.0, bc, autotune=0, **kw)
    b.set_tile(E.FP64, 1, 10)
    for p, q in ((a.apply_filter(x, f), b.apply_filter(x, f)), (a.apply_A(x), b.apply_A(x))):
        assert float((p - q).norm() / q.norm()) <= TOL


@pytest.mark.parametrize("n,bc,nt", [
    ((2, 3), (2, 2, 2, 2), 7), ((40, 31), (2, 2, 2, 2), 30), ((50, 50), (2, 0, 2, 1), 23), ((64, 70), (0, 2, 1, 2), 33),
    ((105, 47), (0, 0, 2, 0), 21), ((131, 66), (2, 2, 0, 0), 44),
])
def test_two_field_matches_oracle(E, n, bc, nt):
    shape = (n[1] + 1, n[0] + 1)
    length = (1.1, 1.0)
    rho, lam, mu = _media(shape, 7 * n[0] + n[1])
    prob = Problem(2, n, length=length, bc=tuple(FREE if b else 0 for b in bc))
    op = Operator(prob, rho, lam, mu)
    omega = 2 * np.pi / (nt * 0.8 * 2 / np.sqrt(op.gershgorin())) * 1.001
    t = TwoField(op, omega, [(k // 2, k % 2) for k in range(4) if bc[k] == 2], nt=nt)
    rng = np.random.default_rng(2)
    u0, u1, f = (rng.standard_normal((2,) + shape) for _ in range(3))
    u1 *= omega
    ctx = E.Context(2, n, rho, lam, mu, omega, bc, length=length, nt=nt)
    a, b = (v.cpu().numpy() for v in ctx.apply_filter2(u0, u1, f))
    r0, r1 = t.apply_filter(prob.gather(u0), prob.gather(u1), prob.gather(f))
    assert _rel(prob.gather(a), r0) <= TOL and _rel(prob.gather(b), r1) <= TOL
    a, b = (v.cpu().numpy() for v in ctx.apply_A2(u0, u1))
    r0, r1 = t.apply_filter(prob.gather(u0), prob.gather(u1))
    assert _rel(prob.gather(a), prob.gather(u0) - r0) <= TOL and _rel(prob.gather(b), prob.gather(u1) - r1) <= TOL


@pytest.mark.parametrize("n", [(900, 600)])
def test_two_field_many_rounds_match_marching(E, n):
    import torch
    shape = (n[1] + 1, n[0] + 1)
    rho, lam, mu = _media(shape, 9)
    g = torch.Generator(device="cuda").manual_seed(4)
    x0, x1 = (torch.randn((2,) + shape, generator=g, device="cuda", dtype=torch.float64) for _ in range(2))
    kw = dict(length=(n[0] / 100, n[1] / 100), nt=29)
    a = E.Context(2, n, rho, lam, mu, 40.0, (2, 2, 2, 2), **kw)
    b = E.Context(2, n, rho, lam, mu, 40.0, (2, 2, 2, 2), autotune=0, **kw)
    b.set_tile(E.FP64, 1, 8)
    for p, q in zip(a.apply_A2(x0, x1), b.apply_A2(x0, x1)):
        assert float((p - q).norm() / q.norm()) <= TOL
