"""GPU checks of wide grids of a few rows, on both sides of the line between the
register tiles and the marching kernels: filter with forcing and A_h against the
oracle.  Bar: rel-L2 <= 1e-12 per application, the stated FP64 tolerance of either
path."""

import numpy as np
import pytest

from oracle import stepping as S
from oracle.curvilinear import MappedOperator
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


def _omega(op, nt):
    """The frequency at which the time-step rule gives nt steps."""
    return 2 * np.pi / (nt * 0.8 * 2 / np.sqrt(op.gershgorin())) * 1.001


@pytest.mark.parametrize("n,bc", [((26000, 3), (0, 0, 0, 1)), ((28000, 3), (0, 0, 1, 0)), ((27001, 2), (0, 0, 0, 0)),
                                  ((61000, 7), (0, 0, 0, 1))])
def test_one_field(E, n, bc):
    shape, length, nt = (n[1] + 1, n[0] + 1), (n[0] / 100, n[1] / 100), 11
    rho, lam, mu = _media(shape, n[1])
    prob = Problem(2, n, length=length, bc=bc)
    op = Operator(prob, rho, lam, mu)
    om = _omega(op, nt)
    wh = S.WaveHoltz(op, om, nt=nt)
    rng = np.random.default_rng(1)
    u0, f = rng.standard_normal((2,) + shape), rng.standard_normal((2,) + shape)
    ctx = E.Context(2, n, rho, lam, mu, om, bc, length=length, nt=nt)
    x, g = prob.gather(u0), prob.gather(f)
    assert _rel(prob.gather(ctx.apply_filter(u0, f).cpu().numpy()), wh.apply_filter(x, g)) <= TOL
    assert _rel(prob.gather(ctx.apply_A(u0).cpu().numpy()), x - wh.apply_filter(x)) <= TOL


@pytest.mark.parametrize("n,bc", [((26000, 3), (2, 2, 0, 2)), ((28000, 3), (2, 0, 2, 0)), ((71000, 5), (0, 2, 0, 1))])
def test_two_fields(E, n, bc):
    shape, length, nt = (n[1] + 1, n[0] + 1), (n[0] / 100, n[1] / 100), 10
    rho, lam, mu = _media(shape, n[1] + 20)
    prob = Problem(2, n, length=length, bc=tuple(FREE if b else 0 for b in bc))
    op = Operator(prob, rho, lam, mu)
    om = _omega(op, nt)
    t = TwoField(op, om, [(k // 2, k % 2) for k in range(4) if bc[k] == 2], nt=nt)
    rng = np.random.default_rng(2)
    u0, u1, f = (rng.standard_normal((2,) + shape) for _ in range(3))
    u1 *= om
    ctx = E.Context(2, n, rho, lam, mu, om, bc, length=length, nt=nt)
    a, b = (v.cpu().numpy() for v in ctx.apply_filter2(u0, u1, f))
    r0, r1 = t.apply_filter(prob.gather(u0), prob.gather(u1), prob.gather(f))
    assert _rel(prob.gather(a), r0) <= TOL and _rel(prob.gather(b), r1) <= TOL


@pytest.mark.parametrize("nq,nr,bc", [(26000, 3, (0, 0, 1, 1)), (28000, 3, (0, 0, 0, 1)), (71000, 5, (0, 0, 0, 0))])
def test_mapped(E, nq, nr, bc):
    q, r = np.arange(nq + 1) / 100.0, np.arange(nr + 1) / 100.0
    x = q[None, :] + 0.3 * r[:, None] + 0.002 * np.sin(9 * q)[None, :]
    y = r[:, None] + 0.004 * np.sin(5 * q)[None, :]
    rho, lam, mu = _media(x.shape, nr + 40)
    op = MappedOperator(x, y, rho, lam, mu, bc=bc)
    om = _omega(op, 9)
    wh = S.WaveHoltz(op, om)
    prob = op.prob
    rng = np.random.default_rng(3)
    u0, f = (rng.standard_normal(prob.field_shape) for _ in range(2))
    ctx = E.MappedContext(x, y, rho, lam, mu, om, bc=bc)
    assert ctx.info()["nt"] == wh.nt
    gu, gf = prob.gather(u0), prob.gather(f)
    assert _rel(prob.gather(ctx.apply_filter(u0, f).cpu().numpy()), wh.apply_filter(gu, gf)) <= TOL
    assert _rel(prob.gather(ctx.apply_A(u0).cpu().numpy()), gu - wh.apply_filter(gu)) <= TOL
