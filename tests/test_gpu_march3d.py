"""GPU checks of the marching FP64 step (3-D Cartesian): sizes at the edges of its
strips (62 columns), row groups (6 rows) and chunks of planes, every pair of z
faces, against the oracle; a size with several rounds of workgroups against the
kernels an explicit tiling selects.  Bar: rel-L2 <= 1e-12 per application, the
stated FP64 tolerance of either path against the oracle."""

import numpy as np
import pytest

from oracle import stepping as S
from oracle.operator import Operator
from oracle.problem import Problem

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


@pytest.mark.parametrize("n,lo,hi,periods", [
    ((2, 2, 2), 0, 0, 1), ((2, 3, 2), 1, 1, 1), ((63, 7, 3), 0, 1, 1), ((64, 8, 5), 1, 0, 2), ((65, 6, 9), 1, 1, 1),
    ((5, 13, 40), 0, 0, 1), ((125, 14, 20), 1, 1, 1), ((20, 20, 21), 0, 1, 1),
])
def test_filter_matches_oracle(E, n, lo, hi, periods):
    bc = (0, 0, 0, 0, lo, hi)
    shape = tuple(k + 1 for k in n[::-1])
    length = (1.0, 0.9, 0.8)
    rho, lam, mu = _media(shape, sum(n))
    prob = Problem(3, n, length=length, bc=bc)
    op = Operator(prob, rho, lam, mu)
    nt = 9
    omega = 2 * np.pi / (nt * 0.8 * 2 / np.sqrt(op.gershgorin())) * 1.001
    wh = S.WaveHoltz(op, omega, nt=nt, periods=periods)
    rng = np.random.default_rng(1)
    u0, f = rng.standard_normal((3,) + shape), rng.standard_normal((3,) + shape)
    ctx = E.Context(3, n, rho, lam, mu, omega, bc, length=length, nt=nt, periods=periods)
    x, g = prob.gather(u0), prob.gather(f)
    assert _rel(prob.gather(ctx.apply_filter(u0, f).cpu().numpy()), wh.apply_filter(x, g)) <= TOL
    y = ctx.apply_A(u0).cpu().numpy()
    assert _rel(prob.gather(y), x - wh.apply_filter(x)) <= TOL
    known = prob.scatter(np.ones(op.ndof)) == 0
    assert not np.any(y[known])          # Dirichlet nodes are written as zero


def test_many_rounds_match_tilings(E):
    import torch
    n, bc = (200, 150, 90), (0, 0, 0, 0, 1, 1)
    shape = tuple(k + 1 for k in n[::-1])
    rho, lam, mu = _media(shape, 5)
    g = torch.Generator(device="cuda").manual_seed(3)
    x, f = (torch.randn((3,) + shape, generator=g, device="cuda", dtype=torch.float64) for _ in range(2))
    kw = dict(length=(2.0, 1.5, 0.9), nt=21, autotune=0)
    a = E.Context(3, n, rho, lam, mu, 5.0, bc, **kw)
    b = E.Context(3, n, rho, lam, mu, 5.0, bc, **kw)
    b.set_tile(E.FP64, 4, 8)
    for p, q in ((a.apply_filter(x, f), b.apply_filter(x, f)), (a.apply_A(x), b.apply_A(x))):
        assert float((p - q).norm() / q.norm()) <= TOL


@pytest.mark.parametrize("n,lo,hi", [((1300, 1290, 2), 0, 0), ((1001, 1555, 2), 0, 1), ((1250, 1210, 3), 1, 0),
                                     ((700, 4, 1100), 1, 1)])
def test_few_planes_or_rows_of_large_grids_match_tilings(E, n, lo, hi):
    """One to four planes, or three rows, are marched through where they are large."""
    import torch
    bc = (0, 0, 0, 0, lo, hi)
    shape = tuple(k + 1 for k in n[::-1])
    rho, lam, mu = _media(shape, 6)
    g = torch.Generator(device="cuda").manual_seed(4)
    x, f = (torch.randn((3,) + shape, generator=g, device="cuda", dtype=torch.float64) for _ in range(2))
    kw = dict(length=tuple(k / 100 for k in n), nt=12, autotune=0)
    a = E.Context(3, n, rho, lam, mu, 50.0, bc, **kw)
    b = E.Context(3, n, rho, lam, mu, 50.0, bc, **kw)
    b.set_tile(E.FP64, 4, 8)
    for p, q in ((a.apply_filter(x, f), b.apply_filter(x, f)), (a.apply_A(x), b.apply_A(x))):
        assert float((p - q).norm() / q.norm()) <= TOL
