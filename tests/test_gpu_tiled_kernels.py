"""GPU checks of the tiled FP64 step kernels where contexts take register tiles or
the march unless elwh_set_tile asks for a tiling: every remainder of N_T against
the oracle.  Bar: rel-L2 <= 1e-12 per application, the stated FP64 tolerance."""

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


@pytest.mark.parametrize("nt", [3, 4, 5, 6, 8, 9])
@pytest.mark.parametrize("n,bc,fuse,tiles", [
    # half step, four-step launches, and the remainder of N_T - 1 in shorter ones
    ((131, 23), (0, 0, 1, 1), 4, [(1, 4), (1, 8), (1, 10), (1, 12), (1, 16), (2, 4), (2, 8), (2, 16)]),
    # half step, pairs and a last single step; and single steps throughout
    ((47, 13, 21), (0, 0, 0, 0, 1, 1), 2, [(2, 8), (4, 16), (6, 32), (1, 16), (1, 32)]),
])
def test_every_step_count(E, n, bc, fuse, tiles, nt):
    dim, shape = len(n), tuple(k + 1 for k in reversed(n))
    rho, lam, mu = _media(shape, 500 + nt)
    prob = Problem(dim, n, bc=bc)
    op = Operator(prob, rho, lam, mu)
    om = 2 * np.pi / (nt * 0.8 * 2 / np.sqrt(op.gershgorin())) * 1.001
    wh = S.WaveHoltz(op, om, nt=nt)
    rng = np.random.default_rng(nt)
    u0, f = (rng.standard_normal(prob.field_shape) * prob.unknown_mask() for _ in range(2))
    ref = prob.scatter(wh.apply_filter(prob.gather(u0), prob.gather(f)))
    refA = prob.scatter(wh.apply_A(prob.gather(u0)))
    ctx = E.Context(dim, n, rho, lam, mu, om, bc, nt=nt, fuse=fuse, autotune=0)
    for tile in tiles:
        ctx.set_tile(E.FP64, *tile)
        assert _rel(ctx.apply_filter(u0, f).cpu().numpy(), ref) <= TOL, tile
        assert _rel(ctx.apply_A(u0).cpu().numpy(), refA) <= TOL, tile
