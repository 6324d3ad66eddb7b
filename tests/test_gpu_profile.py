"""GPU checks of the kernel timing: the number of time steps is that of the steps
inside the timed span, whichever kernels take them."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def E():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2205_12344_amd import elwh
    return elwh


def _read(ctx, call, n=3):
    ctx.profile_enable(True)
    for _ in range(n):
        call()
    p = ctx.profile_read()
    assert p["ninit"] == n and p["step_ms"] > 0.0
    return p["nstep"] / n


def test_step_counts(E):
    one, nt = np.ones((48, 61)), 17
    x = np.random.default_rng(0).standard_normal((2, 48, 61))
    ctx = E.Context(2, (60, 47), one, 2 * one, one, 20.0, (0, 0, 0, 1), nt=nt, autotune=0)
    assert _read(ctx, lambda: ctx.apply_A(x)) == nt              # register tiles: the start among them
    ctx.set_tile(E.FP64, 1, 8)
    assert _read(ctx, lambda: ctx.apply_A(x)) == nt - 1          # the half step timed apart
    two = E.Context(2, (60, 47), one, 2 * one, one, 20.0, (2, 2, 2, 2), nt=nt, autotune=0)
    assert _read(two, lambda: two.apply_A2(x, x)) == nt + 1      # and one step past the period, for its velocity
    q, r = np.arange(61) / 60.0, np.arange(48) / 60.0
    grid = q[None, :] + 0.1 * r[:, None], r[:, None] + 0.0 * q[None, :]
    mapped = E.MappedContext(*grid, one, 2 * one, one, 20.0, nt=nt, autotune=0)
    assert _read(mapped, lambda: mapped.apply_A(x)) == nt
    mapped.set_tile(E.FP64, 1, 8)
    assert _read(mapped, lambda: mapped.apply_A(x)) == nt - 1
