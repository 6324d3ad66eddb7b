"""GPU checks of the FP64 autotuner: the register tiles and the march are among
what it times, its choice decides what runs (also after elwh_set_tile, and from
the cache file), and nothing is timed at create where the sizes decide.  Which
kernel ran is told by the bits: the kernels add in different orders."""

import json

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


def _problem(n, seed):
    shape = tuple(k + 1 for k in reversed(n))
    rng = np.random.default_rng(seed)
    rho, mu = np.exp(0.25 * rng.standard_normal(shape)), np.exp(0.25 * rng.standard_normal(shape))
    return (rho, 2 * mu, mu), rng.standard_normal((len(n),) + shape)


def _bits(ctx, u):
    return ctx.apply_A(u).cpu().numpy().tobytes()


def _entries(path):
    return [json.loads(line) for line in open(path)] if path.exists() else []


@pytest.mark.parametrize("n,tile", [((211, 97), (1, 8)), ((37, 41, 33), (4, 8))])
def test_autotune_decides_what_runs(E, n, tile):
    """Register tiles in 2-D, the march in 3-D: left by set_tile, timed against
    the tilings (which they beat two to one at these sizes) and returned to."""
    media, u = _problem(n, 1)
    bc = (0,) * (2 * len(n))
    ctx = E.Context(len(n), n, *media, 9.0, bc, autotune=0)
    own = _bits(ctx, u)
    ctx.set_tile(E.FP64, *tile)
    assert _bits(ctx, u) != own
    assert ctx.autotune(E.FP64) > 0.0
    assert _bits(ctx, u) == own
    ctx.set_tile(E.FP64, *tile)
    assert ctx.autotune(E.FP64) == -1.0      # this process's choice for the size
    assert _bits(ctx, u) == own


def test_create_times_only_what_may_run(E, tmp_path, monkeypatch):
    path = tmp_path / "tiles.jsonl"
    monkeypatch.setenv("ELWH_TUNE_CACHE", str(path))
    media, u = _problem((83, 61), 2)
    E.Context(2, (83, 61), *media, 9.0, (0, 0, 0, 1))
    assert not _entries(path)
    E.Context(2, (83, 61), *media, 9.0, (0, 0, 0, 1), fuse=2)      # marching kernels: their tilings are timed
    assert [e["variant"] for e in _entries(path)] == [2]
    q, r, z = (np.arange(k + 1) / k for k in (6, 7, 8))
    grid = [a + np.zeros((9, 8, 7)) for a in (q[None, None, :], r[None, :, None], z[:, None, None])]
    one = np.ones((9, 8, 7))
    mapped = E.MappedContext3(*grid, one, 2 * one, one, 3.0, prec=E.FP32_STEP)     # one tiling
    assert len(_entries(path)) == 1 and mapped.autotune(E.FP64) == mapped.autotune(E.FP32_STEP) == -1.0
    media, _ = _problem((128, 128, 5), 3)                           # near the line: the march and the tilings are
    E.Context(3, (128, 128, 5), *media, 9.0, (0,) * 6)
    assert [(e["dim"], e["variant"]) for e in _entries(path)] == [(2, 2), (3, 2 | 32)]


def test_cache_file_decides(E, tmp_path, monkeypatch):
    """An entry of a context that could take register tiles selects its tiling;
    entries without that mark are of other candidates and do not apply."""
    import torch
    n = (89, 67)
    media, u = _problem(n, 4)
    args = (2, n) + media + (9.0, (0, 0, 0, 1))
    own, marching = E.Context(*args, autotune=0), E.Context(*args, autotune=0)
    marching.set_tile(E.FP64, 1, 8)
    assert _bits(own, u) != _bits(marching, u)
    arch = torch.cuda.get_device_properties(0).gcnArchName.split(":")[0]
    entry = {"arch": arch, "dim": 2, "prec": 0, "variant": 3 << 1, "n": [n[0], n[1], 0], "V": 1, "rows": 8, "us": 1.0}
    path = tmp_path / "tiles.jsonl"
    monkeypatch.setenv("ELWH_TUNE_CACHE", str(path))
    path.write_text("".join(json.dumps(dict(entry, n=[n[0], n[1], k])) + "\n" for k in (0, 1)))
    assert _bits(E.Context(*args), u) == _bits(own, u)
    n = (89, 68)
    media, u = _problem(n, 5)
    args = (2, n) + media + (9.0, (0, 0, 0, 1))
    marching = E.Context(*args, autotune=0)
    marching.set_tile(E.FP64, 1, 8)
    path.write_text("".join(json.dumps(dict(entry, variant=3 << 1 | 32, n=[n[0], n[1], k])) + "\n" for k in (0, 1)))
    assert _bits(E.Context(*args), u) == _bits(marching, u)
