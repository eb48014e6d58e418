"""The sorts at the edges of their tiles and of their choices, against a stable
sort of the cells on the CPU (the permutation of a stable sort is unique, so all
comparisons are bit for bit).

General sort: stores just below, at and above the size from which the fields are
gathered by records, with every remainder of a record part, over cell counts
whose digits take two passes of eight, two of nine and three of eight bits.
Neighbour sort: grids down to three cells an axis, with empty cells and cells of
more ions than a wavefront loads at once, moved to random neighbours."""
import numpy as np
import pytest

from paper_2305_05600_amd import workloads as W
from tests.helpers import announce

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

RECORDS = 3 << 19  # ions from which the general sort gathers by records


@pytest.fixture(scope="module")
def H():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2305_05600_amd import hvpic

    hvpic.lib()
    return hvpic


def _cfg(nx, ny, nz):
    return W.Config(name="tiles", ndim=3 if nz > 1 else 2, nx=nx, ny=ny, nz=nz, dx=0.5, dy=0.4,
                    dz=0.7 if nz > 1 else 1.0, dt=0.05, nsub=3, te=0.2, eta=1e-3)


def _store(cfg, cell, rng):
    parts = {"cell": cell.astype(np.int32)}
    for k in ["ox", "oy"] + (["oz"] if cfg.ndim == 3 else []) + ["ux", "uy", "uz", "w"]:
        parts[k] = rng.uniform(-1.0, 1.0, cell.size).astype(np.float32)
    return parts


def _check(cfg, parts, got, cs, order):
    for k, v in parts.items():
        assert np.array_equal(got[k], v[order]), k
    count = np.bincount(parts["cell"], minlength=cfg.ncell)
    assert np.array_equal(cs.cpu().numpy(), np.concatenate([[0], np.cumsum(count)]))


@pytest.mark.parametrize("shape,n", [((255, 256, 1), RECORDS - 1), ((255, 256, 1), RECORDS),
                                     ((300, 219, 1), RECORDS + 1), ((512, 300, 1), RECORDS + 2),
                                     ((640, 411, 1), RECORDS + 3), ((64, 64, 64), RECORDS + 1),
                                     ((70, 61, 62), RECORDS + 3), ((300, 219, 1), 2049)])
def test_general(H, shape, n):
    announce("sort-general", shape, n)
    cfg = _cfg(*shape)
    rng = np.random.Generator(np.random.PCG64(n))
    parts = _store(cfg, rng.integers(0, cfg.ncell, n), rng)
    parts["cell"][:3] = cfg.ncell - 1
    order = np.argsort(parts["cell"], kind="stable")
    ctx = H.Context(cfg, n)
    p, q = H.Particles.from_numpy(parts, cfg.ndim), H.Particles(cfg.ndim, n, "cuda")
    cs = torch.full((cfg.ncell + 1,), -1, dtype=torch.int32, device="cuda")
    H.hvpic_sort(ctx.ctx, p, q, None, cs, full=True)
    _check(cfg, parts, q.to_numpy(), cs, order)


@pytest.mark.parametrize("shape", [(3, 3, 1), (4, 5, 1), (7, 9, 1), (66, 17, 1), (3, 3, 3),
                                   (4, 4, 3), (9, 8, 5), (34, 5, 4)])
@pytest.mark.parametrize("ppc", [0.6, 70.0])
def test_neighbour(H, shape, ppc):
    announce("sort-neighbour", shape, ppc)
    cfg = _cfg(*shape)
    rng = np.random.Generator(np.random.PCG64(int(ppc * 10) + cfg.ncell))
    count = rng.poisson(ppc, cfg.ncell)
    count[rng.integers(0, cfg.ncell, 1 + cfg.ncell // 5)] = 0
    count[cfg.ncell // 2] = 1100
    old = np.repeat(np.arange(cfg.ncell), count)
    ijk = [old % cfg.nx, old // cfg.nx % cfg.ny, old // (cfg.nx * cfg.ny)]
    dims = [cfg.nx, cfg.ny, cfg.nz]
    new = [(a + rng.integers(-1, 2, old.size)) % m if m > 1 else a for a, m in zip(ijk, dims)]
    parts = _store(cfg, new[0] + cfg.nx * (new[1] + cfg.ny * new[2]), rng)
    order = np.argsort(parts["cell"], kind="stable")
    n = old.size
    ctx = H.Context(cfg, n)
    p, q = H.Particles.from_numpy(parts, cfg.ndim), H.Particles(cfg.ndim, n, "cuda")
    prev = torch.from_numpy(np.concatenate([[0], np.cumsum(count)]).astype(np.int32)).cuda()
    cs = torch.full((cfg.ncell + 1,), -1, dtype=torch.int32, device="cuda")
    H.hvpic_sort(ctx.ctx, p, q, prev, cs, full=False)
    _check(cfg, parts, q.to_numpy(), cs, order)
    perm = torch.full((n,), -1, dtype=torch.int32, device="cuda")
    H.hvpic_sort_perm(ctx.ctx, p, prev, perm, cs)
    assert np.array_equal(perm.cpu().numpy(), order)
    flags, _ = H.hvpic_sync_status(ctx.ctx)
    assert not flags & H.FLAG_MOVE_GT1


@pytest.mark.parametrize("shape", [(3, 3, 1), (7, 9, 1), (66, 17, 1), (3, 3, 3), (9, 8, 5)])
@pytest.mark.parametrize("ppc", [30.0, 110.0, 230.0])
def test_neighbour_by_density(H, shape, ppc):
    """The same at the densities that select four, two and one cells per wavefront."""
    test_neighbour(H, shape, ppc)
