"""The particle kernels' chunk and window plans on uneven densities, against
the FP64 oracle.

A block takes its chunk of a sorted store through LDS windows over the chunk's
cells, in several passes where a sparse region's chunk spans more cells than
one window holds.  Boxes whose rows alternate between dense and sparse are
pushed in place and through a map, with and without the fused deposit, at the
average densities that select each plan (2D: 3072 and 1024 ions per block;
3D: windows of 24, 40 and 64 cells), and boxes so sparse that a chunk needs
more passes than a block makes.

Tolerances: cells, sort order and cell_start bit-exact; velocities FP32
rounding; moments 1e-5 relative L2."""
import numpy as np
import pytest

import oracle as O
from paper_2305_05600_amd import workloads as W
from tests import graph_nodes
from tests.helpers import announce, compare_particles, deposit_point_straddlers, drop_push_straddlers, rel_l2

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def H():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2305_05600_amd import hvpic

    hvpic.lib()
    return hvpic


def _cfg(ndim, shape):
    dims = dict(nx=61, ny=24, nz=1, dz=1.0) if ndim == 2 else dict(nx=19, ny=10, nz=6, dz=0.7)
    return W.Config(name="win", ndim=ndim, dx=0.5, dy=0.4, dt=0.05, nsub=3, shape=shape, te=0.2,
                    eta=1e-3, **dims)


def dev(a, dtype=None):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=dtype)).cuda()


def _uneven(cfg, seed, ppc, thin):
    """A sorted box of ppc ions per cell on average whose rows come in bands
    of three dense ones and three with `thin` times the dense density."""
    _, parts, B = W.random_box(seed, cfg, 2.0 * ppc / (1.0 + thin), vmax_cells=0.9)
    rng = np.random.Generator(np.random.PCG64(seed + 1))
    row = parts["cell"] // cfg.nx
    keep = ((row // 3) % 2 == 0) | (rng.uniform(size=row.size) < thin)
    parts = {k: np.ascontiguousarray(v[keep]) for k, v in parts.items()}
    E = W.random_field(seed + 2, cfg, 0.3)
    parts = drop_push_straddlers(cfg, parts, E, B, back=0.5 * cfg.dt)
    perm, cs = O.sort(cfg, parts["cell"])
    return {k: np.ascontiguousarray(v[perm]) for k, v in parts.items()}, E, B, cs


PLANS = [(2, 90.0, 0.1), (2, 60.0, 0.1), (2, 30.0, 0.2), (2, 3.0, 0.05), (3, 70.0, 0.1),
         (3, 45.0, 0.1), (3, 24.0, 0.2), (3, 5.0, 0.05)]


@pytest.mark.parametrize("shape", [W.SHAPE_QS, W.SHAPE_NGP])
@pytest.mark.parametrize("ndim,ppc,thin", PLANS)
@pytest.mark.parametrize("mapped", [False, True])
def test_uneven_density(H, ndim, ppc, thin, shape, mapped):
    announce("uneven_density", ndim, ppc, thin, shape, mapped)
    cfg = _cfg(ndim, shape)
    parts, E, B, cs0 = _uneven(cfg, 900 + int(ppc), ppc, thin)
    n = parts["cell"].size
    ctx = H.Context(cfg, n)
    cs_prev, cs = dev(cs0, np.int32), torch.zeros(cfg.ncell + 1, dtype=torch.int32, device="cuda")
    n_mid = torch.full((cfg.ncell,), 7.0, device="cuda")
    J_mid = torch.full((3, cfg.ncell), 7.0, device="cuda")
    diag = torch.zeros(4, dtype=torch.float64, device="cuda")
    ref = {k: v.copy() for k, v in O.particles64(parts).items()}
    rd, st = O.push(cfg, ref, E, B)
    rn, rJ = O.deposit(cfg, ref, 0.5 * cfg.dt)
    rperm, rcs = O.sort(cfg, ref["cell"])
    q = H.Particles(ndim, n)
    if mapped:
        # the store shuffled within itself, the map restoring its order
        rng = np.random.Generator(np.random.PCG64(77))
        order = rng.permutation(n)
        inv = np.empty(n, np.int64)
        inv[order] = np.arange(n)
        p = H.Particles.from_numpy({k: np.ascontiguousarray(v[order]) for k, v in parts.items()}, ndim)
        H.hvpic_gather_push_perm(ctx.ctx, p, dev(inv, np.int32), q, cs_prev, dev(E), dev(B), n_mid,
                                 J_mid, diag)
        pushed, perm = q, torch.zeros(n, dtype=torch.int32, device="cuda")
        H.hvpic_sort_perm(ctx.ctx, q, cs_prev, perm, cs)
        torch.cuda.synchronize()
        assert np.array_equal(perm.cpu().numpy(), rperm)
    else:
        p = H.Particles.from_numpy(parts, ndim)
        H.hvpic_gather_push(ctx.ctx, p, cs_prev, dev(E), dev(B), n_mid, J_mid, diag)
        pushed = p
        H.hvpic_sort(ctx.ctx, p, q, cs_prev, cs)
    flags, counts = H.hvpic_sync_status(ctx.ctx)
    assert flags == 0 and counts[0] == st.moved_gt1 == 0
    compare_particles(cfg, pushed.to_numpy(), ref, band=0.0)
    assert np.array_equal(cs.cpu().numpy(), rcs)
    assert rel_l2(n_mid.cpu().numpy(), rn) < 1e-5
    assert rel_l2(J_mid.cpu().numpy(), rJ) < 1e-5
    assert np.allclose(diag.cpu().numpy(), rd, rtol=1e-5, atol=1e-6 * abs(rd[0]))
    # the stand-alone deposit of the pushed store in its old order
    H.hvpic_deposit(ctx.ctx, pushed, None, 0.5 * cfg.dt, n_mid, J_mid)
    torch.cuda.synchronize()
    assert rel_l2(n_mid.cpu().numpy(), rn) < 1e-5
    assert rel_l2(J_mid.cpu().numpy(), rJ) < 1e-5


# plans and chunks whose ions went to the FP64 accumulators one by one before the chunks were cut to the windows:
# 1024 and 2048 ions a block, windows of 40 and 64 cells, several passes, more passes than a block makes
SPARSE = [(2, 30.0, 1.0), (2, 45.0, 1.0), (2, 90.0, 0.05), (2, 5.0, 1.0), (2, 0.4, 1.0), (3, 45.0, 1.0), (3, 24.0, 1.0),
          (3, 70.0, 0.05), (3, 4.0, 1.0), (3, 0.4, 1.0)]


@pytest.mark.parametrize("ndim,ppc,thin", SPARSE)
@pytest.mark.parametrize("call", ["deposit", "push", "push_perm"])
def test_sparse_sums_are_rounded_once(H, ndim, ppc, thin, call):
    """Weights with all 24 bits in use, velocities +-1 and +-1/2 and no fields:
    every product is exact in FP32 and every sum in FP64, so the moments of
    sparse stores are the exact sums rounded to FP32, bit for bit.  (Of a store
    with thin bands the middle row of each band is looked at.)"""
    announce("sparse_sums", ndim, ppc, thin, call)
    dims = dict(nx=61, ny=24, nz=1) if ndim == 2 else dict(nx=19, ny=12, nz=6)
    if ppc < 1:
        dims["ny"] *= 4
    cfg = W.Config(name="sums", ndim=ndim, dx=1.0, dy=1.0, dz=1.0, dt=0.05, nsub=3, shape=W.SHAPE_NGP, te=0.2, eta=1e-3, **dims)
    rng = np.random.Generator(np.random.PCG64(int(10 * ppc) + ndim))
    rate = np.full(cfg.ncell, 2.0 * ppc / (1.0 + thin))
    thinned = (np.arange(cfg.ncell) // cfg.nx // 3) % 2 == 1
    rate[thinned] *= thin
    cell = np.repeat(np.arange(cfg.ncell), rng.poisson(rate)).astype(np.int32)
    n = cell.size
    parts = {"cell": cell}
    for k in ["ox", "oy"] + (["oz"] if ndim == 3 else []):
        parts[k] = rng.uniform(-0.5, 0.5, n).astype(np.float32)
    for k in ("ux", "uy", "uz"):
        parts[k] = rng.choice(np.array([-1.0, -0.5, 0.5, 1.0], np.float32), n)
    parts["w"] = (1.0 + rng.integers(0, 1 << 23, n) * 2.0 ** -23).astype(np.float32)
    sums = [np.bincount(cell, parts["w"].astype(np.float64) * f, cfg.ncell) for f in (1.0, parts["ux"], parts["uy"], parts["uz"])]
    ctx = H.Context(cfg, n)
    cs = dev(np.concatenate([[0], np.cumsum(np.bincount(cell, minlength=cfg.ncell))]), np.int32)
    nd, Jd = torch.zeros(cfg.ncell, device="cuda"), torch.zeros((3, cfg.ncell), device="cuda")
    zero = torch.zeros((3, cfg.ncell), device="cuda")
    p, q = H.Particles.from_numpy(parts, ndim), H.Particles(ndim, n)
    if call == "deposit":
        H.hvpic_deposit(ctx.ctx, p, cs, 0.0, nd, Jd)
    elif call == "push":
        H.hvpic_gather_push(ctx.ctx, p, cs, zero, zero, nd, Jd)
    else:
        H.hvpic_gather_push_perm(ctx.ctx, p, torch.arange(n, dtype=torch.int32, device="cuda"), q, cs, zero, zero, nd, Jd)
    torch.cuda.synchronize()
    look = np.arange(cfg.ncell) // cfg.nx % 6 == 4 if thin < 1 else np.ones(cfg.ncell, bool)
    got = [nd.cpu().numpy()] + list(Jd.cpu().numpy())
    for g, s in zip(got, sums):
        assert np.array_equal(g[look], s[look].astype(np.float32))


def test_bad_map_entry_is_counted_once(H):
    """A map entry outside the store, in a chunk that takes several passes:
    flagged, and counted once (in the status block at the workspace's start)."""
    announce("bad_map_entry")
    cfg = _cfg(2, W.SHAPE_QS)
    parts, E, B, _ = _uneven(cfg, 950, 90.0, 0.05)
    n = parts["cell"].size
    row = parts["cell"] // cfg.nx
    at = int(np.flatnonzero(row == 4)[0])  # the middle of a thin band
    perm = np.arange(n, dtype=np.int32)
    perm[at] = n + 5
    ctx = H.Context(cfg, n)
    p, q = H.Particles.from_numpy(parts, 2), H.Particles(2, n)
    n_mid, J_mid = torch.zeros(cfg.ncell, device="cuda"), torch.zeros((3, cfg.ncell), device="cuda")
    H.hvpic_gather_push_perm(ctx.ctx, p, dev(perm, np.int32), q, None, dev(E), dev(B), n_mid, J_mid)
    torch.cuda.synchronize()
    # flags, unused, moved_gt1, nonfinite, floor_hits, bad_input
    assert int(ctx.workspace[:40].view(torch.int64)[4]) == 1
    flags, _ = H.hvpic_sync_status(ctx.ctx)
    assert flags & H.FLAG_BAD_INPUT


def _banded(cfg, seed, ppc, thin):
    """As _uneven, the straddlers looked for on a copy (the oracle's push moves the cells of the store that it is given)."""
    _, parts, B = W.random_box(seed, cfg, 2.0 * ppc / (1.0 + thin), vmax_cells=0.9)
    rng = np.random.Generator(np.random.PCG64(seed + 1))
    keep = ((parts["cell"] // cfg.nx // 3) % 2 == 0) | (rng.uniform(size=parts["cell"].size) < thin)
    parts = {k: np.ascontiguousarray(v[keep]) for k, v in parts.items()}
    E = W.random_field(seed + 2, cfg, 0.3)
    ref = {k: v.copy() for k, v in O.particles64(parts).items()}
    O.push(cfg, ref, E, B)
    near = deposit_point_straddlers(cfg, ref, 0.0) | deposit_point_straddlers(cfg, ref, 0.5 * cfg.dt)
    parts = {k: v[~near] for k, v in parts.items()}
    perm, cs = O.sort(cfg, parts["cell"])
    return {k: np.ascontiguousarray(v[perm]) for k, v in parts.items()}, E, B, cs


def _passes(cfg, cell):
    """Window passes of every chunk of a sorted store, and the number of chunks (the library's plan, in numpy)."""
    ppc = cell.size / cfg.ncell
    if cfg.ndim == 2:
        chunk, win = (3072 if ppc >= 55 else 1024), 64
    else:
        chunk, win = 1024, (24 if ppc >= 56 else 40 if ppc >= 31 else 64)
    first = np.arange(0, cell.size, chunk)
    cells = cell[np.minimum(first + chunk, cell.size) - 1] - cell[first] + 1
    return -(-cells // (win - 4)), first.size


QS, NGP = W.SHAPE_QS, W.SHAPE_NGP
# boxes of more chunks than the GPU has CUs, whose push takes two kernels: per plan one with chunks of one and of several
# windows, and with either shape one with chunks of more than a block takes (12 with QS, 4 with NGP)
LARGE = [(2, (183, 60, 1), 90.0, 0.05, QS), (2, (183, 72, 1), 45.0, 0.05, QS), (2, (183, 60, 1), 30.0, 0.05, NGP),
         (2, (640, 640, 1), 0.8, 1.0, QS), (2, (400, 300, 1), 3.0, 1.0, NGP), (3, (19, 24, 12), 70.0, 0.05, QS),
         (3, (19, 24, 15), 45.0, 0.05, QS), (3, (19, 30, 24), 24.0, 0.05, NGP), (3, (64, 80, 80), 0.8, 1.0, QS)]


@pytest.mark.parametrize("ndim,dims,ppc,thin,shape", LARGE)
@pytest.mark.parametrize("mapped", [False, True])
def test_two_kernels_of_larger_stores(H, ndim, dims, ppc, thin, shape, mapped):
    announce("larger_stores", ndim, dims, ppc, thin, shape, mapped)
    cfg = _cfg(ndim, shape).replace(nx=dims[0], ny=dims[1], nz=dims[2])
    parts, E, B, cs0 = _banded(cfg, 970 + int(ppc), ppc, thin)
    passes, chunks = _passes(cfg, parts["cell"])
    most = 12 if shape == QS else 4
    assert chunks > 256
    if thin == 1.0:
        assert (passes > most).mean() > 0.9  # (more than a block makes: global accesses)
    else:
        assert (passes == 1).any() and ((passes > 1) & (passes <= most)).any()
    n = parts["cell"].size
    ctx = H.Context(cfg, n)
    cs_prev, cs = dev(cs0, np.int32), torch.zeros(cfg.ncell + 1, dtype=torch.int32, device="cuda")
    n_mid, J_mid = torch.full((cfg.ncell,), 7.0, device="cuda"), torch.full((3, cfg.ncell), 7.0, device="cuda")
    diag = torch.zeros(4, dtype=torch.float64, device="cuda")
    ref = {k: v.copy() for k, v in O.particles64(parts).items()}
    rd, st = O.push(cfg, ref, E, B)
    rn, rJ = O.deposit(cfg, ref, 0.5 * cfg.dt)
    rperm, rcs = O.sort(cfg, ref["cell"])
    p, q = H.Particles.from_numpy(parts, ndim), H.Particles(ndim, n)
    H.hvpic_path_stats(ctx.ctx)
    for again in range(2):  # (the list of the second kernel is empty again after the first time)
        if mapped:
            perm = torch.arange(n, dtype=torch.int32, device="cuda")
            H.hvpic_gather_push_perm(ctx.ctx, p, perm, q, cs_prev, dev(E), dev(B), n_mid, J_mid, diag)
            H.hvpic_sort_perm(ctx.ctx, q, cs_prev, perm, cs)
            torch.cuda.synchronize()
            assert np.array_equal(perm.cpu().numpy(), rperm)
            pushed = q.to_numpy()
        else:
            p = H.Particles.from_numpy(parts, ndim)
            H.hvpic_gather_push(ctx.ctx, p, cs_prev, dev(E), dev(B), n_mid, J_mid, diag)
            H.hvpic_sort(ctx.ctx, p, q, cs_prev, cs)
            pushed, ordered = p.to_numpy(), q.to_numpy()
            for k in pushed:
                assert np.array_equal(ordered[k], pushed[k][rperm]), k
        flags, counts = H.hvpic_sync_status(ctx.ctx)
        assert flags == 0 and counts[0] == st.moved_gt1 == 0
        win, glob = H.hvpic_path_stats(ctx.ctx)
        assert win + glob == chunks and glob == (passes > most).sum()
        compare_particles(cfg, pushed, ref, band=0.0)
        assert np.array_equal(cs.cpu().numpy(), rcs)
        assert rel_l2(n_mid.cpu().numpy(), rn) < 1e-5
        assert rel_l2(J_mid.cpu().numpy(), rJ) < 1e-5
        assert np.allclose(diag.cpu().numpy(), rd, rtol=1e-5, atol=1e-6 * abs(rd[0]))
    H.hvpic_deposit(ctx.ctx, H.Particles.from_numpy(pushed, ndim), None, 0.5 * cfg.dt, n_mid, J_mid)
    torch.cuda.synchronize()
    assert rel_l2(n_mid.cpu().numpy(), rn) < 1e-5
    assert rel_l2(J_mid.cpu().numpy(), rJ) < 1e-5


@pytest.mark.parametrize("ndim,ppc", [(2, 90.0), (2, 30.0), (3, 70.0), (3, 24.0)])
def test_small_stores_take_one_kernel(H, ndim, ppc):
    """A push of no more chunks than the GPU has CUs enqueues one kernel, and one more with its moments."""
    announce("one_kernel", ndim, ppc)
    cfg = _cfg(ndim, W.SHAPE_QS)
    _, parts, B = W.random_box(77, cfg, ppc)
    n = parts["cell"].size
    order = np.argsort(parts["cell"], kind="stable")
    p = H.Particles.from_numpy({k: np.ascontiguousarray(v[order]) for k, v in parts.items()}, ndim)
    ctx = H.Context(cfg, n)
    E, Bd = torch.zeros((3, cfg.ncell), device="cuda"), dev(B)
    n_mid, J_mid = torch.zeros(cfg.ncell, device="cuda"), torch.zeros((3, cfg.ncell), device="cuda")
    stream = lambda s: H.hvpic_set_stream(ctx.ctx, s)  # noqa: E731
    assert graph_nodes.count(lambda: H.hvpic_gather_push(ctx.ctx, p, None, E, Bd), stream) == 1
    assert graph_nodes.count(lambda: H.hvpic_gather_push(ctx.ctx, p, None, E, Bd, n_mid, J_mid), stream) == 2
