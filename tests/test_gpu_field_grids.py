"""GPU parity of the 2D field advance on grids at the edges of its choices,
against the FP64 oracle: above and below the size from which the substeps with
hyper-resistivity, the energy equation or open boundaries take tiles of 16 rows;
grids too narrow for tiles, which take their stages one by one; more tiles
than finish their diagnostics in the last block.

Tolerances as for the other field tests: B, E and p_e within 1e-5 relative L2,
the diagnostics by check_field_diag."""
import numpy as np
import pytest

import oracle as O
from paper_2305_05600_amd import workloads as W
from tests import graph_nodes
from tests.helpers import announce, check_field_diag, rel_l2

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def H():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2305_05600_amd import hvpic

    hvpic.lib()
    return hvpic


def _cfg(nx, ny, **kw):
    base = dict(name="grids", ndim=2, nx=nx, ny=ny, nz=1, dx=0.5, dy=0.3, dz=1.0, dt=0.05, nsub=3, te=0.2, eta=1e-3)
    base.update(kw)
    return W.Config(**base)


HYPER = dict(eta_h=2e-3, gamma_e=5.0 / 3.0)
ENERGY = dict(gamma_e=5.0 / 3.0, energy_eq=1, kappa0=0.05, eta_h=2e-3)
OPEN = dict(open_x=1, buffer_cells=2, eta_h_buffer=0.05)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()


def _check(H, cfg, seed=701):
    """One advance against the oracle; the number of kernels it takes."""
    B = W.random_field(seed, cfg, 0.2, (1.0, 0.3, -0.2))
    nh, npv = W.random_density(seed + 1, cfg, 0.02, 1.5), W.random_density(seed + 2, cfg, 0.5, 1.5)
    Jh, Jp = W.random_field(seed + 3, cfg, 0.2), W.random_field(seed + 4, cfg, 0.2)
    pe = W.random_density(seed + 5, cfg, 0.1, 0.4)
    ctx = H.Context(cfg, 1)
    E, diag = torch.zeros((3, cfg.ncell), device="cuda"), torch.zeros(3, dtype=torch.float64, device="cuda")
    Bd, ped, Bt = dev(B), dev(pe), torch.zeros((3, cfg.ncell), device="cuda")
    if cfg.open_x:
        B0 = np.zeros_like(B)
        B0[1] = 1.0
        nh, npv, Jh, Jp, B = (O.open_fill(cfg, a) for a in (nh, npv, Jh, Jp, B))
        Bd = dev(B)
        b0, ins = dev(B0), [dev(a) for a in (nh, Jh, npv, Jp)]
        call = lambda: H.hvpic_open_field_advance(ctx.ctx, b0, Bd, Bt, *ins, E, 0, diag)  # noqa: E731
        call()
        rB, rE, _, rd, _ = O.open_field_advance(cfg, B0, B, nh, Jh, npv, Jp, mode=0)
    else:
        ins = [dev(a) for a in (nh, Jh, npv, Jp)]
        if cfg.energy_eq:
            call = lambda: H.hvpic_field_advance_pe(ctx.ctx, Bd, ped, *ins, E, 0, diag)  # noqa: E731
            call()
            rB, rpe, rE, rd, _ = O.field_advance_pe(cfg, B, pe, nh, Jh, npv, Jp, mode=0)
            assert rel_l2(ped.cpu().numpy(), rpe) < 1e-5
        else:
            call = lambda: H.hvpic_field_advance(ctx.ctx, Bd, *ins, E, 0, diag)  # noqa: E731
            call()
            rB, rE, rd, _ = O.field_advance(cfg, B, nh, Jh, npv, Jp, mode=0)
    assert rel_l2(Bd.cpu().numpy(), rB) < 1e-5
    assert rel_l2(E.cpu().numpy(), rE) < 1e-5
    check_field_diag(diag.cpu().numpy(), rd)
    return graph_nodes.count(call, lambda s: H.hvpic_set_stream(ctx.ctx, s))


# 32 x 8 tiles: 14 * 41 = 574 and 13 * 39 = 507, either side of the 512 from which they have 16 rows; 512 and 544 exactly
@pytest.mark.parametrize("nx,ny", [(421, 331), (402, 311), (512, 256), (512, 265)])
@pytest.mark.parametrize("kind", ["hyper", "energy", "open"])
@pytest.mark.parametrize("nsub", [2, 3])
def test_tiles_of_either_height(H, nx, ny, kind, nsub):
    announce("tile_rows", nx, ny, kind, nsub)
    cfg = _cfg(nx, ny, nsub=nsub, **dict(hyper=HYPER, energy=ENERGY, open=OPEN)[kind])
    n = _check(H, cfg)
    assert n <= nsub + 4  # a kernel per substep, the final ones and the ghosts' first fill


# eight rows and fewer: no taller tiles, however many
@pytest.mark.parametrize("nx,ny", [(17001, 8), (20011, 3)])
@pytest.mark.parametrize("kind", ["hyper", "energy", "open"])
def test_flat_grids(H, nx, ny, kind):
    announce("flat", nx, ny, kind)
    _check(H, _cfg(nx, ny, **dict(hyper=HYPER, energy=ENERGY, open=OPEN)[kind]))


@pytest.mark.parametrize("nx,ny", [(4, 40003), (8, 50001)])
@pytest.mark.parametrize("kind", ["hyper", "energy", "open"])
def test_narrow_grids_take_their_stages(H, nx, ny, kind):
    announce("narrow", nx, ny, kind)
    cfg = _cfg(nx + (2 if kind == "open" else 0), ny, **dict(hyper=HYPER, energy=ENERGY, open=OPEN)[kind])
    assert _check(H, cfg) >= 6 * cfg.nsub  # six kernels a substep


@pytest.mark.parametrize("nx,ny", [(600, 500), (1024, 256), (1025, 256)])
@pytest.mark.parametrize("nsub", [2, 3, 4])
def test_diagnostics_of_many_tiles(H, nx, ny, nsub):
    """1197, 1024 and 1056 tiles: either side of the 1024 whose diagnostics the last block finishes."""
    announce("many_tiles", nx, ny, nsub)
    _check(H, _cfg(nx, ny, nsub=nsub))
