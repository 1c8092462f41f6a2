"""The DG kernel at the edges of its tiles (8 x 4 elements for k = 3, 7 x 6 for k = 2,
8 x 8 for k = 1): one element, whole tiles, one element more or less, grids one element
wide or high, walls and x-periodic, and states on both sides of the pressure series'
range.  Bounds: those of the operator's parity tests (a constant times the rounding
scale that the oracle gives)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2505_24504_amd import jfmg, workloads as W  # noqa: E402

from gpu_common import C_JVP, C_LH, DEV, EPS, dg_mass, lh_scale, node_total_norm, pair, rand_state, to_dev, to_np  # noqa: E402

TILE = {1: (8, 8), 2: (7, 6), 3: (8, 4)}
# grid sizes as (tiles, extra elements) in x and z
SIZES = [((0, 1), (0, 1)), ((1, 0), (1, 0)), ((1, 1), (1, 1)), ((2, -1), (1, 1)), ((0, 1), (2, 1)), ((2, 1), (0, 1))]


def setup_module(module):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    jfmg.load_library()


def _cfg(k, size, physics, bc):
    tx, tz = TILE[k]
    nx, nz = size[0][0] * tx + size[0][1], size[1][0] * tz + size[1][1]
    return W.small(nx=nx, nz=nz, k=k, physics=physics, mu=75.0 if physics else 0.0, bc=bc, background=bc,
                   N=0.01 if bc else 0.0, u_mean=20.0 if bc else 5.0, x1=1000.0 * nx, z1=1000.0 * nz, mg_levels=1)


@pytest.mark.parametrize("k", [1, 2, 3])
@pytest.mark.parametrize("size", SIZES)
@pytest.mark.parametrize("physics,bc", [(0, 0), (1, 0), (1, 1)])
def test_tile_edges(k, size, physics, bc):
    d = _cfg(k, size, physics, bc)
    print(f"case k={k} {d['nx']}x{d['nz']} physics={physics} bc={bc}", flush=True)
    p, o = pair(d)
    m = np.tile(dg_mass(d), 4)
    for rel in (1e-5, 2e-2):
        U, Ub = rand_state(o, 71, rel), rand_state(o, 72, rel)
        # the vectors one double off their allocation's alignment
        buf = torch.empty(2 * o.ndof + 2, dtype=torch.float64, device=DEV)
        Ud, Bd = buf[1:o.ndof + 1], buf[o.ndof + 1:2 * o.ndof + 1]
        Ud.copy_(to_dev(U))
        Bd.copy_(to_dev(Ub))
        for minv in (False, True):
            err = np.linalg.norm(to_np(p.residual(Ud, minv)) - o.residual(U, int(minv)))
            assert err <= C_LH * EPS * lh_scale(o, d, U, minv)
        G, nrm = p.stage_residual(Ud, Bd, 0.4)
        Go = o.stage_residual(U, Ub, 0.4)
        tol = C_LH * EPS * 0.4 * lh_scale(o, d, U, True) + 4 * EPS * (np.linalg.norm(U) + np.linalg.norm(Ub))
        assert np.linalg.norm(to_np(G) - Go) <= tol
        assert abs(nrm - np.linalg.norm(Go)) <= tol + 1e-13 * nrm
    adt = 0.9
    p.linearize(to_dev(U), adt)
    o.linearize(U, adt)
    y = rand_state(o, 73, 1.0)
    eps = np.sqrt(EPS) * node_total_norm(o, d, U)[0] / np.linalg.norm(y)
    scale = (adt / eps) * EPS * np.linalg.norm(o.residual(U, 3) / m)
    assert np.linalg.norm(to_np(p.jvp(to_dev(y))) - o.jvp(y)) <= C_JVP * scale


@pytest.mark.parametrize("k,physics", [(1, 0), (2, 1), (3, 1)])
@pytest.mark.parametrize("rel", [9e-4, 4.9e-2, 0.12])
def test_pressure_range(k, physics, rel):
    """States whose rho theta deviates by up to rel (and rel exactly at some nodes): inside
    the binomial series' range, at its end and beyond, where the power is taken."""
    d = _cfg(k, ((1, 1), (1, 1)), physics, 0)
    p, o = pair(d)
    rng = np.random.default_rng(5)
    U = rand_state(o, 74, 1e-3)
    n = o.ndof // 4
    s = rng.uniform(-rel, rel, n)
    s[::7] = rel
    U[3 * n:] = 300.0 * s
    for minv in (False, True):
        err = np.linalg.norm(to_np(p.residual(to_dev(U), minv)) - o.residual(U, int(minv)))
        assert err <= C_LH * EPS * lh_scale(o, d, U, minv)


def test_noalloc_more_tiles_than_partials():
    """The allocation-free residual on a flat grid whose tiles outnumber the scratch array's
    partial sums: the norm is then summed from G."""
    d = W.small(nx=1_100_000, nz=1, k=1, x1=1.1e8, z1=100.0, mg_levels=1, gmres_m=1)
    p, o = pair(d)
    U, Ub = rand_state(o, 75, 1e-3), rand_state(o, 76, 1e-3)
    G, nrm = p.stage_residual(to_dev(U), to_dev(Ub), 0.3)
    Gs, n2 = jfmg.stage_residual_noalloc(d, to_dev(U), to_dev(Ub), 0.3)
    tol = 2 * EPS * 0.3 * np.linalg.norm(o.residual(U, 3) / np.tile(dg_mass(d), 4))
    assert np.linalg.norm(to_np(G) - to_np(Gs)) <= tol
    assert abs(float(np.sqrt(to_np(n2)[0])) - nrm) <= 1e-13 * nrm + tol


@pytest.mark.parametrize("k", [1, 2])
def test_jvp_beyond_one_round_of_tiles(k):
    """The product's form for more tiles than run at once (its loads in another order) against
    the form for fewer: a member's steps in a lock-step batch of more than 512 tiles have the
    bits of the member alone."""
    d = W.small(nx=26, nz=21, k=k, scheme=0, dt=0.6, mg_levels=1, rk_stages=1, newton_rtol=1e-8, newton_stall=1e-7,
                gmres_m=30, x0=0.0, x1=40.0 * 26, z0=0.0, z1=40.0 * 21)
    per = -(-26 // TILE[k][0]) * -(-21 // TILE[k][1])
    members = 512 // per + 1
    perts = [dict(shape=0, amp=1.0 + 0.01 * m, xc=500.0, zc=400.0, xr=200.0, zr=200.0) for m in range(members)]
    print(f"case k={k} members={members}", flush=True)
    q = jfmg.Problem(d, device=DEV)
    U0 = [q.initial_state(p) for p in perts]
    pb = jfmg.Problem(dict(d, batch=members), device=DEV)
    U = torch.cat([u.reshape(-1) for u in U0])
    assert pb.implicit_step(U)["status"] == 0
    n = U0[0].numel()
    for m in (0, members // 2, members - 1):
        V = U0[m].clone()
        assert q.implicit_step(V)["status"] == 0
        assert not torch.equal(V, U0[m])
        assert torch.equal(V.reshape(-1), U[m * n:(m + 1) * n]), m
