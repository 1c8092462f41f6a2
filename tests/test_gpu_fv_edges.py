"""The FV operator's tile kernels at the edges of their tiles: levels narrower than a
tile, one cell more or less than whole tiles, single rows, walls and x-periodic (the
wrapped halo column), in the FP64 matvec, whose ||x||^2 is one finished sum, against its
parity bound; steps with more partial sums of ||x||^2 than a consumer adds up; and the
coarsest levels in one launch."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2505_24504_amd import jfmg, workloads as W  # noqa: E402

from gpu_common import C_FV, fv_scale, pair, rand_state, to_dev, to_np  # noqa: E402

# (k, nx, nz): finest levels of (k + 1) nx x (k + 1) nz cells
SIZES = [(1, 1, 1), (1, 4, 2), (1, 33, 3), (2, 3, 1), (2, 21, 3), (3, 17, 1), (1, 160, 60)]


def setup_module(module):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    jfmg.load_library()


@pytest.mark.parametrize("size", SIZES)
@pytest.mark.parametrize("bc,physics", [(0, 1), (1, 0)])
def test_matvec_tile_edges(size, bc, physics):
    k, nx, nz = size
    d = W.small(nx=nx, nz=nz, k=k, bc=bc, physics=physics, mu=75.0 if physics else 0.0, background=bc,
                N=0.01 if bc else 0.0, u_mean=10.0 if bc else 0.0, mg_levels=1, x1=500.0 * nx, z1=500.0 * min(nz, 20))
    print(f"case {size} bc={bc} physics={physics}", flush=True)
    p, o = pair(d)
    U = rand_state(o, 81, 1e-3)
    adt = 0.5
    o.linearize(U, adt)
    rng = np.random.default_rng(82)
    x = rng.standard_normal(o.fv_size(0)) * np.repeat([1e-2, 1.0, 1.0, 3.0], o.fv_size(0) // 4)
    want = o.fv_matvec(0, x)
    tol = C_FV * fv_scale(o, d, 0, o.fv_level_state(0), x, adt)
    for tile in jfmg.TILES:
        p.set_tiles([tile])
        p.linearize(to_dev(U), adt)
        err = np.linalg.norm(to_np(p.fv_matvec(0, to_dev(x))) - want)
        assert err <= tol, (tile, err, tol)


@pytest.mark.parametrize("prec", [32, 64])
def test_partials_summed_before_their_consumers(prec):
    """More than 3072 partial sums of ||x||^2 (the density current's 1024 x 256 cells in 8x4
    tiles: 8192) are added up by a kernel before their consumers.  A small member of a ragged
    batch, whose partials then go that way too, keeps the bits that it has alone, where each
    consumer adds them itself; the large one agrees with its step in 64x4 tiles (1024
    partials) as two steps do whose Newton iterations stop at the same relative residual: to
    ten times that residual, relative to the update."""
    a, pert, _ = W.density_current()
    a = dict(a, mg_precision=prec)
    b = dict(a, nx=64, nz=16)
    tiles = ["8x4"] * a["mg_levels"]
    pb = jfmg.Problem([a, b], device="cuda:0")
    pb.set_tiles(tiles)
    U0 = [jfmg.Problem(m, device="cuda:0").initial_state(pert) for m in (a, b)]
    U = torch.cat(U0)
    assert pb.implicit_step(U)["status"] == 0
    parts = [U[s] for s in pb.member_slices()]
    for i, (m, shapes) in enumerate([(a, ["64x4"] * len(tiles)), (b, tiles)]):
        q = jfmg.Problem(m, device="cuda:0")
        q.set_tiles(shapes)
        V = U0[i].clone()
        assert q.implicit_step(V)["status"] == 0
        rel = float((V - parts[i]).norm() / (V - U0[i]).norm())
        print(f"fp{prec} member {i}: rel(update) {rel:.3e}", flush=True)
        assert torch.equal(V, parts[i]) if i else rel <= 10 * a["newton_rtol"]


# (k, nx, nz, levels, stages, bc, physics, precision): the coarser levels, small enough for one
# launch of one work-group, are 16x16 and 8x8 cells; 18x6 (behind 36x12, which is too large);
# 12x4 and 6x2, x-periodic; 18x12 and 9x6 (behind 36x24); 2x2, less than a tile
TAILS = [(1, 16, 16, 3, 3, 0, 0, 64), (2, 24, 8, 3, 1, 0, 1, 32), (3, 6, 2, 3, 1, 1, 0, 64), (2, 24, 16, 4, 2, 1, 1, 32),
         (1, 2, 2, 2, 1, 0, 0, 64)]


@pytest.mark.parametrize("case", TAILS)
def test_coarse_levels_in_one_launch(case):
    """The coarsest levels of a V-cycle go in one launch where all members' fit; in a ragged
    batch with a member whose levels do not, each level takes its own kernels.  A member's step
    has the same bits either way."""
    k, nx, nz, levels, stages, bc, physics, prec = case
    h = 50.0
    d = W.small(nx=nx, nz=nz, k=k, bc=bc, physics=physics, mu=75.0 if physics else 0.0, scheme=0, dt=0.015 * h,
                mg_levels=levels, rk_stages=stages, mg_precision=prec, newton_rtol=1e-8, newton_stall=1e-7, gmres_m=30,
                x0=0.0, x1=h * nx, z0=0.0, z1=h * nz)
    big = dict(d, nx=96, nz=64, x1=h * 96, z1=h * 64)
    members = [(big, dict(shape=0, amp=2.0, xc=48 * h, zc=30 * h, xr=20 * h, zr=20 * h)),
               (d, dict(shape=0, amp=2.0, xc=h * nx / 2, zc=h * nz / 2, xr=h * nx / 3, zr=h * nz / 3))]
    print(f"case {case}", flush=True)
    pb = jfmg.Problem([m for m, _ in members], device="cuda:0")
    tiles = ["8x4"] * levels
    pb.set_tiles(tiles)
    U0 = [jfmg.Problem(m, device="cuda:0").initial_state(pert) for m, pert in members]
    U = torch.cat(U0)
    assert pb.implicit_step(U)["status"] == 0
    q = jfmg.Problem(d, device="cuda:0")
    q.set_tiles(tiles)
    V = U0[1].clone()
    assert q.implicit_step(V)["status"] == 0
    assert not torch.equal(V, U0[1])
    assert torch.equal(V, U[pb.member_slices()[1]])
