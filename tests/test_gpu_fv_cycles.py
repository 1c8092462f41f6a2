"""FV cycles where the kernels' routes and shapes meet their edges: three coarse levels in one
launch, sweep counts that differ or are single, every tile shape on levels that are not whole
tiles, in both precisions.  References: the FP64 oracle, and the same step by other kernels."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
from paper_2505_24504_amd import jfmg, workloads as W  # noqa: E402

from gpu_common import DEV, REL_MG_FV, rand_state, to_dev, to_np  # noqa: E402

REL_MG_FV_FP32 = 2e-3   # FD step sqrt(2^-23) ||u||/||x||: truncation of some 3e-4 per product
REL_SHAPES_FP32 = 1e-6  # shapes change the order of the FP64 norm sums, which the FP32 step rounds away


def setup_module(module):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    jfmg.load_library()


def _cycle_cfg(k, nx, nz, levels, stages, bc, physics, key, prec):
    return W.small(nx=nx, nz=nz, k=k, bc=bc, physics=physics, mu=75.0 if physics else 0.0, background=bc,
                   N=0.01 if bc else 0.0, u_mean=10.0 if bc else 0.0, mg_levels=levels, mg_key=key, rk_stages=stages,
                   mg_precision=prec, x0=0.0, x1=500.0 * nx, z0=0.0, z1=250.0 * nz)


def _cycle_errors(d, tiles):
    """Relative errors of the FV cycle against the oracle's, per entry of tiles, and the results."""
    o = oracle.Oracle(dict(d, mg_precision=64))
    U = rand_state(o, 91)
    b = W.random_state(o.fv_size(0), 92, [1e-3, 1.0, 1.0, 0.3])
    o.linearize(U, 0.8)
    want = o.mg_fv(b)
    p = jfmg.Problem(d, device=DEV)
    errs, res = [], []
    for t in tiles:
        p.set_tiles([t] * d["mg_levels"])
        p.linearize(to_dev(U), 0.8)
        res.append(to_np(p.mg_fv(to_dev(b, p.fv_dtype))))
        errs.append(np.linalg.norm(res[-1] - want) / np.linalg.norm(want))
    return errs, res


# (k, nx, nz, levels, stages, bc, physics, key, precision).  Coarse levels in one launch: 16x8,
# 8x4 and 4x2 cells; 32x8, 16x4 and 8x2 (608 of the 640 threads have a face); 18x12 and 9x6,
# x-periodic, behind 36x24; 12x20, 6x10 and 3x5
ONE_LAUNCH = [(1, 16, 8, 4, 1, 0, 0, "mg002222V", 64), (1, 16, 8, 4, 3, 0, 1, "mg002222V", 32),
              (1, 16, 8, 4, 1, 0, 0, "mg001111V", 32), (1, 16, 8, 4, 3, 1, 0, "mg001112V", 64),
              (1, 32, 8, 4, 1, 1, 1, "mg002221V", 64), (1, 32, 8, 4, 2, 0, 1, "mg001113V", 32),
              (2, 24, 16, 4, 1, 1, 1, "mg002231V", 64), (3, 6, 10, 4, 1, 0, 1, "mg001121V", 64),
              (3, 6, 10, 4, 4, 1, 0, "mg002212V", 32)]


@pytest.mark.parametrize("case", ONE_LAUNCH)
def test_one_launch_levels_against_the_oracle(case):
    d = _cycle_cfg(*case)
    print(f"case {case}", flush=True)
    (err,), _ = _cycle_errors(d, ["8x4"])
    print(f"rel err {err:.3e}", flush=True)
    assert err <= (REL_MG_FV if case[-1] == 64 else REL_MG_FV_FP32)


@pytest.mark.parametrize("case", ONE_LAUNCH)
def test_one_launch_levels_keep_the_bits(case):
    """A member's step is the same to the bit alone, where its coarse levels go in one launch,
    and in a ragged batch with a member whose levels do not fit (its coarsest: 384 cells or
    more), where each takes its own kernels."""
    k, nx, nz, levels, stages, bc, physics, key, prec = case
    h = 50.0
    d = W.small(nx=nx, nz=nz, k=k, bc=bc, physics=physics, mu=75.0 if physics else 0.0, scheme=0, dt=0.015 * h,
                mg_levels=levels, rk_stages=stages, mg_key=key, mg_precision=prec, newton_rtol=1e-8,
                newton_stall=1e-7, gmres_m=30, x0=0.0, x1=h * nx, z0=0.0, z1=h * nz)
    members = [dict(d, nx=96, nz=64, x1=h * 96, z1=h * 64), d]
    pert = [dict(shape=0, amp=2.0, xc=48 * h, zc=30 * h, xr=20 * h, zr=20 * h),
            dict(shape=0, amp=2.0, xc=h * nx / 2, zc=h * nz / 2, xr=h * nx / 3, zr=h * nz / 3)]
    print(f"case {case}", flush=True)
    pb = jfmg.Problem(members, device=DEV)
    pb.set_tiles(["8x4"] * levels)
    U0 = [jfmg.Problem(m, device=DEV).initial_state(q) for m, q in zip(members, pert)]
    U = torch.cat(U0)
    assert pb.implicit_step(U)["status"] == 0
    q = jfmg.Problem(d, device=DEV)
    q.set_tiles(["8x4"] * levels)
    V = U0[1].clone()
    q.profile_enable(["fv_stage_small"])
    st = q.implicit_step(V)
    # one launch per cycle for the coarse levels (more products than timed launches)
    assert q.profile_read()["fv_stage_small"]["launches"] < sum(st["fv_matvecs"])
    assert st["status"] == 0 and not torch.equal(V, U0[1])
    assert torch.equal(V, U[pb.member_slices()[1]])


# (k, nx, nz, levels, stages, bc, physics, key): 154x78 and 77x39 cells (400 tiles of 8x4);
# 102x42 and 51x21; 52x20, 26x10 and 13x5
RAGGED = [(1, 77, 39, 2, 1, 1, 1, "mg002222V"), (1, 77, 39, 2, 3, 0, 0, "mg001111V"),
          (2, 34, 14, 2, 1, 1, 0, "mg002222V"), (3, 13, 5, 3, 1, 0, 1, "mg002211W"), (3, 13, 5, 3, 2, 1, 1, "mg002222V")]


@pytest.mark.parametrize("prec", [32, 64])
@pytest.mark.parametrize("case", RAGGED)
def test_cycle_on_ragged_tiles(case, prec):
    """Stage, defect, correction and transfer of every tile shape on levels that are not whole
    tiles."""
    d = _cycle_cfg(*case, prec)
    print(f"case {case} fp{prec}", flush=True)
    errs, res = _cycle_errors(d, jfmg.TILES)
    print("rel err " + " ".join(f"{t} {e:.2e}" for t, e in zip(jfmg.TILES, errs)), flush=True)
    assert max(errs) <= (REL_MG_FV if prec == 64 else REL_MG_FV_FP32)
    if prec == 32:
        for t, r in zip(jfmg.TILES, res):
            assert np.linalg.norm(r - res[0]) <= REL_SHAPES_FP32 * np.linalg.norm(res[0]), t


@pytest.mark.parametrize("size", [(1, 1, 1), (1, 4, 2), (1, 33, 3), (2, 3, 1), (2, 21, 3), (3, 17, 1)])
@pytest.mark.parametrize("bc,physics", [(0, 1), (1, 0)])
def test_matvec_tile_edges_fp32(size, bc, physics):
    """The FP32 operator of every tile shape on levels narrower than a tile and of single rows."""
    k, nx, nz = size
    d = W.small(nx=nx, nz=nz, k=k, bc=bc, physics=physics, mu=75.0 if physics else 0.0, background=bc,
                N=0.01 if bc else 0.0, u_mean=10.0 if bc else 0.0, mg_levels=1, x1=500.0 * nx, z1=500.0 * nz,
                mg_precision=32)
    print(f"case {size} bc={bc} physics={physics}", flush=True)
    p, o = jfmg.Problem(d, device=DEV), oracle.Oracle(dict(d, mg_precision=64))
    U = rand_state(o, 81, 1e-3)
    adt = 0.5
    o.linearize(U, adt)
    rng = np.random.default_rng(82)
    x = rng.standard_normal(o.fv_size(0)) * np.repeat([1e-2, 1.0, 1.0, 3.0], o.fv_size(0) // 4)
    want = o.fv_matvec(0, x)
    scale = np.linalg.norm(want - x) + np.linalg.norm(x)
    first = None
    for tile in jfmg.TILES:
        p.set_tiles([tile])
        p.linearize(to_dev(U), adt)
        got = to_np(p.fv_matvec(0, to_dev(x, torch.float32)))
        first = got if first is None else first
        assert np.linalg.norm(got - want) <= REL_MG_FV_FP32 * scale, tile
        assert np.linalg.norm(got - first) <= REL_SHAPES_FP32 * scale, tile
