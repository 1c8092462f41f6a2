"""The FV operator's tile kernels at the edges of their tiles: levels narrower than a
tile, one cell more or less than whole tiles, single rows, walls and x-periodic (the
wrapped halo column), and more partial sums of ||x||^2 than a wave holds.  Bound: the
matvec's parity bound."""
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
