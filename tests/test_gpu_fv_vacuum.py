"""The FP32 FV operator at states whose pressure rounds to zero."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2505_24504_amd import jfmg, workloads as W  # noqa: E402

from gpu_common import pair, to_dev  # noqa: E402


def setup_module(module):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    jfmg.load_library()


@pytest.mark.parametrize("u", [0.0, 50.0, -50.0])
@pytest.mark.parametrize("tile", jfmg.TILES)
def test_zero_pressure(u, tile):
    """rho theta is 2e-6 of the (uniform, g = 0) background's in a block of elements moving with
    one velocity: (2e-6)^gamma is 1e-8, so that p - pb rounds to -pb in FP32 and the pressure,
    and with it the speed of sound, to zero.  Between two such cells the flux is the physical
    one of either side, and all of the operator is finite."""
    k, n, h = 1, 12, 10.0
    d = W.small(nx=n, nz=n, k=k, mg_levels=1, mg_precision=32, x1=h * n, z1=h * n, g=0.0)
    p, o = pair(d)
    n1 = k + 1
    U = np.zeros((4, n, n, n1, n1))
    blk = slice(3, 9)
    xi = np.polynomial.legendre.leggauss(n1)[0]
    for ez in range(3, 9):
        for b in range(n1):
            Ub, _ = o.background((ez + 0.5 * (1 + xi[b])) * h)
            U[1, ez, blk, b, :] = Ub[0] * u
            U[3, ez, blk, b, :] = -Ub[3] * (1.0 - 2e-6)
    p.set_tiles([tile])
    p.linearize(to_dev(U.reshape(-1)), 1e-3)
    x = np.zeros((4, n1 * n, n1 * n))
    x[3, :4] = 1.0
    out = p.fv_matvec(0, to_dev(x.reshape(-1), torch.float32))
    assert torch.isfinite(out).all()
    # where neither a cell nor its neighbours change, g'x = x = 0
    inner = out.reshape(4, n1 * n, n1 * n)[:, n1 * 3 + 1:n1 * 9 - 1, n1 * 3 + 1:n1 * 9 - 1]
    assert torch.count_nonzero(inner).item() == 0
