"""The adjoint on lists with fixed and mixed faces and tiles cut by the block's
end, for both reconstructions, hydro and MHD in 1D to 3D and every scheme:
element by element against the oracle's reverse mode, the boundary data's
adjoint included."""
import numpy as np
import pytest

import helpers
import oracle
from paper_1407_2052_amd import amrvac as A

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)

from test_gpu_adjoint import fixed_dt, gpu_adjoint_recon, random_cotangent  # noqa: E402

# block widths, ny, nz: one full tile in 2D, cut tiles, several tiles a block
GRIDS = {1: [([40, 9], 1, 1)], 2: [([16, 16], 16, 1), ([17, 9], 20, 1)], 3: [([9, 8], 10, 5)]}


@pytest.mark.parametrize("scheme", [oracle.RK3, oracle.SSPRK43, oracle.SSPRK54])
@pytest.mark.parametrize("recon", [A.MP5, A.LIM03])
@pytest.mark.parametrize("mhd", [False, True])
@pytest.mark.parametrize("ndim,xs,ny,nz", [(d, *g) for d in GRIDS for g in GRIDS[d]])
def test_fixed_faces_against_the_oracle(ndim, xs, ny, nz, mhd, recon, scheme):
    print(f"[adjoint fixed] {ndim}d {xs} mhd={mhd} recon={recon} scheme={scheme}", flush=True)
    # seed: no two cells within rounding of each other as the maximiser of c_max
    bs = helpers.strip_blocks(ndim, mhd, xs, ny, nz, seed=13, periodic=False)
    if ndim == 3:   # mixed: periodic along y
        for b in range(bs.nb):
            bs.nbr[b, 2] = bs.nbr[b, 3] = b
    with oracle.use_recon(recon):
        dt = fixed_dt(bs)
        lam_n = random_cotangent(bs, 31)
        ref = oracle.run_vjp(bs, lam_n, scheme, 2, dt)
    got = gpu_adjoint_recon(bs, scheme, dt, 2, 1, lam_n, recon)
    scale = max(float(np.abs(r).max()) for r in ref)
    worst = max(float(np.abs(g - r).max()) for g, r in zip(got, ref))
    print(f"  max |gpu - oracle| / max |oracle| = {worst / scale:.2e}", flush=True)
    assert worst <= 1e-10 * scale
