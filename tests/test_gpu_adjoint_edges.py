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


def test_refusal_counts_the_tables():
    """A checkpoint interval whose stage states cannot fit is refused before
    anything is allocated, with the tables among the figures: 512 + 16 bytes a
    tile of the recompute, 448 + 16 + 24 a tile of the VJP, the ghost cells'
    adjoint, and 24 bytes a stage state for its c_max."""
    bs = helpers.strip_blocks(3, True, [9] * 256, 9, 5, seed=13, periodic=False)
    ctx, flat, views = A.context_for(bs)
    lam = [torch.zeros_like(v) for v in views]
    free, _ = torch.cuda.mem_get_info()
    # a stage state: 64 bytes a cell of the slot and 3 code words
    k = int(1.2 * free / (5 * 256 * 9 * 9 * 5 * (64 + 24)))
    with pytest.raises(A.AmrvacError) as e:
        ctx.ssprk_adjoint(A.SSPRK54, 1e-4, k, k, lam)
    ctx.close()
    assert e.value.status == A.ERR_NOMEM
    ghosts = 256 * 2 * 3 * (9 * 5 + 9 * 9) + 2 * 3 * 9 * 5
    want = 256 * (8 * (512 + 16) + 4 * (448 + 16 + 24)) + 64 * ghosts + 24 * 5 * k
    assert f"{want / 1e9:.4f} GB of tables" in str(e.value)
