"""The role-split stage kernel (2D and 3D) against the general stage kernel on
the same lists: bitwise the same states where tiles are cut by the block's end
(one cell, one short of a tile, one over, halos that reach past the block into
its neighbour), for periodic and fixed faces, every scheme and a right-hand
side."""
import numpy as np
import pytest

import helpers
from paper_1407_2052_amd import amrvac as A

pytestmark = pytest.mark.gpu


def run(bs, variant, scheme, recon, rhs):
    ctx, flat, views = A.context_for(bs, recon=recon)
    ctx.set_variant(variant)
    name = ctx.current_variant()
    if rhs:
        out, cm = ctx.fd_rhs()
        got = [o.cpu().numpy() for o in out] + [cm]
    else:
        ctx.ssprk_step(scheme, 3, cfl=0.4, t=0.0)
        got = [v.cpu().numpy() for v in views]
    ctx.close()
    return name, got


@pytest.mark.parametrize("recon", [A.MP5, A.LIM03])
@pytest.mark.parametrize("ndim,mhd", [(2, False), (2, True), (3, False), (3, True)])
@pytest.mark.parametrize("xs,ny,nz,periodic", [([3, 17, 16], 15, 5, True), ([9, 8, 10], 17, 4, True),
                                               ([1 + 16, 33], 3, 9, False), ([7], 16, 3, True)])
def test_bitwise_the_general_kernel(ndim, mhd, recon, xs, ny, nz, periodic):
    bs = helpers.strip_blocks(ndim, mhd, xs, ny, nz, seed=11, periodic=periodic)
    names = A.context_for(bs, recon=recon)[0].variants()
    roles = [i for i, n in enumerate(names) if "roles" in n]
    general = [i for i, n in enumerate(names) if "roles" not in n]
    assert roles and general
    for scheme, rhs in ((A.SSPRK54, False), (A.SSPRK43, False), (A.RK3, False), (A.RK3, True)):
        _, want = run(bs, general[0], scheme, recon, rhs)
        for i in roles:
            name, got = run(bs, i, scheme, recon, rhs)
            print(name, scheme, rhs, flush=True)
            assert all(np.array_equal(a, b) for a, b in zip(want, got)), name
