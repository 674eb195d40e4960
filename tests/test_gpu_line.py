"""Whole runs of a small 1D list in one launch against the stage kernels, one
launch per block and stage: bitwise the same states and end time, for blocks
at the limits of the form (3 cells, a block that is its own neighbour, cells in
the halos of both neighbours, one work-group full to the last thread and one
cell too many), periodic and fixed faces, and more steps than one launch takes."""
import numpy as np
import pytest

import helpers
from paper_1407_2052_amd import amrvac as A

pytestmark = pytest.mark.gpu

LISTS = [([3], True), ([4, 3], False), ([3, 5, 4, 9], True), ([64] * 8, True), ([7, 31, 100], False), ([512], True),
         ([634], False), ([635], False), ([1018], False), ([1019], False)]


@pytest.mark.parametrize("recon", [A.MP5, A.LIM03])
@pytest.mark.parametrize("mhd", [False, True])
@pytest.mark.parametrize("xs,periodic", LISTS)
def test_bitwise_the_stage_kernels(xs, periodic, mhd, recon):
    bs = helpers.strip_blocks(1, mhd, xs, seed=3, periodic=periodic)
    for scheme in (A.RK3, A.SSPRK43, A.SSPRK54):
        for dt in (None, 1e-4):
            got = []
            for form in (A.EXEC_BATCHED, A.EXEC_PER_BLOCK):
                ctx, flat, views = A.context_for(bs, exec=form, recon=recon)
                t = ctx.ssprk_step(scheme, 66, cfl=0.4, dt=dt, t=0.25)
                got.append((flat.cpu().numpy(), t))
                ctx.close()
            assert got[0][1] == got[1][1]
            assert np.array_equal(got[0][0], got[1][0])


def test_a_non_physical_state_is_reported():
    bs = helpers.strip_blocks(1, False, [16, 16], seed=3)
    bs.interior(1)[0, ..., 5] = -1.0
    ctx, flat, views = A.context_for(bs)
    with pytest.raises(A.AmrvacError) as e:
        ctx.ssprk_step(A.RK3, 1, t=0.0)
    assert e.value.status == A.ERR_NONPHYSICAL
    ctx.close()
