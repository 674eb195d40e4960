"""Blocks beyond the role-split kernel's 32-bit offsets (the bound lowered so that
small blocks exceed it): the general kernel runs and is reported, for steps,
right-hand sides and the adjoint's recompute, bitwise as the role-split forms;
the autotuner times it once."""
import numpy as np
import pytest

import helpers
from paper_1407_2052_amd import amrvac as A

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def outputs(bs, recon):
    ctx, flat, views = A.context_for(bs, recon=recon)
    name = ctx.current_variant()
    rhs, cm = ctx.fd_rhs()
    got = [o.cpu().numpy() for o in rhs] + [cm]
    for scheme in (A.RK3, A.SSPRK43, A.SSPRK54):
        torch.manual_seed(7)
        lam = [torch.randn(v.shape, dtype=torch.float64).cuda() for v in views]
        ctx.ssprk_adjoint(scheme, 0.2 * bs.dx[0, 0] / cm.sum(), 3, 2, lam)
        got += [x.cpu().numpy() for x in lam]
    t = ctx.ssprk_step(A.SSPRK54, 9, cfl=0.4, t=0.0)
    got += [v.cpu().numpy() for v in views] + [np.array(t)]
    ctx.close()
    return name, got


@pytest.mark.parametrize("periodic", [True, False])
@pytest.mark.parametrize("recon", [A.MP5, A.LIM03])
@pytest.mark.parametrize("ndim,mhd,xs,ny,nz", [(2, False, [17, 9], 20, 1), (2, True, [17, 9], 20, 1),
                                               (3, False, [9, 8], 10, 5), (3, True, [9, 8], 10, 5)])
def test_general_kernel_serves_and_is_reported(ndim, mhd, xs, ny, nz, recon, periodic, monkeypatch):
    bs = helpers.strip_blocks(ndim, mhd, xs, ny, nz, seed=17, periodic=periodic)
    name, want = outputs(bs, recon)
    assert "roles" in name
    # exactly at the bound, then one cell beyond it
    extent = 24 * (max(xs) + 6) + (12 * (max(xs) + 6) * (ny + 6) if ndim == 3 else 0)
    monkeypatch.setenv("AMRVAC_ROLES_MAX_OFFSET", str(extent))
    assert "roles" in outputs(bs, recon)[0]
    monkeypatch.setenv("AMRVAC_ROLES_MAX_OFFSET", str(extent - 1))
    name, got = outputs(bs, recon)
    assert "roles" not in name
    assert all(np.array_equal(a, b) for a, b in zip(want, got))


def test_choice_and_autotune_beyond_the_bound(monkeypatch):
    monkeypatch.setenv("AMRVAC_ROLES_MAX_OFFSET", str(24 * 30))
    bs = helpers.strip_blocks(2, True, [16, 40], 16, seed=17)
    ctx, flat, views = A.context_for(bs)
    names = ctx.variants()
    roles = [i for i, n in enumerate(names) if "roles" in n]
    ctx.set_variant(roles[0])
    assert "roles" not in ctx.current_variant()
    name, ms = ctx.autotune(A.RK3, 1)
    assert "roles" not in name
    assert all((m > 0) == (i not in roles) for i, m in enumerate(ms))
    # a list within the bound: a choice of the role-split form holds again
    ctx.set_variant(roles[0])
    small = helpers.strip_blocks(2, True, [16, 20], 16, seed=17)
    keep, v = A.device_blocks(small)
    ctx.set_blocks(v, small.n, small.dx, small.xlo, small.nbr)
    assert ctx.current_variant() == names[roles[0]]
    ctx.close()
