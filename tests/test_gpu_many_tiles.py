"""Lists whose work-groups process several tiles each, full and cut ones in turn:
the role-split stage kernel (the next tile's loads ahead of this one's stores, the
LDS reused across tiles, square roots skipped by the running maximum) bitwise
against the general kernel and against one tile per work-group, and the adjoint
against the oracle's JVP by the dot product."""
import math

import numpy as np
import pytest

import helpers
import oracle
from paper_1407_2052_amd import amrvac as A

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)

CUS = 256


def many(ndim, mhd, periodic, blocks):
    # 2D: 6 tiles of 16x8 or 4 of 16x16 in a block of 17x17, 3 or 2 in one of
    # 16x17 or 5x17; 3D: 8 tiles of 8x8x4 in one of 9x9x5, 4 in one of 8x9x5
    widths = [17, 16, 5, 17] if ndim == 2 else [9, 8, 5, 9]
    xs = [widths[b % 4] for b in range(blocks)]
    return helpers.strip_blocks(ndim, mhd, xs, 17 if ndim == 2 else 9, 5, seed=21, periodic=periodic)


def tiles(bs, shape):
    return sum(int(np.prod([-(-int(n) // t) for n, t in zip(nn, shape)])) for nn in bs.n)


@pytest.mark.parametrize("periodic", [True, False])
@pytest.mark.parametrize("recon", [A.MP5, A.LIM03])
@pytest.mark.parametrize("ndim,mhd", [(2, False), (2, True), (3, False), (3, True)])
def test_role_split_kernel(ndim, mhd, recon, periodic):
    bs = many(ndim, mhd, periodic, 1200 if ndim == 2 else 800)
    assert tiles(bs, (16, 16, 1) if ndim == 2 else (8, 8, 4)) > 6 * 2 * CUS
    ctx, flat, views = A.context_for(bs, recon=recon)
    names = ctx.variants()
    start = flat.clone()
    roles = [i for i, n in enumerate(names) if "roles" in n]
    general = [i for i, n in enumerate(names) if "core" in n][0]
    want = {}
    for i, exec in [(general, A.EXEC_BATCHED)] + [(r, e) for r in roles for e in
                                                 (A.EXEC_BATCHED, A.EXEC_BATCHED_SINGLE, A.EXEC_PER_BLOCK)]:
        ctx.set_exec(exec)
        ctx.set_variant(i)
        assert ctx.current_variant() == names[i]
        for scheme in (A.RK3, A.SSPRK43, A.SSPRK54):
            print(f"[many tiles] {names[i]} exec={exec} scheme={scheme}", flush=True)
            flat.copy_(start)
            t = ctx.ssprk_step(scheme, 2, cfl=0.4, t=0.0)
            got = (t, flat.clone())
            ref = want.setdefault(scheme, got)
            assert got[0] == ref[0] and torch.equal(got[1], ref[1])
        flat.copy_(start)
        out, cm = ctx.fd_rhs()
        got = (cm, torch.cat([o.flatten() for o in out]))
        ref = want.setdefault("rhs", got)
        assert np.array_equal(got[0], ref[0]) and torch.equal(got[1], ref[1])
    ctx.close()


@pytest.mark.timeout(300)
@pytest.mark.parametrize("recon", [A.MP5, A.LIM03])
@pytest.mark.parametrize("ndim,mhd", [(2, True), (3, False), (3, True)])
def test_adjoint(ndim, mhd, recon):
    from test_gpu_adjoint import fixed_dt, gpu_adjoint_recon, interior_dot, random_cotangent
    from test_oracle_vjp import random_with_ghosts
    bs = many(ndim, mhd, False, 900 if ndim == 2 else 400)
    assert tiles(bs, (16, 16, 1) if ndim == 2 else (8, 8, 8)) > 2 * 2 * CUS
    print(f"[many tiles adjoint] {ndim}d mhd={mhd} recon={recon}", flush=True)
    with oracle.use_recon(recon):
        dt = fixed_dt(bs)
        lam_n = random_cotangent(bs, 31)
        tang = random_with_ghosts(bs, 3)
        _, du = oracle.run_jvp(bs, tang, oracle.SSPRK54, 1, dt)
    lam0 = gpu_adjoint_recon(bs, oracle.SSPRK54, dt, 1, 1, lam_n, recon)
    lhs = math.fsum(float(np.vdot(g, t)) for g, t in zip(lam0, tang))
    rhs = interior_dot(bs, lam_n, du)
    print(f"  {lhs!r} {rhs!r}", flush=True)
    assert abs(lhs - rhs) <= 1e-10 * abs(rhs)
