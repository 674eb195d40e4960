"""The shape a context reports is the one that runs: the one-launch form of small
1D lists at the edges of what it holds (threads in hydro, LDS in MHD, one block
and many), and where a choice, an execution form or passive blocks rule it out;
bitwise the same states from it, from every general shape and per block."""
import numpy as np
import pytest

import helpers
from paper_1407_2052_amd import amrvac as A

pytestmark = pytest.mark.gpu

# (mhd, widths, periodic, whether the one-launch form holds the list)
EDGES = [(False, [1018], False, True), (False, [1019], False, False), (False, [1024], True, True),
         (False, [8] * 125, True, True), (False, [8] * 128, True, False), (True, [598], True, True),
         (True, [599], True, False), (True, [598], False, True), (True, [16] * 30 + [13], True, True),
         (True, [16] * 30 + [14], True, False), (True, [16] * 32, True, False)]


def stepped(bs, recon, exec=A.EXEC_BATCHED, variant=None):
    ctx, flat, views = A.context_for(bs, exec=exec, recon=recon)
    if variant is not None:
        ctx.set_variant(variant)
    name = ctx.current_variant()
    t = ctx.ssprk_step(A.SSPRK54, 9, cfl=0.4, t=0.0)
    ctx.close()
    return name, (flat.cpu().numpy(), t)


@pytest.mark.parametrize("recon", [A.MP5, A.LIM03])
@pytest.mark.parametrize("mhd,xs,periodic,fits", EDGES)
def test_one_launch_form_at_its_limits(mhd, xs, periodic, fits, recon):
    bs = helpers.strip_blocks(1, mhd, xs, seed=4, periodic=periodic)
    name, got = stepped(bs, recon)
    assert ("line" in name) == fits
    pname, want = stepped(bs, recon, A.EXEC_PER_BLOCK)
    assert "line" not in pname
    names = A.context_for(bs, recon=recon)[0].variants()
    others = [stepped(bs, recon, variant=i) for i in range(len(names))]
    for i, (n, _) in enumerate(others):
        assert n == names[i] or ("line" in names[i] and not fits)
    for g in [got] + [o for _, o in others]:
        assert g[1] == want[1] and np.array_equal(g[0], want[0])


@pytest.mark.parametrize("mhd", [False, True])
def test_choice_execution_form_and_passive_blocks(mhd):
    bs = helpers.strip_blocks(1, mhd, [12, 9, 20], seed=4)
    ctx, flat, views = A.context_for(bs)
    line = ctx.current_variant()
    assert "line" in line
    ctx.set_exec(A.EXEC_PER_BLOCK)
    assert "line" not in ctx.current_variant()
    ctx.set_exec(A.EXEC_BATCHED_SINGLE)
    assert ctx.current_variant() == line
    ctx.set_active([1, 0, 1])
    assert "line" not in ctx.current_variant()
    ctx.ssprk_step(A.RK3, 2, t=0.0)
    ctx.set_active(None)
    assert ctx.current_variant() == line
    ctx.set_variant(0)
    assert ctx.current_variant() == ctx.variants()[0] != line
    ctx.set_variant(ctx.variants().index(line))
    assert ctx.current_variant() == line
    # another list: the choice stands and runs where it fits
    big = helpers.strip_blocks(1, mhd, [700, 600], seed=4)
    keep, v = A.device_blocks(big)
    ctx.set_blocks(v, big.n, big.dx, big.xlo, big.nbr)
    assert "line" not in ctx.current_variant()
    ctx.set_blocks(views, bs.n, bs.dx, bs.xlo, bs.nbr)
    assert ctx.current_variant() == line
    ctx.close()


@pytest.mark.parametrize("recon", [A.MP5, A.LIM03])
@pytest.mark.parametrize("mhd", [False, True])
def test_autotune_times_the_form_that_runs(mhd, recon):
    for xs, fits in (([64] * 8, True), ([700, 600], False)):
        bs = helpers.strip_blocks(1, mhd, xs, seed=4)
        ctx, flat, views = A.context_for(bs, recon=recon)
        before = flat.clone()
        name, ms = ctx.autotune(A.SSPRK54, 16)
        assert (flat == before).all()
        print(mhd, recon, xs, dict(zip(ctx.variants(), ms)), flush=True)
        for n, m in zip(ctx.variants(), ms):
            assert (m > 0) == (fits or "line" not in n)
        assert name == ctx.current_variant() == ctx.variants()[ms.index(min(m for m in ms if m > 0))]
        ctx.close()
