"""The general tile shapes keep their positions and names, which callers pass to
set_variant and tuning files hold: the first shapes of every context, each
accepted, and a file that names one of them reused without timing."""
import numpy as np
import pytest

import helpers
from paper_1407_2052_amd import amrvac as A, inputs

pytestmark = pytest.mark.gpu

RUNS1, CORE1 = "64x1x1-nt64-g1-w1-runs", "64x1x1-nt64-g1-w1-runs-core"
# (ndim, physics, reconstruction, eta_h): the shapes in order, without the prefix
SHAPES = {
    (1, A.HD, A.MP5, 0): ["128x1x1-nt128-g1-w1", "64x1x1-nt64-g1-w1", CORE1],
    (1, A.MHD, A.MP5, 0): ["128x1x1-nt128-g1-w1", "64x1x1-nt64-g1-w1", RUNS1, CORE1],
    (2, A.HD, A.MP5, 0): ["16x16x1-nt256-g1-w1", "16x16x1-nt256-g1-w3", "32x8x1-nt256-g1-w1",
                          "16x16x1-nt256-g1-w1-runs", "16x16x1-nt256-g1-w2-runs-core"],
    (2, A.MHD, A.MP5, 0): ["16x16x1-nt256-g2-w1", "16x16x1-nt256-g1-w1", "16x16x1-nt256-g2-w3",
                           "32x8x1-nt256-g2-w1", "16x16x1-nt256-g1-w1-runs", "16x16x1-nt256-g2-w2-runs",
                           "16x16x1-nt256-g1-w2-runs-core", "16x16x1-nt256-g2-w2-runs-core"],
    (3, A.HD, A.MP5, 0): ["8x8x4-nt256-g1-w2-runs-core", "8x8x8-nt512-g2-w1", "8x8x4-nt256-g1-w1",
                          "8x8x4-nt256-g1-w2-runs"],
    (3, A.MHD, A.MP5, 0): ["8x8x8-nt512-g1-w2-runs-core", "8x8x4-nt256-g1-w2-runs-core",
                           "8x4x4-nt128-g1-w2-runs-core", "8x8x4-nt256-g2-w3-runs-core", "8x8x4-nt256-g2-w4-runs",
                           "8x8x4-nt256-g2-w3-runs", "8x8x8-nt512-g2-w4-runs", "8x8x4-nt256-g1-w2-runs",
                           "8x8x4-nt256-g2-w3"],
    (1, A.HD, A.LIM03, 0): ["128x1x1-nt128-g1-w1-lim03", "64x1x1-nt64-g1-w1-lim03"],
    (1, A.MHD, A.LIM03, 0): [RUNS1 + "-lim03", "64x1x1-nt64-g1-w1-runs-lim03-core", "128x1x1-nt128-g1-w1-lim03",
                             "64x1x1-nt64-g1-w1-lim03"],
    (2, A.HD, A.LIM03, 0): ["16x16x1-nt256-g1-w1-runs-lim03", "16x16x1-nt256-g1-w2-runs-lim03-core",
                            "16x16x1-nt256-g1-w1-lim03", "32x8x1-nt256-g1-w1-lim03"],
    (2, A.MHD, A.LIM03, 0): ["16x16x1-nt256-g1-w1-runs-lim03", "16x16x1-nt256-g2-w2-runs-lim03",
                             "16x16x1-nt256-g1-w2-runs-lim03-core", "16x16x1-nt256-g2-w1-lim03",
                             "16x16x1-nt256-g1-w1-lim03", "32x8x1-nt256-g2-w1-lim03"],
    (3, A.HD, A.LIM03, 0): ["8x8x4-nt256-g1-w2-runs-lim03-core", "8x8x4-nt256-g1-w2-runs-lim03",
                            "8x8x4-nt256-g1-w1-lim03", "8x8x8-nt512-g2-w1-lim03"],
    (3, A.MHD, A.LIM03, 0): ["8x8x4-nt256-g1-w2-runs-lim03-core", "8x8x8-nt512-g1-w2-runs-lim03-core",
                             "8x8x4-nt256-g2-w4-runs-lim03", "8x8x4-nt256-g2-w3-runs-lim03",
                             "8x8x8-nt512-g2-w4-runs-lim03", "8x8x4-nt256-g2-w3-lim03"],
    (1, A.GLM, A.MP5, 0): [RUNS1 + "-rec0"],
    (2, A.GLM, A.MP5, 0): ["16x16x1-nt256-g2-w2-runs-rec0", "16x16x1-nt256-g1-w1-runs-rec0",
                           "16x16x1-nt256-g1-w2-runs-rec0-core"],
    (3, A.GLM, A.MP5, 0): ["8x8x4-nt256-g1-w2-runs-rec0-core", "8x8x8-nt512-g1-w2-runs-rec0-core",
                           "8x8x4-nt256-g3-w3-runs-rec0-core", "8x8x4-nt256-g2-w3-runs-rec0",
                           "8x8x4-nt256-g3-w4-runs-rec0"],
    (1, A.GLM, A.LIM03, 0): [RUNS1 + "-rec1"],
    (2, A.GLM, A.LIM03, 0): ["16x16x1-nt256-g2-w2-runs-rec1"],
    (3, A.GLM, A.LIM03, 0): ["8x8x4-nt256-g1-w2-runs-rec1-core", "8x8x4-nt256-g2-w4-runs-rec1",
                             "8x8x4-nt256-g2-w3-runs-rec1"],
    (1, A.MHD, A.MP5, 0.1): [RUNS1 + "-rec0"],
    (2, A.MHD, A.MP5, 0.1): ["16x16x1-nt256-g2-w2-runs-rec0"],
    (3, A.MHD, A.MP5, 0.1): ["8x8x4-nt256-g1-w2-runs-rec0-core", "8x8x4-nt256-g2-w4-runs-rec0",
                             "8x8x4-nt256-g2-w2-runs-rec0"],
    (1, A.MHD, A.LIM03, 0.1): [RUNS1 + "-rec1"],
    (2, A.MHD, A.LIM03, 0.1): ["16x16x1-nt256-g2-w2-runs-rec1"],
    (3, A.MHD, A.LIM03, 0.1): ["8x8x4-nt256-g1-w2-runs-rec1-core", "8x8x4-nt256-g2-w4-runs-rec1"],
}


@pytest.mark.parametrize("ndim,physics,recon,eta_h", list(SHAPES))
def test_positions_and_names_of_the_general_shapes(ndim, physics, recon, eta_h):
    code = "glm" if physics == A.GLM else "hall" if eta_h > 0 else "true" if physics == A.MHD else "false"
    want = [f"{ndim}d-{code}-tile{s}" for s in SHAPES[ndim, physics, recon, eta_h]]
    ctx = A.Context(ndim, physics, 5 / 3, recon=recon, eta_h=eta_h)
    assert ctx.variants()[:len(want)] == want
    for i, name in enumerate(want):
        ctx.set_variant(i)
        assert ctx.current_variant() == name
    ctx.close()


def test_a_saved_choice_is_reused(tmp_path, monkeypatch):
    path = tmp_path / "tune.txt"
    monkeypatch.setenv("AMRVAC_TUNE_CACHE", str(path))
    bs = helpers.strip_blocks(3, True, [8, 8], 8, 8, seed=5)
    ctx, flat, views = A.context_for(bs)
    name, ms = ctx.autotune(A.RK3, 1)
    assert all(m > 0 for m in ms)
    saved = "3d-true-tile8x4x4-nt128-g1-w2-runs-core"
    text = path.read_text()
    path.write_text(text.replace(name, saved))
    name, ms = ctx.autotune(A.RK3, 1)
    assert name == saved and all(m < 0 for m in ms)
    ctx.close()


@pytest.mark.parametrize("ndim,physics,recon,shape", [
    (1, A.HD, A.MP5, "1d-false-tile" + CORE1), (1, A.HD, A.LIM03, "1d-false-tile64x1x1-nt64-g1-w1-lim03"),
    (1, A.MHD, A.MP5, "1d-true-tile128x1x1-nt128-g1-w1"), (1, A.MHD, A.LIM03, "1d-true-tile" + RUNS1 + "-lim03-core"),
    (2, A.GLM, A.MP5, "2d-glm-tile16x16x1-nt256-g1-w2-runs-rec0-core"),
    (3, A.GLM, A.MP5, "3d-glm-tile8x8x4-nt256-g1-w2-runs-rec0-core"),
    (2, A.HD, A.MP5, "2d-false-roles16x8x1-nt256-w4"), (3, A.MHD, A.LIM03, "3d-true-roles8x8x4-nt512-w4-lim03")])
def test_default_shape(ndim, physics, recon, shape):
    bs = helpers.strip_blocks(ndim, physics != A.HD, [700, 600] if ndim == 1 else [8, 8], 8, 8, seed=5)
    if physics == A.GLM:
        bs = inputs.as_glm(bs)
    ctx, flat, views = A.context_for(bs, recon=recon)
    assert ctx.current_variant() == shape
    ctx.set_exec(A.EXEC_PER_BLOCK)
    first = ndim == 1 and physics == A.HD and recon == A.LIM03   # faster there
    assert ctx.current_variant() == ("1d-false-tile128x1x1-nt128-g1-w1-lim03" if first else shape)
    ctx.set_exec(A.EXEC_BATCHED)
    assert ctx.current_variant() == shape
    ctx.close()
