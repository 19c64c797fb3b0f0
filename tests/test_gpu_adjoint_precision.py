"""The adjoint by blocks, whose sums are moved from a block's centre to the splat's mean,
against the adjoint by tiles, whose sums are about the mean: narrow splats, which lie off
the centre, must not lose precision."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2601_22026_amd as gs
    return gs.Context(0)


from gpu_common import GpuScene, log  # noqa: E402


@pytest.mark.parametrize("t_mode", [0, 1])
@pytest.mark.parametrize("seed", [1, 2, 3])
def test_blocks_are_as_exact_as_tiles(ctx, seed, t_mode):
    """Both forms sum the same FP32 terms, so their errors in the gradient's norm are
    alike: at most half as much again, above the 5e-7 that the terms' own rounding
    leaves.  (The second plan is beside a view of a megapixel that sees nothing, which
    makes it one of many tiles.)"""
    P = synth.random_gaussians(1500, seed=seed, logscale_mean=-4.5, logscale_std=0.6, mean_range=0.9)
    cam = synth.look_at_camera([0.1, 0.2, -3.0], width=131, height=99)
    away = synth.look_at_camera([0.0, 0.0, -3.0], target=(0.0, 0.0, -6.0), width=1056, height=1024)
    ref = oracle.render(P, cam)
    dl = np.random.default_rng(seed).normal(size=(4, cam.npix))
    dl[:, ref.flags != 0] = 0.0
    dl = dl.astype(np.float32)
    G = oracle.backward(P, cam, dl.astype(np.float64))
    err = []
    for cams in ([cam], [cam, away]):
        sc = GpuScene(ctx, P, cams, tile=16, batch=64, t_mode=t_mode)
        sc.forward()
        g = sc.backward([dl] + [np.zeros((4, c.npix), np.float32) for c in cams[1:]])
        err.append(float(np.linalg.norm(g - G) / np.linalg.norm(G)))
    log(f"[adjoint precision] seed {seed} t_mode {t_mode}: blocks {err[0]:.3e}, tiles {err[1]:.3e}")
    assert err[0] <= max(1.5 * err[1], 5e-7)
