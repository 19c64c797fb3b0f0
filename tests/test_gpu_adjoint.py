"""The two forms of the compositing adjoint (one wave per 8 x 8 block, one wave
per tile or quarter tile) against the FP64 oracle at the sizes where their chunks, groups and
clamp-free path begin and end."""
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


from gpu_common import GpuScene, grads_close, log  # noqa: E402


def _stack(n, logit):
    """n wide splats in front of one another, all reaching the middle of the view."""
    P = synth.random_gaussians(n, seed=21, logscale_mean=-1.2, logscale_std=0.2, mean_range=0.3)
    P[10] = logit
    return P


@pytest.mark.parametrize("t_mode", [0, 1, 2])
@pytest.mark.parametrize("tile", [8, 16, 32])
@pytest.mark.parametrize("n,logit", [(1, -3.0), (3, 4.0), (63, -4.0), (64, -4.0), (65, 6.0),
                                     (130, -5.0), (193, -5.5)])
def test_adjoint_forms_match_oracle(ctx, n, logit, tile, t_mode):
    """List lengths about the 64-record chunk and the group sizes, opacities with
    and without the alpha clamp (0.98 and 0.9975 reach it), a view of odd size;
    alone (a plan of few tiles) and beside a view of a megapixel that sees nothing
    (a plan of many)."""
    P = _stack(n, logit)
    cam = synth.look_at_camera([0.1, 0.2, -3.0], width=43, height=37, bg=(0.2, 0.4, 0.1))
    away = synth.look_at_camera([0.0, 0.0, -3.0], target=(0.0, 0.0, -6.0), width=1056, height=1024)
    ref = oracle.render(P, cam)
    dl = np.random.default_rng(3).normal(size=(4, cam.npix))
    dl[:, ref.flags != 0] = 0.0
    dl = dl.astype(np.float32)
    G = oracle.backward(P, cam, dl.astype(np.float64))
    for cams in ([cam], [cam, away]):
        log(f"[adjoint] n {n} logit {logit} tile {tile} t_mode {t_mode} views {len(cams)}")
        sc = GpuScene(ctx, P, cams, tile=tile, batch=64, t_mode=t_mode)
        sc.forward()
        dls = [dl] + [np.ones((4, c.npix), np.float32) for c in cams[1:]]
        g = sc.backward(dls)
        rep = grads_close(g, G)
        assert all(nb == 0 for _, nb, _ in rep), rep
        again = sc.backward(dls)
        np.testing.assert_array_equal(g.view(np.uint32), again.view(np.uint32))
