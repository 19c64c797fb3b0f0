"""The fit step's loss, finished by a workgroup of the adjoint, against the loss call of
its own on the same image: the same bits (the order of the sum does not depend on the
workgroup)."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2601_22026_amd as gs
    return gs.Context(0)


from gpu_common import DEV, log  # noqa: E402


def _step(gs, ctx, n, sizes, deg=0, **cfg):
    P = torch.from_numpy(synth.random_gaussians(n, seed=5, sh_degree=deg)).to(DEV)
    cams = [synth.look_at_camera([0.3 * k, 0.2, -3.0], width=w, height=h, bg=(0.2, 0.4, 0.1))
            for k, (w, h) in enumerate(sizes)]
    planes = 4 if cfg.get("alpha_loss") else 3
    tgt = torch.rand(planes * sum(w * h for w, h in sizes), device=DEV,
                     generator=torch.Generator(device=DEV).manual_seed(7))
    return gs.FitStep(ctx, P, cams, tgt, cfg=gs.FitConfig(lr=1e-2, **cfg))


@pytest.mark.parametrize("t_mode", [0, 1, 2])
@pytest.mark.parametrize("tile", [8, 16, 32])
@pytest.mark.parametrize("sizes", [[(8, 8)], [(43, 37)], [(199, 101), (64, 64)], [(1056, 1024), (1024, 1056)]])
def test_step_loss_is_the_loss_call(ctx, sizes, tile, t_mode):
    """From one partial sum to more than a workgroup reads at once, with every number
    of waves a workgroup of the adjoint has (few tiles and many)."""
    import paper_2601_22026_amd as gs
    log(f"[step loss] {sizes} tile {tile} t_mode {t_mode}")
    st = _step(gs, ctx, 300, sizes, tile=tile, t_mode=t_mode, lds_batch=64)
    loss, dl = torch.zeros(1, device=DEV), torch.zeros_like(st.dl)
    for k in range(2):
        st.step()
        st.plan.loss_l1(st.rgba, st.targets, loss, dl)
        torch.cuda.synchronize()
        assert st.steps_done() == k + 1
        assert np.float32(loss.item()).tobytes() == np.float32(st.loss.item()).tobytes()
        assert torch.equal(dl, st.dl)
