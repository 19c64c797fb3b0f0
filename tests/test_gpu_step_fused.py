"""The fit step's loss, finished by a workgroup of the adjoint, and its Adam update, done
by the kernel that finishes the gradient, against the calls of their own on the same
image and gradient: the same bits (the order of the loss's sum does not depend on the
workgroup, and both updates are the same operations)."""
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


@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("deg", [0, 1, 2])
@pytest.mark.parametrize("n", [1, 63, 128, 129, 1000])
def test_step_update_is_the_adam_call(ctx, n, deg, masked):
    """Gaussian counts about the wave and the workgroup, one and two views, three steps
    (moments other than zero), a learning rate per plane."""
    import paper_2601_22026_amd as gs
    for sizes in ([(64, 48)], [(64, 48), (40, 56)]):
        log(f"[step adam] n {n} deg {deg} masked {masked} {sizes}")
        st = _step(gs, ctx, n, sizes, deg=deg, masked_adam=masked, lr_boost=1.5)
        lr = gs.plane_learning_rates(deg, 1e-2, 1.5)
        for k in range(3):
            p, m, v = st.params.clone(), st.m.clone(), st.v.clone()
            done = st.step_dev.clone()
            st.step()
            if masked:
                gs.adam_masked(ctx, p, st.grads, m, v, done, lr,
                               torch.from_numpy(st.visibility()).to(DEV))
            else:
                off, rate = [0], [lr[0]]
                for c in range(1, st.C):
                    if lr[c] != rate[-1]:
                        off.append(c * n)
                        rate.append(lr[c])
                gs.adam(ctx, p.view(-1), st.grads.view(-1), m.view(-1), v.view(-1), done, off + [st.C * n], rate)
            torch.cuda.synchronize()
            assert done.item() == st.steps_done() == k + 1
            for a, b in ((p, st.params), (m, st.m), (v, st.v)):
                assert torch.equal(a.view(torch.int32), b.view(torch.int32))


@pytest.mark.parametrize("masked", [False, True])
def test_step_after_overflow_updates_nothing(ctx, masked):
    import paper_2601_22026_amd as gs
    st = _step(gs, ctx, 500, [(64, 48)], masked_adam=masked, key_capacity=64)
    p = st.params.clone()
    st.step()
    torch.cuda.synchronize()
    assert torch.equal(p, st.params) and st.steps_done() == 0
    assert not st.m.any() and not st.v.any()
    assert st.ensure_capacity()
    st.step()
    torch.cuda.synchronize()
    assert st.steps_done() == 1 and not torch.equal(p, st.params)
