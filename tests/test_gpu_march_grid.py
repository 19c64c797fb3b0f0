"""The ray march with and without its grid of occupied cells: the same bits.  A
captured march has no grid (the graph could run beside a later call that fills it)
and reads every segment, so it is the oracle here; the march itself is held
against the FP64 definition elsewhere."""
import ctypes as ct

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from gpu_common import DEV, log  # noqa: E402


def _cams():
    return [synth.look_at_camera([0.5, -0.8, -2.8], width=65, height=33, bg=(0.2, 0.1, 0.3)),
            synth.look_at_camera([0.0, 0.0, -3.0], width=16, height=9),      # along an axis
            synth.look_at_camera([0.3, 0.2, -0.4], width=7, height=1),       # from inside
            synth.look_at_camera([2.0, 2.0, 2.0], width=40, height=48)]      # along the diagonal


def _march(gs, ctx, vol, cams_dev, cams, out, threshold, extinction, step):
    w = (ct.c_int32 * len(cams))(*[c.width for c in cams])
    h = (ct.c_int32 * len(cams))(*[c.height for c in cams])
    ctx.use_stream()
    ctx.check(gs.lib().gsf_raymarch(ctx.handle, vol.data_ptr(), vol.shape[0], cams_dev.data_ptr(), len(cams), w, h,
                                    step, extinction, 1e-4, threshold, 1800.0, (ct.c_float * 3)(0.8, 0.3, 0.2),
                                    (ct.c_float * 3)(1.0, 0.95, 0.9), out.data_ptr()), "gsf_raymarch")


# one cell a voxel, up to the largest such volume; two and three voxels a cell, with
# the last cell full and ragged
@pytest.mark.parametrize("n", [1, 2, 3, 5, 127, 128, 129, 255, 257])
@pytest.mark.parametrize("threshold,extinction,steps", [(1200.0, 40.0, 1.0), (0.0, 2.0, 0.37), (-5.0, 2.0, 1.0),
                                                        (float("nan"), 2.0, 1.0), (1200.0, float("inf"), 1.0)])
def test_grid_changes_no_bit(n, threshold, extinction, steps):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2601_22026_amd as gs
    rng = np.random.default_rng(n)
    vol = np.zeros((n, n, n), np.uint16)
    k = max(1, n ** 3 // 5000)
    vol.reshape(-1)[rng.integers(0, n ** 3, k)] = rng.integers(1100, 3000, k)      # scattered voxels
    vol[n // 3:n // 3 + max(1, n // 6), :n // 2, n // 2:] = 1500                     # a slab, out to two faces
    vol_d = torch.from_numpy(vol.view(np.int16)).to(DEV)
    empty = torch.zeros_like(vol_d)
    cams = _cams()
    ctx = gs.Context(0)
    cams_dev = gs.cameras_to_device(cams, DEV)
    total = 4 * sum(c.width * c.height for c in cams)
    got, again, want = (torch.full((total,), v, device=DEV) for v in (-1.0, -2.0, -3.0))
    args = (threshold, extinction, steps / n)
    other = torch.cuda.Stream()
    other.wait_stream(torch.cuda.current_stream())
    _march(gs, ctx, vol_d, cams_dev, cams, got, *args)
    with torch.cuda.stream(other):                                   # an empty grid, then the first again
        _march(gs, ctx, empty, cams_dev, cams, again, *args)
        _march(gs, ctx, vol_d, cams_dev, cams, again, *args)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        _march(gs, ctx, vol_d, cams_dev, cams, want, *args)
    graph.replay()
    torch.cuda.synchronize()
    assert torch.equal(got.view(torch.int32), again.view(torch.int32))
    same = got.view(torch.int32) == want.view(torch.int32)
    log(f"[march grid] n {n} threshold {threshold} extinction {extinction}: {int((~same).sum())} of {total} differ")
    assert bool(same.all())
