"""Small plans' tile lists (binned, each list sorted by itself) against a sort of the
same keys on the host: lists around the sizes where the sort changes its form (a
wave, one to eight keys a thread, runs merged through memory), boxes listed row by
row, several views to a block of records, equal depths, and a plan that is too crowded
for the bins beside one that is not."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from gpu_common import GpuScene, log  # noqa: E402
from paper_2601_22026_amd import _abi  # noqa: E402


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2601_22026_amd as gs
    return gs.Context(0)


def _check(sc, tile):
    """The lists are every tile's records by (depth, record); each record is listed
    count times in all, and in the tiles of its box alone."""
    sizes = [(c.width, c.height) for c in sc.cams]
    tiles = [((w + tile - 1) // tile, (h + tile - 1) // tile) for w, h in sizes]
    T, R = sum(x * y for x, y in tiles), sc.n * len(sc.cams)
    count = sc.debug(_abi.GSF_DBG_COUNT, np.uint32, R).astype(np.int64)
    M = int(count.sum())
    depth = sc.debug(_abi.GSF_DBG_DEPTH, np.uint32, R).astype(np.int64)
    rect = sc.debug(_abi.GSF_DBG_RECT, np.uint32, 2 * R).reshape(R, 2).astype(np.int64)
    keys = sc.debug(_abi.GSF_DBG_KEYS, np.uint32, M).astype(np.int64)
    vals = sc.debug(_abi.GSF_DBG_VALS, np.uint32, M).astype(np.int64)
    ranges = sc.debug(_abi.GSF_DBG_RANGES, np.uint32, 2 * T).reshape(T, 2).astype(np.int64)
    order = sc.debug(_abi.GSF_DBG_ORDER, np.uint32, T).astype(np.int64)
    np.testing.assert_array_equal(np.lexsort((vals, depth[vals], keys)), np.arange(M))
    np.testing.assert_array_equal(np.bincount(vals, minlength=R), count)
    pair = keys * R + vals
    assert np.unique(pair).size == M
    v = vals // sc.n
    off = np.concatenate([[0], np.cumsum([x * y for x, y in tiles])])
    tx = np.array([x for x, _ in tiles])[v]
    local = keys - off[v]
    x, y = local % tx, local // tx
    assert (x >= rect[vals, 0] & 0xFFFF).all() and (x <= rect[vals, 1] & 0xFFFF).all()
    assert (y >= rect[vals, 0] >> 16).all() and (y <= rect[vals, 1] >> 16).all()
    np.testing.assert_array_equal(ranges[:, 1] - ranges[:, 0], np.bincount(keys, minlength=T))
    assert (np.diff(ranges[:, 0]) >= 0).all()
    np.testing.assert_array_equal(np.sort(order), np.arange(T))
    length = ranges[order, 1] - ranges[order, 0]
    cls = np.floor(np.log2(np.maximum(length, 0.5))).astype(int)
    assert (np.diff(cls) <= 0).all()
    return int((ranges[:, 1] - ranges[:, 0]).max())


def _crowd(n, seed):
    """n Gaussians within a tile or two, half of them at
    depths that others have too."""
    P = synth.random_gaussians(n, seed=seed)
    rng = np.random.default_rng(seed)
    P[0:3] = rng.uniform(-0.02, 0.02, (3, n)) + 0.05
    P[2, : n // 2] = P[2, rng.integers(0, min(8, n), n // 2)]
    P[3:6] = -6.0
    return P


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 128, 129, 1023, 1024, 1025, 2048, 2049, 4097, 8192, 8193, 16385,
                               40000])
def test_list_lengths(ctx, n):
    sc = GpuScene(ctx, _crowd(n, n), [synth.axis_camera(256, 384)])
    sc.forward()
    longest = _check(sc, 16)
    log(f"[bins] {n} Gaussians, longest list {longest}")


@pytest.mark.parametrize("n,every", [(2304, 2), (4096, 4), (6144, 6), (8192, 8)])
def test_sample_that_misleads(ctx, n, every):
    """One tile whose every second (fourth, ...) record, those a sample taken at equal
    steps finds, lies in front of all others: one bucket holds most of the list."""
    P = _crowd(n, n)
    P[0:2] = P[0:2] * 0.01 + 0.05
    P[2] += np.where(np.arange(n) % every == 0, -0.5, 0.5)
    sc = GpuScene(ctx, P, [synth.axis_camera(256, 384)])
    sc.forward()
    log(f"[bins] {n} Gaussians, every {every}th in front, longest list {_check(sc, 16)}")


@pytest.mark.parametrize("tile", [8, 16, 32])
def test_views_and_boxes(ctx, tile):
    P = synth.with_near_splats(synth.random_gaussians(300, seed=12), 8, seed=12)
    cams = [synth.axis_camera(512, 512), synth.look_at_camera([1.2, -0.8, -2.6], width=77, height=53),
            synth.look_at_camera([0.0, 3.0, 0.2], width=40, height=300)]
    sc = GpuScene(ctx, P, cams, tile=tile)
    sc.forward()
    _check(sc, tile)


# more tiles than the counters of a workgroup, more records than a tile should hold
@pytest.mark.parametrize("n,size,tile", [(500, (1040, 512), 8), (500, (1024, 512), 8), (4097, (32, 64), 32)])
def test_either_side_of_the_rule(ctx, n, size, tile):
    sc = GpuScene(ctx, synth.random_gaussians(n, seed=n), [synth.axis_camera(*size)], tile=tile)
    sc.forward()
    _check(sc, tile)


def test_overflow_lists_nothing(ctx):
    sc = GpuScene(ctx, _crowd(500, 1), [synth.axis_camera(256, 384)], host_sized=False, key_capacity=100)
    sc.forward()
    ranges = sc.debug(_abi.GSF_DBG_RANGES, np.uint32, 2 * 16 * 24)
    assert not ranges.any()
    assert (sc.images()[0][3] == 0).all()
