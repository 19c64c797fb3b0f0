"""The seeding's choice of the cap smallest priorities, against the generator's
definition (bit-exact): remainders of tiles and lanes, caps around the number of
candidates, thresholds at the ends of the values, a volume that is not 16-byte
aligned, and priorities that crowd more than the list of undecided keys holds."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from gpu_common import DEV, log  # noqa: E402

UNDECIDED = 4096   # the list's room


def _check(vol, cap, seed, threshold, offset=0):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2601_22026_amd as gs
    n = vol.shape[0]
    buf = torch.zeros(vol.size + offset, dtype=torch.int16, device=DEV)
    v = buf[offset:].view(n, n, n)
    v.copy_(torch.from_numpy(vol.view(np.int16)))
    ref = synth.seed_from_volume(vol, threshold=threshold, cap=cap, seed=seed)
    got = gs.seed_volume(gs.Context(0), v, cap=cap, seed=seed, threshold=threshold).cpu().numpy()
    assert got.shape == ref.shape
    log(f"[select] n {n} cap {cap}: kept {got.shape[1]}")
    # the colour's transfer function has a fixed threshold there
    rows = slice(0, 11) if threshold != synth.TF_THRESHOLD else slice(0, 14)
    np.testing.assert_array_equal(got[rows].view(np.uint32), ref[rows].view(np.uint32))


@pytest.mark.parametrize("n,fill", [(1, 1.0), (2, 0.5), (3, 0.5), (13, 0.3), (13, 1.0), (40, 0.01), (65, 0.9)])
@pytest.mark.parametrize("cap", ["one", "less", "all", "more"])
@pytest.mark.parametrize("threshold,offset", [(1200.0, 0), (1200.0, 1), (1200.5, 0), (-0.5, 0), (65534.0, 3)])
def test_selection_matches_generator(n, fill, cap, threshold, offset):
    rng = np.random.default_rng(n)
    vol = rng.choice(np.array([1200, 1201, 2000, 40000, 65534, 65535], np.uint16), (n, n, n))
    vol[rng.random((n, n, n)) > fill] = 0
    total = int((vol > threshold).sum())
    _check(vol, dict(one=1, less=max(1, total - 1), all=max(1, total), more=total + 1)[cap], 7, threshold, offset)


# nearly the most voxels that one histogram is enough for, all of them candidates: the
# digit of the cap-th priority is shared by more of them than the list holds
def test_crowded_priorities_take_another_digit():
    n, bits = 161, 10
    vol = np.full((n, n, n), 3000, np.uint16)
    assert n ** 3 >> bits <= UNDECIDED
    pri = synth.cap_priority(np.arange(n ** 3), 5, n ** 3)
    count = np.bincount((pri >> np.uint64(64 - bits)).astype(np.int64), minlength=1 << bits)
    d = int(np.argmax(count))
    assert count[d] > UNDECIDED
    _check(vol, int(count[:d].sum() + count[d] // 2), 5, synth.TF_THRESHOLD)


# two histograms enqueued: the second needed, and not
@pytest.mark.parametrize("every", [1, 50])
def test_two_histograms(every):
    n = 170
    assert n ** 3 >> 10 > UNDECIDED
    vol = np.zeros((n, n, n), np.uint16)
    vol[:, ::every] = 3000
    _check(vol, 20_001, 11, synth.TF_THRESHOLD)
