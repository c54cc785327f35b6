"""Centre-finder entry points on the CPU: exports and host validation (no
device work)."""
import ctypes as C

import numpy as np

from paper_1411_3396_amd import _sr

FAKE = C.c_void_p(0x10000)  # never dereferenced: every case fails validation first


def _create(offsets, H=None):
    off = np.ascontiguousarray(np.asarray(offsets, np.int64))
    plan = C.c_void_p()
    nbytes = C.c_size_t()
    code = _sr.lib().sr_centres_plan_create(len(off) - 1 if H is None else H, off.ctypes.data_as(C.c_void_p),
                                            C.byref(plan), C.byref(nbytes))
    return code, plan, nbytes.value


def test_plan_validation():
    assert _create([0, 3])[0] == 0
    assert _create([1, 3])[0] == 1  # must start at 0
    assert _create([0, 5, 3])[0] == 1  # decreasing
    assert _create([0], H=0)[0] == 1  # no halos
    assert _create([0, 1 << 31])[0] == 5  # more particles than 32-bit indices
    code, plan, nbytes = _create([0, 0, 1, 65, 65, 1000])
    assert code == 0 and nbytes % 256 == 0 and nbytes > 0
    assert _sr.lib().sr_centres_plan_destroy(plan) == 0


def test_run_validation_before_device():
    code, plan, nbytes = _create([0, 10, 300])
    L = _sr.lib()
    run = lambda eps, ws=FAKE, wsb=nbytes, phi=FAKE, mbp=FAKE: L.sr_centres(  # noqa: E731
        plan, FAKE, FAKE, eps, ws, wsb, phi, mbp, None, None)
    assert run(-1.0) == 1
    assert run(float("nan")) == 1
    assert run(0.02, mbp=None) == 1
    assert run(0.02, phi=None) == 1
    assert run(0.02, wsb=nbytes - 1) == 2
    assert run(0.02, ws=C.c_void_p(0x10004)) == 2  # misaligned
    assert L.sr_centres(None, FAKE, FAKE, 0.02, FAKE, nbytes, FAKE, FAKE, None, None) == 4
    assert L.sr_centres_plan_destroy(plan) == 0


def test_workspace_grows_with_items():
    a = _create([0, 100])[2]
    b = _create(np.arange(0, 100001, 100))[2]
    assert 0 < a < b


def test_item_slots_fit_their_bits():
    # 2^26 halos, all but one of a single particle: the last one's chunks come on top, and an
    # item's slot among the partial minima no longer fits 26 bits
    off = np.arange((1 << 26) + 1, dtype=np.int64)
    off[-1] += 299
    code, plan, _ = _create(off)
    if code == 0:
        _sr.lib().sr_centres_plan_destroy(plan)
    assert code == 5


def _need(sizes):
    code, plan, nbytes = _create(np.concatenate([[0], np.cumsum(sizes)]))
    assert code == 0
    _sr.lib().sr_centres_plan_destroy(plan)
    return nbytes


def test_pair_once_of_small_catalogues():
    # a few small halos do not pay for the pair-once launches (no slots), many or larger ones do
    slots = lambda k, n: k * 8 * n * ((n + 255) // 256 + 1)  # noqa: E731
    for k, n, once in ((1, 300, 0), (100, 400, 0), (100, 500, 0), (1, 600, 0), (1, 800, 1), (500, 300, 1), (100, 700, 1),
                       (2000, 300, 1)):
        assert (_need([n] * k) >= slots(k, n)) == bool(once), (k, n)
    assert _need([100] * 300 + [700] * 3) < 40000 < slots(3, 700)
    assert _need([100] * 300 + [2000]) >= slots(1, 2000)


def test_pair_once_beside_a_halo_too_large_for_it():
    # a halo whose rows alone exceed 1 GiB of slots is summed from both ends and leaves waves
    # idle; a few others fill them from both ends too (no slots), many go pair-once
    assert _need([737460]) > 1000 << 20 and _need([737461]) < 1 << 20
    assert _need([4000] * 50) > 50 * 8 * 4000 * 17
    assert _need([968359] + [4000] * 50) < 1 << 20
    assert _need([968359] + [270000] * 7 + [100000] * 35) > 7 * 8 * 270000 * 67
