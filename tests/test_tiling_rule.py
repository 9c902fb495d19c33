"""The automatic tiling as a function of the problem and the device's compute units,
checkpoints included: host-side, for devices that need not be there."""
import ctypes
import os

import numpy as np
import pytest

from paper_2109_05496_amd import _lib

pytestmark = pytest.mark.skipif(not os.path.exists(_lib.LIB_PATH), reason="libctv.so not built")


def choice(m, n, iters, batch=1, ckpt=0, cus=256, **kw):
    p = _lib.make_params("1i", iters=iters, **kw)
    out = [ctypes.c_int32() for _ in range(3)]
    _lib.call("ctv_tune_cache_clear")
    _lib.call("ctv_debug_tiling", ctypes.byref(p), batch, m, n, ckpt, cus, *(ctypes.byref(o) for o in out))
    return tuple(o.value for o in out)


def tiles(m, n, batch, T):
    return -(-m // (64 - 2 * T)) * -(-n // (64 - 2 * T)) * min(batch, 32)


@pytest.mark.parametrize("m,n,batch", [(2048, 2048, 1), (8192, 8192, 1), (1500, 1345, 1), (769, 769, 4), (512, 512, 16)])
def test_more_tiles_than_compute_units(m, n, batch):
    """Above three tiles per CU the 64 x 64 region runs as 16 waves x 4 rows, T = 8;
    9 to 11 iterations between checkpoints in one launch, others in even parts."""
    assert tiles(m, n, batch, 8) > 3 * 256
    assert choice(m, n, 200, batch) == (8, 16, 4)
    for ckpt in range(5, 15):
        T, waves, rows = choice(m, n, 50, batch, ckpt=ckpt)
        assert (waves, rows) == (16, 4)
        assert T == (ckpt if 9 <= ckpt <= 11 else 8), ckpt
    for iters in (5, 9, 11):  # no checkpoint inside the run: nothing to cross
        assert choice(m, n, iters, batch, ckpt=11) == (min(8, iters), 16, 4)
    assert choice(m, n, 200, batch, fuse=6) == (6, 8, 8)
    assert choice(m, n, 200, batch, tile=(8, 4)) == (8, 8, 4)


def test_a_part_of_the_device():
    """The rule follows the compute units that there are."""
    rng = np.random.default_rng(1)
    for cus in (32, 64, 128, 256):
        for _ in range(60):
            m, n = (int(v) for v in np.exp(rng.uniform(0, np.log(3000), 2)))
            T, waves, rows = choice(m, n, 40, cus=cus)
            region = -(-m // (waves * rows - 2 * T)) * -(-n // (64 - 2 * T))
            if (waves * rows, T) != (64, 8):
                assert region <= 2 * cus, (m, n, cus)
            elif region > 3 * cus:
                assert (waves, rows) == (16, 4), (m, n, cus)


@pytest.mark.parametrize("m,n", [(64, 64), (100, 100), (500, 500), (700, 700)])
def test_as_many_iterations_as_an_int_holds(m, n):
    assert choice(m, n, 2 ** 31 - 1) == choice(m, n, 2 ** 30)
    assert choice(m, n, 2 ** 31 - 5, ckpt=2 ** 31 - 1) == choice(m, n, 2 ** 30)
