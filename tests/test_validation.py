"""The host's check of a graph's rows, at the edges of its 64 x 64 blocks: it
runs before any device call, so a bad graph is MCE_E_INVAL without a GPU too."""
import ctypes

import numpy as np
import pytest

import synth


def _prepare(mce, rows):
    h = ctypes.c_void_p()
    n, rw = rows.shape
    rc = mce._lib().mce_prepare(n, rows.ctypes.data, rw, None, 0, None, ctypes.byref(h))
    if rc == mce.OK:
        mce._lib().mce_release(h)
    return rc


# blocks of few bits (compared bit by bit) and of many (transposed), one block
# and several, full and partly filled
@pytest.mark.parametrize("p", [0.003, 0.02, 0.5, 1.0])
@pytest.mark.parametrize("n", [2, 63, 64, 65, 128, 130, 191])
@pytest.mark.parametrize("pad", [0, 1])
def test_bad_rows_refused(n, p, pad):
    from paper_1801_00202_amd import mce
    good = np.zeros((n, (n + 63) // 64 + pad), dtype=np.uint64)
    rows = synth.complete(n) if p == 1.0 else synth.gnp(n, p, 5)
    good[:, :rows.shape[1]] = rows
    assert _prepare(mce, good) in (mce.OK, mce.E_DEVICE)
    one = np.uint64(1)
    for i in sorted({0, n // 2, n - 1}):
        for j in sorted({0, 1, 31, 32, 62, 63, 64, 65, 127, 128, n - 1, n, 64 * good.shape[1] - 1}):
            if j >= 64 * good.shape[1]:
                continue
            # one bit flipped: an edge one way, a loop, a bit past the last column
            bad = good.copy()
            bad[i, j // 64] ^= one << np.uint64(j % 64)
            assert _prepare(mce, bad) == mce.E_INVAL, (i, j)
            if j < n and i != j:
                # both ways: a simple graph again
                bad[j, i // 64] ^= one << np.uint64(i % 64)
                assert _prepare(mce, bad) in (mce.OK, mce.E_DEVICE), (i, j)
    # as many bits in a block and its mirror image, in other places
    if n > 66:
        bad = good.copy()
        for i, j in ((0, 65), (66, 1)):
            bad[i, j // 64] ^= one << np.uint64(j % 64)
        assert _prepare(mce, bad) == mce.E_INVAL
