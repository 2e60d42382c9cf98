"""Device setup of the shared-offset SELL layout: which matrices it takes and
what it stores, against the definition restated on the host."""

import numpy as np
import pytest

import oracle
import spkgen
from gpu_util import mat_on_gpu, need_gpu, to_dev
from test_gpu_spmv import _shared_layout

pytestmark = pytest.mark.gpu


def _band(n, k, drop=()):
    """Rows i holding columns i .. i + k - 1 (clipped to n); rows in drop keep none."""
    rows = [list(range(i, min(n, i + k))) if i not in drop else [] for i in range(n)]
    rowptr = np.zeros(n + 1, np.int32)
    rowptr[1:] = np.cumsum([len(r) for r in rows])
    col = np.array([c for r in rows for c in r], np.int32)
    return spkgen.CSR(n, rowptr, col, np.random.default_rng(n + k).integers(-9, 10, col.size).astype(np.float64))


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 200, 4 * 64 * 2048 + 3])
@pytest.mark.parametrize("k", [1, 5, 31, 32])
def test_shared_lists_sizes(n, k):
    """Slice remainders, the widest list, more slices than the grid has
    wavefronts: products are exact on integers, the counts as defined."""
    if n > 4096 and k != 5:
        pytest.skip("one width is enough at this size")
    spk = need_gpu()
    if n > 4096:
        A = spkgen.laplace_grid((n,))
    else:
        A = _band(n, k, drop={3, 64})
    M = mat_on_gpu(spk, A)
    spk.mat_set_kernel(M, spk.KERNEL_SELL, spk.SELL_SHARED)
    widths, nlist = _shared_layout(A)
    assert M.info.lanes == 0 and M.info.stored_nnz == 64 * sum(widths)
    x = np.random.default_rng(1).integers(-9, 10, A.n).astype(np.float64)
    y = to_dev(np.full(A.n, np.nan))
    spk.mat_mult(M, to_dev(x), y)
    assert np.array_equal(y.cpu().numpy(), oracle.spmv(A, x))
    M.close()


@pytest.mark.parametrize("where", [0, 70, 199])
@pytest.mark.parametrize("what", ["repeated", "descending", "33_offsets"])
def test_shared_lists_refused(where, what):
    """One row out of order, one repeated column, one slice of 33 offsets."""
    spk = need_gpu()
    A = _band(200, 3)
    col = A.col.copy()
    if what == "33_offsets":
        A = spkgen.CSR(200, np.arange(201, dtype=np.int32), np.arange(200, dtype=np.int32), np.ones(200))
        s0 = min(where // 64 * 64, 200 - 40)
        col = A.col.copy()
        col[s0:s0 + 40] = s0 + 39 - np.arange(40)  # 40 offsets in the slice, or 33 and more in one of two
        if _shared_layout(spkgen.CSR(200, A.rowptr, col, A.val)) is not None:
            pytest.skip("the offsets fell into two slices")
    else:
        a = A.rowptr[where]
        if A.rowptr[where + 1] - a < 2:
            a = A.rowptr[where - 1]
        col[a:a + 2] = col[a] if what == "repeated" else col[a:a + 2][::-1]
    B = spkgen.CSR(A.n, A.rowptr, col, A.val)
    M = mat_on_gpu(spk, B)
    with pytest.raises(spk.SpkError) as e:
        spk.mat_set_kernel(M, spk.KERNEL_SELL, spk.SELL_SHARED)
    assert e.value.status == spk.EINVAL
    spk.mat_set_kernel(M, spk.KERNEL_SELL, 0)
    assert M.info.lanes == 16
    x = np.random.default_rng(1).integers(-9, 10, B.n).astype(np.float64)
    y = to_dev(np.full(B.n, np.nan))
    spk.mat_mult(M, to_dev(x), y)
    assert np.array_equal(y.cpu().numpy(), oracle.spmv(B, x))
    M.close()
