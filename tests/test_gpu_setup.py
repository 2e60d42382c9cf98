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


def _outputs(spk, M, n):
    """Products (FP64, FP32, eight columns), smoother and solves of a handle."""
    import torch

    x = to_dev(spkgen.rhs_uniform(n, 2))
    y, y32 = torch.full_like(x, np.nan), torch.full_like(x.float(), np.nan)
    spk.mat_mult(M, x, y)
    spk.mat_mult_f32(M, x.float(), y32)
    X = torch.stack([x, x + 1, 2 * x, x * x, -x, x - 3, x / 3, x * 5], dim=1).contiguous()
    Y = torch.full_like(X, np.nan)
    spk.mat_mult_multi(M, X, Y)
    out = [y, y32, Y]
    if M.info.zero_diag_rows == 0:
        s = torch.full_like(x, np.nan)
        spk.pc_chebyshev(M, x, s, 3, 0.2, 2.0)
        out.append(s)
        for kw in ({}, {"precision": spk.PREC_MIXED}, {"single_reduction": 1}):
            z = torch.zeros_like(x)
            r = spk.ksp_solve(M, x, z, spk.ksp_opts(**kw))
            assert r.reason == spk.CONVERGED_RTOL
            out.append(z)
        Z = torch.zeros_like(X[:, :4]).contiguous()
        spk.ksp_solve_multi(M, X[:, :4].contiguous(), Z)
        out.append(Z)
    return [o.cpu().numpy() for o in out]


@pytest.mark.parametrize("case", ["lap2d_61", "lap3d_23", "box_13", "grid_1d_130", "empty_rows"])
def test_uniform_values_same_bits(case):
    """A matrix of one value per offset stores one list (automatic choice);
    every kernel family of the layout gives the bits of a value per entry."""
    spk = need_gpu()
    A = {"lap2d_61": lambda: spkgen.laplace2d5(61, 0.3), "lap3d_23": lambda: spkgen.laplace3d7(23),
         "box_13": lambda: spkgen.diffusion3d27_lognormal(13, seed=1),
         "grid_1d_130": lambda: spkgen.laplace_grid((130,), 0.5),
         "empty_rows": lambda: _band(200, 5, drop={3, 64, 65, 199})}[case]()
    if case == "box_13":  # 27 points, constant coefficients
        r = np.repeat(np.arange(A.n), np.diff(A.rowptr))
        A = spkgen.CSR(A.n, A.rowptr, A.col, np.where(A.col == r, 27.0, -1.0 + 0.25 * (np.abs(A.col - r) == 1)))
    if case == "empty_rows":
        A = spkgen.CSR(A.n, A.rowptr, A.col, np.repeat(np.arange(A.n), np.diff(A.rowptr)) * 0 + 1.5)
    widths, _ = _shared_layout(A)
    distinct = len(np.unique(A.col - np.repeat(np.arange(A.n), np.diff(A.rowptr))))
    res = []
    for param in (0, spk.SELL_SHARED, 16):
        M = mat_on_gpu(spk, A, flags=spk.MAT_MIXED)
        spk.mat_set_kernel(M, spk.KERNEL_SELL, param)
        assert M.info.stored_nnz == (distinct if param == 0 else 64 * sum(widths)) or param == 16
        res.append(_outputs(spk, M, A.n))
        M.close()
    for other in res[1:]:
        for a, b in zip(res[0], other):
            assert np.array_equal(a, b, equal_nan=True)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("case", ["lap2d_521", "lap3d_67"])
def test_one_diagonal_same_bits(case, precision):
    """Solves too large for one launch: a matrix of one value per offset forms
    z = D^-1 r where it is used, with the bits of a stored D^-1 and z; stopped
    early, started from a guess, and over refinements that keep or restart the
    direction."""
    spk = need_gpu()
    import torch

    A = {"lap2d_521": lambda: spkgen.laplace2d5(521, 0.3), "lap3d_67": lambda: spkgen.laplace3d7(67)}[case]()
    assert A.n > 262144
    b = to_dev(spkgen.rhs_uniform(A.n, 3))
    prec = {"fp64": spk.PREC_FP64, "mixed": spk.PREC_MIXED}[precision]
    res = []
    for param in (0, 16):
        M = mat_on_gpu(spk, A, flags=spk.MAT_MIXED)
        spk.mat_set_kernel(M, spk.KERNEL_SELL, param)
        for kw in ({}, {"maxit": 13}, {"rtol": 1e-12}):
            x = b * 0.125
            r = spk.ksp_solve(M, b, x, spk.ksp_opts(precision=prec, **kw))
            res.append((r.reason, r.iterations, x.cpu().numpy()))
        M.close()
    for a, c in zip(res[:3], res[3:]):
        assert a[:2] == c[:2]
        assert np.array_equal(a[2], c[2])


@pytest.mark.parametrize("entry", ["first", "last", "sign_of_zero"])
def test_uniform_values_need_every_entry(entry):
    """One entry that differs, in its sign bit alone too, keeps a value per entry."""
    spk = need_gpu()
    A = spkgen.laplace2d5(37)
    val = A.val.copy()
    k = {"first": 0, "last": A.nnz - 1, "sign_of_zero": 700}[entry]
    if entry == "sign_of_zero":
        val[A.val < 0] = 0.0
        k = int(np.nonzero(A.val < 0)[0][k])
        val[k] = -0.0
    else:
        val[k] += 2.0 ** -40
    B = spkgen.CSR(A.n, A.rowptr, A.col, val)
    widths, _ = _shared_layout(B)
    M = mat_on_gpu(spk, B)
    assert M.info.lanes == 0 and M.info.stored_nnz == 64 * sum(widths)
    x = spkgen.rhs_uniform(A.n, 2)
    y = to_dev(np.full(A.n, np.nan))
    spk.mat_mult(M, to_dev(x), y)
    yo = oracle.spmv(B, x)
    assert np.all(np.abs(y.cpu().numpy() - yo) <= 8 * 2.0 ** -53 * oracle.spmv_abs(B, x))
    M.close()


@pytest.mark.parametrize("distinct", [27, 28, 65])
def test_uniform_values_offset_limit(distinct):
    """27 distinct offsets in the whole matrix at most, however few each slice has."""
    spk = need_gpu()
    n = 64 * 70
    rng = np.random.default_rng(distinct)
    off = np.concatenate([[0], 1 + rng.choice(80, distinct - 1, replace=False) * 2])
    rows = []
    for i in range(n):  # slice s holds the diagonal and up to 23 of the others
        have = np.unique(np.concatenate([[0], off[(i // 64 * 11 + np.arange(23)) % distinct]]))
        rows.append([i + o for o in have if i + o < n])
    rowptr = np.zeros(n + 1, np.int32)
    rowptr[1:] = np.cumsum([len(r) for r in rows])
    col = np.array([c for r in rows for c in r], np.int32)
    r = np.repeat(np.arange(n), np.diff(rowptr))
    A = spkgen.CSR(n, rowptr, col, np.where(col == r, 40.0, -1.0 - (col - r) / 128))
    M = mat_on_gpu(spk, A)
    widths, _ = _shared_layout(A)
    assert M.info.lanes == 0 and M.info.stored_nnz == (distinct if distinct <= 27 else 64 * sum(widths))
    x = rng.integers(-9, 10, n).astype(np.float64)
    y = to_dev(np.full(n, np.nan))
    spk.mat_mult(M, to_dev(x), y)
    assert np.array_equal(y.cpu().numpy(), oracle.spmv(A, x))
    M.close()


@pytest.mark.parametrize("n", [1, 2, 31, 32, 33, 64, 65, 95, 343, 1000])
def test_coarsest_inverse_blocks(n):
    """The coarsest level alone (one level): the cycle is the dense inverse,
    formed 32 columns a step; remainders of the steps and tiles, and the pivot
    test in the first, a middle and the last step."""
    import torch

    spk = need_gpu()
    A = spkgen.laplace_grid((n,), 0.3)
    D = spkgen.to_dense(A)
    b = spkgen.rhs_uniform(n, 5)
    with mat_on_gpu(spk, A) as M, spk.mg_create(M, (n,), spk.mg_opts(max_levels=1, coarse_max=4096)) as H:
        x = torch.full((n,), np.nan, dtype=torch.float64, device="cuda")
        spk.mg_apply(H, to_dev(b), x)
        # condition below 20: the inverse's error stays below n kappa u of the largest entry
        assert np.max(np.abs(x.cpu().numpy() - np.linalg.solve(D, b))) <= n * 20 * 2.0 ** -50
    r = np.repeat(np.arange(n), np.diff(A.rowptr))
    for at in {0, n // 2, n - 1}:
        val = A.val.copy()
        val[(A.col == r) & (r == at)] = -0.5
        with mat_on_gpu(spk, spkgen.CSR(n, A.rowptr, A.col, val)) as M:
            with pytest.raises(spk.SpkError) as e:
                spk.mg_create(M, (n,), spk.mg_opts(max_levels=1, coarse_max=4096))
            assert e.value.status == spk.EINVAL


@pytest.mark.parametrize("n", [1, 63, 64, 65, 200, 1031])
@pytest.mark.parametrize("offsets", [(0,), (-1, 0), (-3, -1, 0, 2), (-130, -64, -1, 0, 1, 64), "first_and_last", "32"])
def test_shared_offsets_walk_same_bits(offsets, n):
    """Lists of one to 32 positions, odd and even, with slices whose gathers
    all fall inside the matrix, partly do, or that are empty: the bits of the
    walk with an offset per entry, in FP64 and FP32, and where the product is
    fused with others."""
    spk = need_gpu()
    import torch

    if offsets == "first_and_last":
        offsets = (1 - n, 0, n - 1) if n > 1 else (0,)
    elif offsets == "32":
        offsets = tuple(range(-17, 15))
    rng = np.random.default_rng(n)
    rows, cols = [], []
    for o in sorted(offsets):
        i = np.arange(max(0, -o), min(n, n - o))
        rows.append(i)
        cols.append(i + o)
    rows, cols = np.concatenate(rows), np.concatenate(cols)
    keep = (rows // 64 != 1) | (n > 1000)  # an empty slice in the middle
    rows, cols = rows[keep], cols[keep]
    order = np.lexsort((cols, rows))
    rows, cols = rows[order], cols[order]
    rowptr = np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=n))]).astype(np.int32)
    val = np.where(rows == cols, 70.0, 0.0) + rng.standard_normal(rows.size)
    A = spkgen.CSR(n, rowptr, cols.astype(np.int32), val)
    x = to_dev(rng.standard_normal(n))
    lens = np.diff(rowptr)
    longest = sum(lens[i:i + 64].max() for i in range(0, n, 64))
    if 16 * sum(_shared_layout(A)[0]) > 17 * longest:  # grows the storage by more than a sixteenth
        M = mat_on_gpu(spk, A)
        with pytest.raises(spk.SpkError):
            spk.mat_set_kernel(M, spk.KERNEL_SELL, spk.SELL_SHARED)
        return
    res = []
    for param in (spk.SELL_SHARED, 32):
        M = mat_on_gpu(spk, A, flags=spk.MAT_MIXED)
        spk.mat_set_kernel(M, spk.KERNEL_SELL, param)
        y, y32 = torch.full_like(x, np.nan), torch.full_like(x.float(), np.nan)
        spk.mat_mult(M, x, y)
        spk.mat_mult_f32(M, x.float(), y32)
        out = [y, y32]
        if M.info.zero_diag_rows == 0:
            s = torch.full_like(x, np.nan)
            spk.pc_chebyshev(M, x, s, 3, 0.2, 2.0)
            z = torch.zeros_like(x)
            spk.ksp_solve(M, x, z, spk.ksp_opts(maxit=5, precision=spk.PREC_MIXED))
            out += [s, z]
        res.append([o.cpu().numpy() for o in out])
        M.close()
    for a, b in zip(*res):
        assert np.array_equal(a, b, equal_nan=True)


def _shuffled(n, seed):
    """A diagonally dominant tridiagonal matrix, rows and columns permuted alike:
    few entries a row, far more than 32 offsets a slice."""
    A = spkgen.laplace_grid((n,), 0.25)
    to = np.random.default_rng(seed).permutation(n)
    row, col = to[np.repeat(np.arange(n), np.diff(A.rowptr))], to[A.col]
    order = np.lexsort((col, row))
    rowptr = np.concatenate([[0], np.cumsum(np.bincount(row, minlength=n))]).astype(np.int32)
    return spkgen.CSR(n, rowptr, col[order].astype(np.int32), A.val[order])


@pytest.mark.parametrize("kernel,param", [("AUTO", 0), ("SELL", 16), ("SELL", 32), ("SELL_SIGMA", 256), ("STREAM", 8),
                                          ("VECTOR", 4), ("MERGE", 0), ("SLICED", 4), ("SLICED", 2048)])
@pytest.mark.parametrize("flags", [0, 1])
def test_refused_kernel_changes_nothing(kernel, param, flags):
    """Offsets that slices cannot share are found out while building: the
    handle goes on with the layout it had, bit for bit, in every call."""
    spk = need_gpu()
    import torch

    A = _shuffled(3000, 5)
    ref, M = (mat_on_gpu(spk, A, flags=flags) for _ in range(2))
    for m in (ref, M):
        spk.mat_set_kernel(m, getattr(spk, "KERNEL_" + kernel), param)
    for k, p in ((spk.KERNEL_SELL, spk.SELL_SHARED), (spk.KERNEL_VECTOR, 3), (spk.KERNEL_SELL_SIGMA, 100), (99, 0)):
        with pytest.raises(spk.SpkError) as e:
            spk.mat_set_kernel(M, k, p)
        assert e.value.status == spk.EINVAL
    M.info = spk.mat_get_info(M)
    assert (M.info.kernel, M.info.lanes, M.info.stored_nnz) == (
        ref.info.kernel, ref.info.lanes, ref.info.stored_nnz)
    assert M.info.device_bytes <= ref.info.device_bytes  # a SELL copy that is not in use goes
    if M.info.kernel == spk.KERNEL_SELL:
        assert M.info.device_bytes == ref.info.device_bytes
    b = to_dev(spkgen.rhs_uniform(A.n, 1))

    def outputs(m):
        y, x, z = (torch.zeros_like(b) for _ in range(3))
        spk.mat_mult(m, b, y)
        spk.ksp_solve(m, b, x, spk.ksp_opts(precision=spk.PREC_MIXED if flags else spk.PREC_FP64))
        spk.pc_chebyshev(m, b, z, 3)
        return y, x, z

    for got, want in zip(outputs(M), outputs(ref)):
        assert torch.equal(got, want)
    ref.close()
    M.close()
