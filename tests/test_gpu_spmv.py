"""SpMV parity: every kernel family against the oracle on the same seeded
inputs (bit-exact on integer data; per-row bound elsewhere, 1e-14 of
sum_j |a_ij x_j| for the kernels the library selects)."""

import numpy as np
import pytest

import oracle
import spkgen
from gpu_util import U32, U64, check_spmv, mat_on_gpu, need_gpu, spmv_bound_rows, to_dev

pytestmark = pytest.mark.gpu

KERNELS = [("auto", 0), ("stream", 0), ("stream", 64), ("stream", 8), ("merge", 0), ("sell", 0),
           ("sell", 1), ("sell", 16), ("sell", 32), ("sell_sigma", 0), ("sell_sigma", 64), ("sell_sigma", 1024), ("sliced", 0),
           ("sliced", 1), ("sliced", 16), ("sliced", 2048)] + [("vector", L) for L in (1, 2, 4, 8, 16, 32, 64)]


def _set(spk, M, kernel, param):
    if kernel == "auto":
        return spk.KERNEL_NAMES[M.info.kernel], M.info.lanes
    k = {"stream": spk.KERNEL_STREAM, "vector": spk.KERNEL_VECTOR, "merge": spk.KERNEL_MERGE,
         "sell": spk.KERNEL_SELL, "sliced": spk.KERNEL_SLICED, "sell_sigma": spk.KERNEL_SELL_SIGMA}[kernel]
    if kernel == "sell" and param == spk.SELL_SHARED:
        # shared offsets: refused (EINVAL) where a slice's rows use more than 32 offsets
        try:
            spk.mat_set_kernel(M, k, param)
        except spk.SpkError as e:
            assert e.status == spk.EINVAL
            return None, None
        assert M.info.lanes == 0
        return kernel, 0
    spk.mat_set_kernel(M, k, param)
    assert spk.KERNEL_NAMES[M.info.kernel] == kernel
    if kernel == "sell" and param:
        assert M.info.lanes == param
    if kernel == "sell_sigma":
        assert M.info.sell_sigma == (param or 4096)
    return kernel, M.info.lanes


def _matrices():
    rng = np.random.default_rng(7)
    D = rng.integers(-9, 10, size=(300, 300)) * (rng.random((300, 300)) < 0.05)
    D[5] = 0  # an empty row
    D[:, 7] = 0
    yield "int_random_300", spkgen.dense_to_csr(D.astype(np.float64)), True
    yield "lap2d_64", spkgen.laplace2d5(64), True
    yield "lap2d_61_ragged", spkgen.laplace2d5(61), True
    yield "lap3d_23", spkgen.laplace3d7(23), True
    yield "diff27_13", spkgen.diffusion3d27_lognormal(13, seed=1), False
    yield "powerlaw_30k", spkgen.powerlaw_spd(30000, seed=3), False


@pytest.mark.parametrize("kernel,param", KERNELS)
def test_spmv_parity_fp64(kernel, param):
    spk = need_gpu()
    for name, A, integer in _matrices():
        M = mat_on_gpu(spk, A)
        kname, lanes = _set(spk, M, kernel, param)
        if kname is None:
            M.close()
            continue
        if integer:
            x = np.random.default_rng(1).integers(-50, 50, size=A.n).astype(np.float64)
        else:
            x = spkgen.rhs_uniform(A.n, 2)
        y = to_dev(np.full(A.n, np.nan))
        spk.mat_mult(M, to_dev(x), y)
        y = y.cpu().numpy()
        ref = oracle.spmv(A, x)
        if integer:
            assert np.array_equal(y, ref), f"{name} {kname}: not bit-exact"
        else:
            scale = oracle.spmv_abs(A, x)
            bound = np.maximum(spmv_bound_rows(A, kname, lanes, U64), 0.0)
            if kernel == "auto":
                bound = np.minimum(bound, 1e-14)  # the selected kernel meets 1e-14
            check_spmv(y, ref, scale, bound, f"{name} {kname}/{lanes}")
        M.close()


@pytest.mark.parametrize("kernel,param", [("auto", 0), ("stream", 0), ("merge", 0), ("vector", 4),
                                          ("vector", 64), ("sell", 0), ("sell", 1), ("sell", 16),
                                          ("sell_sigma", 512), ("sliced", 0), ("sliced", 2048)])
def test_spmv_parity_fp32(kernel, param):
    spk = need_gpu()
    for name, A, integer in _matrices():
        M = mat_on_gpu(spk, A, flags=spk.MAT_MIXED)
        kname, lanes = _set(spk, M, kernel, param)
        if kname is None:
            M.close()
            continue
        if integer:
            x = np.random.default_rng(1).integers(-50, 50, size=A.n).astype(np.float32)
        else:
            x = spkgen.rhs_uniform(A.n, 2).astype(np.float32)
        y = to_dev(np.full(A.n, np.nan, dtype=np.float32))
        spk.mat_mult_f32(M, to_dev(x), y)
        y = y.cpu().numpy()
        v32 = A.val.astype(np.float32)
        ref = oracle.spmv_f32(A, x, val32=v32)
        if integer:
            assert np.array_equal(y, ref), f"{name} {kname}: FP32 not bit-exact"
        else:
            Af = spkgen.CSR(A.n, A.rowptr, A.col, v32.astype(np.float64))
            scale = oracle.spmv_abs(Af, x.astype(np.float64))
            bound = spmv_bound_rows(A, kname, lanes, U32) + U32  # + final rounding
            check_spmv(y.astype(np.float64), ref.astype(np.float64), scale, bound,
                       f"fp32 {name} {kname}/{lanes}")
        M.close()


def test_spmv_degenerate_sizes():
    spk = need_gpu()
    import torch

    # n = 1
    A = spkgen.dense_to_csr(np.array([[3.0]]))
    M = mat_on_gpu(spk, A)
    y = torch.zeros(1, dtype=torch.float64, device="cuda")
    spk.mat_mult(M, to_dev(np.array([2.0])), y)
    assert y.item() == 6.0
    # n = 0
    E = spkgen.CSR(0, np.zeros(1, np.int32), np.zeros(0, np.int32), np.zeros(0))
    M0 = mat_on_gpu(spk, E)
    e = torch.zeros(0, dtype=torch.float64, device="cuda")
    spk.mat_mult(M0, e, e.clone())
    # all rows empty
    Z = spkgen.CSR(1000, np.zeros(1001, np.int32), np.zeros(0, np.int32), np.zeros(0))
    for k in (spk.KERNEL_STREAM, spk.KERNEL_MERGE, spk.KERNEL_VECTOR, spk.KERNEL_SELL, spk.KERNEL_SLICED):
        MZ = mat_on_gpu(spk, Z)
        spk.mat_set_kernel(MZ, k, 8 if k == spk.KERNEL_VECTOR else 0)
        y = torch.full((1000,), 5.0, dtype=torch.float64, device="cuda")
        spk.mat_mult(MZ, torch.ones(1000, dtype=torch.float64, device="cuda"), y)
        assert (y == 0).all()


def test_spmv_one_long_row():
    """A dense row of 100k entries (beyond every tile), plus short rows."""
    spk = need_gpu()
    n = 100000
    rows = [np.arange(n, dtype=np.int32)] + [np.array([i], dtype=np.int32) for i in range(1, 3000)]
    cols = np.concatenate(rows)
    rowptr = np.zeros(3001, np.int32)
    rowptr[1:] = np.cumsum([r.size for r in rows])
    rowptr_full = np.concatenate([rowptr, np.full(n - 3000, rowptr[-1], np.int32)])
    vals = np.random.default_rng(0).integers(-3, 4, size=cols.size).astype(np.float64)
    A = spkgen.CSR(n, rowptr_full, cols, vals)
    x = np.random.default_rng(1).integers(-3, 4, size=n).astype(np.float64)
    ref = oracle.spmv(A, x)
    for k, p in ((spk.KERNEL_AUTO, 0), (spk.KERNEL_STREAM, 256), (spk.KERNEL_MERGE, 0),
                 (spk.KERNEL_VECTOR, 64)):
        M = mat_on_gpu(spk, A)
        spk.mat_set_kernel(M, k, p)
        y = to_dev(np.zeros(n))
        spk.mat_mult(M, to_dev(x), y)
        assert np.array_equal(y.cpu().numpy(), ref)


def _shuffle_rows(A, seed):
    """The same matrix with the entries of every row in random order."""
    rng = np.random.default_rng(seed)
    key = np.repeat(np.arange(A.n), np.diff(A.rowptr)) * 2.0 + rng.random(A.nnz)
    perm = np.argsort(key, kind="stable")
    return spkgen.CSR(A.n, A.rowptr, A.col[perm].copy(), A.val[perm].copy())


def test_spmv_unsorted_rows_every_family():
    """Rows need not be sorted (only SPK_MAT_VALIDATE asks for it): a
    power-law matrix of 2^19 rows with wide columns (the automatic choice is
    the column-sliced layout, whose setup splits each row by column range)
    and its rows shuffled gives the oracle's product, bit-exact on integer
    values, with every kernel family."""
    spk = need_gpu()
    B = spkgen.powerlaw_spd(1 << 19, seed=4, hi=200)
    vals = np.random.default_rng(2).integers(-9, 10, B.nnz).astype(np.float64)
    A = _shuffle_rows(spkgen.CSR(B.n, B.rowptr, B.col, vals), 5)
    assert np.any(np.diff(A.col[A.rowptr[0]:A.rowptr[1]]) < 0) or np.any(np.diff(A.col) < 0)
    x = np.random.default_rng(3).integers(-50, 50, A.n).astype(np.float64)
    ref = oracle.spmv(A, x)
    M = mat_on_gpu(spk, A)
    assert spk.KERNEL_NAMES[M.info.kernel] == "sliced"
    for k, p in ((spk.KERNEL_AUTO, 0), (spk.KERNEL_SLICED, 8), (spk.KERNEL_SLICED, 2048),
                 (spk.KERNEL_MERGE, 0), (spk.KERNEL_VECTOR, 16), (spk.KERNEL_STREAM, 0), (spk.KERNEL_SELL, 32)):
        spk.mat_set_kernel(M, k, p)
        y = to_dev(np.full(A.n, np.nan))
        spk.mat_mult(M, to_dev(x), y)
        assert np.array_equal(y.cpu().numpy(), ref), spk.KERNEL_NAMES[M.info.kernel]


def _sell_sigma_stored(A, sigma):
    """Stored entries of SELL-C-sigma: rows ordered by length (longest first,
    ties in row order) within windows of sigma rows, slices of 64 rows padded
    to their longest."""
    lens = np.diff(A.rowptr).astype(np.int64)
    order = np.concatenate([w0 + np.argsort(-lens[w0:w0 + sigma], kind="stable")
                            for w0 in range(0, A.n, sigma)])
    sl = lens[order]
    sl = np.concatenate([sl, np.zeros(-A.n % 64, np.int64)])
    return 64 * int(sl.reshape(-1, 64).max(axis=1).sum())


def test_spmv_sell_sigma_layout():
    """SELL-C-sigma on a power-law matrix (rows up to 1000 entries, so 16-bit
    lengths): the stored entries are those of the sorted windows, sorting
    shrinks the padding against plain SELL, and the product is bit-exact on
    integer data for several windows, FP64 and FP32."""
    spk = need_gpu()
    import torch

    B = spkgen.powerlaw_spd(50001, seed=6, hi=1000)
    vals = np.random.default_rng(3).integers(-5, 6, B.nnz).astype(np.float64)
    A = spkgen.CSR(B.n, B.rowptr, B.col, vals)
    assert np.diff(A.rowptr).max() > 255
    x = np.random.default_rng(4).integers(-20, 21, A.n).astype(np.float64)
    ref = oracle.spmv(A, x)
    M = mat_on_gpu(spk, A, flags=spk.MAT_MIXED)
    spk.mat_set_kernel(M, spk.KERNEL_SELL, 0)
    plain = M.info.stored_nnz
    assert plain == _sell_stored(A)
    for sigma in (64, 1024, 50048):
        spk.mat_set_kernel(M, spk.KERNEL_SELL_SIGMA, sigma)
        info = M.info
        assert spk.KERNEL_NAMES[info.kernel] == "sell_sigma" and info.sell_sigma == sigma
        assert info.stored_nnz == _sell_sigma_stored(A, sigma)
        if sigma >= 1024:
            assert info.stored_nnz < plain
        y = to_dev(np.full(A.n, np.nan))
        spk.mat_mult(M, to_dev(x), y)
        assert np.array_equal(y.cpu().numpy(), ref), sigma
        y32 = torch.full((A.n,), float("nan"), dtype=torch.float32, device="cuda")
        spk.mat_mult_f32(M, to_dev(x, torch.float32), y32)
        assert np.array_equal(y32.cpu().numpy().astype(np.float64), ref), sigma
    with pytest.raises(spk.SpkError):
        spk.mat_set_kernel(M, spk.KERNEL_SELL_SIGMA, 100)


def _sell_stored(A):
    lens = np.diff(A.rowptr)
    pad = (-A.n) % 64
    return int(np.pad(lens, (0, pad)).reshape(-1, 64).max(axis=1).sum()) * 64


def test_spmv_sell_layout_and_offsets():
    """SELL-64: int16 offsets when every |col - row| < 2^15, int32 otherwise
    (int16 refused then); padding never enters a sum; bit-exact on integers."""
    spk = need_gpu()
    rng = np.random.default_rng(11)
    n = 70001  # ragged last slice
    lens = rng.integers(0, 10, size=n)
    lens[64:128] = 0  # an all-empty slice
    lens[1000] = 255  # the longest row SELL stores
    rowptr = np.zeros(n + 1, np.int64)
    rowptr[1:] = np.cumsum(lens)
    far = [np.sort(rng.choice(n, size=k, replace=False)) for k in lens]
    near = []
    for i, k in enumerate(lens):
        lo, hi = max(0, i - 30000), min(n, i + 30000)
        near.append(np.sort(rng.choice(np.arange(lo, hi), size=k, replace=False)))
    vals = rng.integers(-4, 5, size=int(rowptr[-1])).astype(np.float64)
    x = rng.integers(-4, 5, size=n).astype(np.float64)
    for cols, width in ((far, 32), (near, 16)):
        A = spkgen.CSR(n, rowptr.astype(np.int32), np.concatenate(cols).astype(np.int32), vals)
        M = mat_on_gpu(spk, A)
        if width == 32:
            with pytest.raises(spk.SpkError):
                spk.mat_set_kernel(M, spk.KERNEL_SELL, 16)
        spk.mat_set_kernel(M, spk.KERNEL_SELL, 0)
        info = M.info
        assert spk.KERNEL_NAMES[info.kernel] == "sell" and info.lanes == width
        stored = _sell_stored(A)
        assert info.stored_nnz == stored
        cw = width // 8
        ns = (n + 63) // 64
        assert info.format_bytes_spmv_f64 == (8 + cw) * stored + 4 * (ns + 1) + n + 16 * n
        y = to_dev(np.full(n, np.nan))
        spk.mat_mult(M, to_dev(x), y)
        assert np.array_equal(y.cpu().numpy(), oracle.spmv(A, x))
        M.close()


def test_kernel_selection():
    spk = need_gpu()
    sel = {}
    for name, A, _ in _matrices():
        M = mat_on_gpu(spk, A)
        sel[name] = spk.KERNEL_NAMES[M.info.kernel]
    # banded short rows: SELL-64 with int16 offsets; skewed rows: merge path
    assert sel["lap3d_23"] == "sell" and sel["diff27_13"] == "sell"
    assert sel["lap2d_64"] == "sell" and sel["int_random_300"] != "sell"
    assert sel["powerlaw_30k"] == "merge"


def test_invalid_csr_rejected():
    spk = need_gpu()
    A = spkgen.laplace2d5(8)
    bad = A.col.copy()
    bad[10] = 64  # out of range
    with pytest.raises(spk.SpkError) as e:
        spk.mat_create_csr(to_dev(A.rowptr), to_dev(bad), to_dev(A.val))
    assert e.value.status == spk.EINVAL
    rp = A.rowptr.copy()
    rp[5], rp[6] = rp[6], rp[5]  # not monotone
    with pytest.raises(spk.SpkError):
        spk.mat_create_csr(to_dev(rp), to_dev(A.col), to_dev(A.val))
    uns = A.col.copy()
    uns[0], uns[1] = uns[1], uns[0]
    with pytest.raises(spk.SpkError):
        spk.mat_create_csr(to_dev(A.rowptr), to_dev(uns), to_dev(A.val), flags=spk.MAT_VALIDATE)
    # host path checks rowptr[n] on the host
    with pytest.raises(spk.SpkError):
        spk.mat_create_csr(A.rowptr[:-1], A.col, A.val)


def test_host_memtype_and_borrow_match():
    spk = need_gpu()
    A = spkgen.diffusion3d27_lognormal(9, seed=2)
    x = to_dev(spkgen.rhs_uniform(A.n, 0))
    M1 = spk.mat_create_csr(A.rowptr, A.col, A.val)  # host arrays
    M2 = spk.mat_create_csr(to_dev(A.rowptr), to_dev(A.col), to_dev(A.val), flags=spk.MAT_BORROW)
    y1 = to_dev(np.zeros(A.n))
    y2 = to_dev(np.zeros(A.n))
    spk.mat_mult(M1, x, y1)
    spk.mat_mult(M2, x, y2)
    assert np.array_equal(y1.cpu().numpy(), y2.cpu().numpy())



def test_sell_load_policy_same_bits():
    """The SELL load policy (ordinary loads for a layout that fits the
    Infinity Cache, nontemporal loads above it or with MAT_STREAM) changes
    speed only: FP64 and FP32 products and FP64 / mixed solves give the same
    bits either way, and both match the oracle."""
    spk = need_gpu()
    import torch

    A = spkgen.diffusion3d27_lognormal(17, seed=6)
    Mc = mat_on_gpu(spk, A, flags=spk.MAT_MIXED)
    Ms = mat_on_gpu(spk, A, flags=spk.MAT_MIXED | spk.MAT_STREAM)
    assert spk.KERNEL_NAMES[Mc.info.kernel] == "sell" == spk.KERNEL_NAMES[Ms.info.kernel]
    assert Mc.info.cached_loads == 15 and Ms.info.cached_loads == 0
    x = spkgen.rhs_uniform(A.n, 2)
    ys = []
    for M in (Mc, Ms):
        y = to_dev(np.zeros(A.n))
        spk.mat_mult(M, to_dev(x), y)
        y32 = to_dev(np.zeros(A.n), torch.float32)
        spk.mat_mult_f32(M, to_dev(x, torch.float32), y32)
        ys.append((y.cpu().numpy(), y32.cpu().numpy()))
    assert np.array_equal(ys[0][0], ys[1][0]) and np.array_equal(ys[0][1], ys[1][1])
    scale = oracle.spmv_abs(A, x)
    check_spmv(ys[0][0], oracle.spmv(A, x), scale, spmv_bound_rows(A, "sell", 0, U64), "sell fp64")
    b = spkgen.rhs_uniform(A.n, 3)
    for prec in (spk.PREC_FP64, spk.PREC_MIXED):
        o = spk.ksp_opts_default()
        o.rtol, o.precision = 1e-8, prec
        sols = []
        for M in (Mc, Ms):
            xs = to_dev(np.zeros(A.n))
            res = spk.ksp_solve(M, to_dev(b), xs, o)
            sols.append((res.iterations, xs.cpu().numpy()))
        assert sols[0][0] == sols[1][0] and np.array_equal(sols[0][1], sols[1][1])

def test_spmv_deterministic_repeat():
    spk = need_gpu()
    A = spkgen.powerlaw_spd(20000, seed=5)
    M = mat_on_gpu(spk, A)
    x = to_dev(spkgen.rhs_uniform(A.n, 5))
    ys = []
    for _ in range(3):
        y = to_dev(np.zeros(A.n))
        spk.mat_mult(M, x, y)
        ys.append(y.cpu().numpy())
    assert np.array_equal(ys[0], ys[1]) and np.array_equal(ys[0], ys[2])


def test_jacobi_and_vector_kernels():
    spk = need_gpu()
    import torch

    A = spkgen.diffusion3d27_lognormal(10, seed=4)
    M = mat_on_gpu(spk, A)
    r = spkgen.rhs_uniform(A.n, 1)
    z = to_dev(np.zeros(A.n))
    spk.pc_jacobi_apply(M, to_dev(r), z)
    dinv = oracle.diag_inv(A)
    assert np.array_equal(z.cpu().numpy(), oracle.jacobi_apply(dinv, r))
    n = 1_000_003
    x = spkgen.rhs_uniform(n, 10)
    y = spkgen.rhs_uniform(n, 11)
    w = spkgen.rhs_uniform(n, 12)
    yd = to_dev(y)
    spk.vec_axpy(0.37, to_dev(x), yd)
    assert np.array_equal(yd.cpu().numpy(), oracle.axpy(0.37, x, y))
    yd = to_dev(y)
    spk.vec_aypx(-1.25, to_dev(x), yd)
    assert np.array_equal(yd.cpu().numpy(), oracle.aypx(-1.25, x, y))
    res = torch.zeros(2, dtype=torch.float64, device="cuda")
    spk.vec_dot(to_dev(x), to_dev(y), res)
    d = res[0].item()
    assert abs(d - oracle.dot(x, y)) <= 1e-13 * np.abs(x * y).sum()
    spk.vec_dot2(to_dev(x), to_dev(y), to_dev(w), res)
    r2 = res.cpu().numpy()
    assert r2[0] == d  # same reduction tree
    assert abs(r2[1] - oracle.dot(x, w)) <= 1e-13 * np.abs(x * w).sum()
    spk.vec_nrm2(to_dev(x), res)
    assert abs(res[0].item() - oracle.nrm2(x)) <= 1e-14 * oracle.nrm2(x)
    # integer vectors: exact
    xi = np.random.default_rng(3).integers(-1000, 1000, size=n).astype(np.float64)
    spk.vec_dot(to_dev(xi), to_dev(xi), res)
    assert res[0].item() == oracle.dot(xi, xi)


@pytest.mark.parametrize("case", ["even_rows", "powerlaw"])
def test_sliced_selection_solves_and_fp32(case):
    """Scattered-column matrices whose x (4.8 MB) exceeds one XCD's L2, with
    even row lengths (16 uniform picks per row, symmetrised) or power-law
    rows, select the column-sliced family (merge path over the slices);
    FP64 and FP32 products meet their bounds, one-lane, four-lane and merge
    launches are bit-exact on integers, and FP64 / mixed Jacobi-PCG solves
    with it match the oracle's counts."""
    spk = need_gpu()
    import torch

    if case == "even_rows":
        A = spkgen.powerlaw_spd(600_000, seed=5, lo=16, hi=16)
    else:
        A = spkgen.powerlaw_spd(600_000, seed=5)
    M = mat_on_gpu(spk, A, flags=spk.MAT_MIXED)
    assert spk.KERNEL_NAMES[M.info.kernel] == "sliced" and M.info.lanes == 2048  # merge path over the slices
    x = spkgen.rhs_uniform(A.n, 1)
    y = torch.empty(A.n, dtype=torch.float64, device="cuda")
    spk.mat_mult(M, to_dev(x), y)
    scale = oracle.spmv_abs(A, x)
    check_spmv(y.cpu().numpy(), oracle.spmv(A, x), scale, 1e-14, "sliced fp64")
    x32 = x.astype(np.float32)
    y32 = torch.empty(A.n, dtype=torch.float32, device="cuda")
    spk.mat_mult_f32(M, to_dev(x32), y32)
    v32 = A.val.astype(np.float32)
    Af = spkgen.CSR(A.n, A.rowptr, A.col, v32.astype(np.float64))
    bound = spmv_bound_rows(A, "sliced", M.info.lanes, U32) + U32
    check_spmv(y32.cpu().numpy().astype(np.float64), oracle.spmv_f32(A, x32, val32=v32).astype(np.float64),
               oracle.spmv_abs(Af, x32.astype(np.float64)), bound, "sliced fp32")
    # integer data: exact whatever the order
    Ai = spkgen.CSR(A.n, A.rowptr, A.col, np.round(A.val * 4))
    Mi = mat_on_gpu(spk, Ai)
    spk.mat_set_kernel(Mi, spk.KERNEL_SLICED, 0)
    xi = np.random.default_rng(2).integers(-20, 20, A.n).astype(np.float64)
    spk.mat_mult(Mi, to_dev(xi), y)
    assert np.array_equal(y.cpu().numpy(), oracle.spmv(Ai, xi))
    for p in (1, 4, 2048):
        spk.mat_set_kernel(Mi, spk.KERNEL_SLICED, p)
        spk.mat_mult(Mi, to_dev(xi), y)
        assert np.array_equal(y.cpu().numpy(), oracle.spmv(Ai, xi))
    # solves on the selected family
    b = spkgen.rhs_uniform(A.n, 0)
    _, ro, _ = oracle.pcg(A, b)
    for prec in (spk.PREC_FP64, spk.PREC_MIXED):
        xs = torch.zeros(A.n, dtype=torch.float64, device="cuda")
        res = spk.ksp_solve(M, to_dev(b), xs, spk.ksp_opts(precision=prec))
        assert res.reason == spk.CONVERGED_RTOL
        it = res.iterations if prec == spk.PREC_FP64 else res.inner_iterations
        assert abs(it - ro["iterations"]) <= max(2, 0.01 * ro["iterations"])
        assert oracle.nrm2(b - oracle.spmv(A, xs.cpu().numpy())) <= 1e-8 * oracle.nrm2(b) * (1 + 1e-6)


def test_cache_flush_reads_only():
    """The cache eviction helper reads its scratch buffer and leaves it as it
    was (the bench's cold SpMV measurement relies on a clean eviction)."""
    spk = need_gpu()
    import torch

    s = torch.arange(1 << 20, dtype=torch.float64, device="cuda")
    ref = s.clone()
    spk.cache_flush(s)
    torch.cuda.synchronize()
    assert torch.equal(s, ref)
    with pytest.raises(spk.SpkError):
        spk.cache_flush(s[:1])  # fewer than 16 bytes


def _shared_layout(A):
    """Slice widths and offset lists of the shared-offset layout, or None when
    a slice's rows use more than 32 distinct offsets (host restatement of the
    layout's definition, for the byte and entry counts)."""
    widths, nlist = [], 0
    for s0 in range(0, A.n, 64):
        offs = set()
        for r in range(s0, min(A.n, s0 + 64)):
            offs.update(int(c) - r for c in A.col[A.rowptr[r]:A.rowptr[r + 1]])
        if len(offs) > 32:
            return None
        widths.append(len(offs))
        nlist += len(offs)
    return widths, nlist


def test_spmv_sell_shared_offsets():
    """Shared offsets (one offset list per slice, a position mask per row)
    against per-lane int16 offsets on the same matrices: the same bits in
    FP64 and FP32 (the row's entries in the same order, unused positions
    never multiplied), stored entries and format bytes as the layout defines
    them; gathers of unused positions near row 0 and row n - 1 stay in
    bounds (ragged last slice, a 3-row matrix); empty rows and an empty
    slice give zeros; matrices whose slices need more than 32
    offsets or whose rows are unsorted keep per-lane offsets under the
    automatic choice and are refused when shared offsets are forced."""
    spk = need_gpu()
    # rows emptied out of a 2D Laplacian: scattered empty rows and one whole
    # empty slice (rows 640..703), which then has no offsets at all
    L = spkgen.laplace2d5(40)
    keep = np.ones(L.n, bool)
    keep[::37] = False
    keep[640:704] = False
    lens = np.where(keep, np.diff(L.rowptr), 0)
    rp = np.zeros(L.n + 1, np.int32)
    rp[1:] = np.cumsum(lens)
    sel = np.repeat(keep, np.diff(L.rowptr))
    holes = spkgen.CSR(L.n, rp, L.col[sel].astype(np.int32), L.val[sel])
    tri3 = spkgen.dense_to_csr(np.array([[4.0, -1, 0], [-1, 4, -1], [0, -1, 4]]))
    mats = [("lap2d_61_ragged", spkgen.laplace2d5(61)), ("lap3d_23", spkgen.laplace3d7(23)),
            ("diff27_13", spkgen.diffusion3d27_lognormal(13, seed=1)), ("lap2d_40_holes", holes),
            ("tridiag_3", tri3)]
    for name, A in mats:
        lay = _shared_layout(A)
        assert lay is not None, name
        widths, nlist = lay
        x = spkgen.rhs_uniform(A.n, 4)
        outs = []
        for param in (spk.SELL_SHARED, 16):
            M = mat_on_gpu(spk, A, flags=spk.MAT_MIXED)
            spk.mat_set_kernel(M, spk.KERNEL_SELL, param)
            info = M.info
            if param == spk.SELL_SHARED:
                assert info.lanes == 0
                stored = 64 * sum(widths)
                assert info.stored_nnz == stored
                ns = (A.n + 63) // 64
                assert info.format_bytes_spmv_f64 == 8 * stored + 4 * (ns + 1) + 16 * A.n + 4 * nlist + 4 * A.n
            y = to_dev(np.full(A.n, np.nan))
            spk.mat_mult(M, to_dev(x), y)
            y32 = to_dev(np.full(A.n, np.nan, dtype=np.float32))
            spk.mat_mult_f32(M, to_dev(x.astype(np.float32)), y32)
            outs.append((y.cpu().numpy(), y32.cpu().numpy()))
            M.close()
        assert np.array_equal(outs[0][0].view(np.int64), outs[1][0].view(np.int64)), name
        assert np.array_equal(outs[0][1].view(np.int32), outs[1][1].view(np.int32)), name
        scale = oracle.spmv_abs(A, x)
        check_spmv(outs[0][0], oracle.spmv(A, x), scale, spmv_bound_rows(A, "sell", 0, U64), name)
    # a slice whose rows use more than 32 offsets between them
    rng = np.random.default_rng(3)
    A = spkgen.powerlaw_spd(3000, seed=2)
    assert _shared_layout(A) is None
    M = mat_on_gpu(spk, A)
    with pytest.raises(spk.SpkError) as e:
        spk.mat_set_kernel(M, spk.KERNEL_SELL, spk.SELL_SHARED)
    assert e.value.status == spk.EINVAL
    spk.mat_set_kernel(M, spk.KERNEL_SELL, 0)
    assert M.info.lanes == 16
    M.close()
    # unsorted rows: per-lane offsets keep each row's own order
    L = spkgen.laplace2d5(20)
    col = L.col.copy()
    for r in range(0, L.n, 7):
        a, b = L.rowptr[r], L.rowptr[r + 1]
        col[a:b] = col[a:b][::-1]
    val = L.val.copy()
    for r in range(0, L.n, 7):
        a, b = L.rowptr[r], L.rowptr[r + 1]
        val[a:b] = val[a:b][::-1]
    U = spkgen.CSR(L.n, L.rowptr, col, val)
    M = mat_on_gpu(spk, U)
    with pytest.raises(spk.SpkError):
        spk.mat_set_kernel(M, spk.KERNEL_SELL, spk.SELL_SHARED)
    spk.mat_set_kernel(M, spk.KERNEL_SELL, 0)
    assert M.info.lanes == 16
    xi = rng.integers(-9, 10, size=U.n).astype(np.float64)
    y = to_dev(np.full(U.n, np.nan))
    spk.mat_mult(M, to_dev(xi), y)
    assert np.array_equal(y.cpu().numpy(), oracle.spmv(U, xi))
    M.close()


BIN, TILE = 16384, 4096  # columns of a bin, merge-path items (rows and entries) of a tile


def _scattered(n, lens, seed):
    """Rows of the given lengths, random columns (with repeats), small integers."""
    rng = np.random.default_rng(seed)
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    col = rng.integers(0, n, rowptr[-1]).astype(np.int32)
    return spkgen.CSR(n, rowptr, col, rng.integers(-9, 10, rowptr[-1]).astype(np.float64))


@pytest.mark.parametrize("case", ["one_row", "one_tile", "two_tiles", "bins_1", "bins_2", "bins_2_full", "bins_3",
                                  "long_row", "longest_row", "empty_rows", "one_bin_used", "no_entries", "bins_512", "bins_513"])
def test_binned_products(case):
    """The sliced family's merge path by column bins and row tiles (beyond 512
    bins: over the slices): exact on integers in FP64 and FP32, twice on the
    same handle, for rows that end with a tile, go on over several or are
    empty, and bins that are full, partly used or unused."""
    spk = need_gpu()
    import torch

    n, lens = {"one_row": (1, [1]), "one_tile": (100, [TILE // 100 - 1] * 99 + [TILE - 100 - 99 * (TILE // 100 - 1)]),
               "two_tiles": (100, [TILE // 100 - 1] * 99 + [TILE - 99 - 99 * (TILE // 100 - 1)]),
               "bins_1": (BIN, 3), "bins_2": (BIN + 1, 3), "bins_2_full": (2 * BIN, 2), "bins_3": (2 * BIN + 3, 5),
               "long_row": (BIN + 500, [1] * 300 + [5 * TILE + 7] + [2] * (BIN + 199)),
               "longest_row": (TILE, [1] * 5 + [25 * TILE] + [1] * (TILE - 7) + [8 * TILE]),
               "empty_rows": (3 * TILE, [0] * (TILE + 5) + [40] * 3 + [0] * (2 * TILE - 8)),
               "one_bin_used": (4 * BIN, 1), "no_entries": (300, 0), "bins_512": (512 * BIN, 1),
               "bins_513": (512 * BIN + 1, 1)}[case]
    lens = np.full(n, lens) if np.isscalar(lens) else np.array(lens)
    assert lens.size == n
    A = _scattered(n, lens, 7)
    if case == "one_bin_used":
        A = spkgen.CSR(n, A.rowptr, (2 * BIN + A.col % BIN).astype(np.int32), A.val)
    M = mat_on_gpu(spk, A, flags=spk.MAT_MIXED)
    spk.mat_set_kernel(M, spk.KERNEL_SLICED, 2048)
    assert spk.KERNEL_NAMES[M.info.kernel] == "sliced" and M.info.lanes == 2048
    for seed in (1, 2):
        x = np.random.default_rng(seed).integers(-50, 50, n).astype(np.float64)
        ref = oracle.spmv(A, x)
        y, y32 = to_dev(np.full(n, np.nan)), to_dev(np.full(n, np.nan, np.float32))
        spk.mat_mult(M, to_dev(x), y)
        spk.mat_mult_f32(M, to_dev(x.astype(np.float32)), y32)
        assert np.array_equal(y.cpu().numpy(), ref)
        assert np.array_equal(y32.cpu().numpy().astype(np.float64), ref)
    spk.mat_set_kernel(M, spk.KERNEL_SLICED, 4)  # and the copy is given back
    spk.mat_mult(M, to_dev(x), y)
    assert np.array_equal(y.cpu().numpy(), ref)
    M.close()


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("n", [1, 2, 3, 255, 511, 512, 513, 1025, 2048 * 256 * 4 + 5])
def test_vector_kernels_pairs(n, shift):
    """Two elements a lane where every operand is 16-byte aligned, one
    otherwise; odd tails; dots whose lanes hold less than, exactly and more
    than the elements loaded ahead.  Exact on integers, nothing written past
    the end."""
    spk = need_gpu()
    import torch

    rng = np.random.default_rng(n)
    xh, yh, dh = (rng.integers(-9, 10, n).astype(np.float64) for _ in range(3))
    dh = 2.0 ** dh  # exact inverses

    def place(a):
        buf = torch.full((n + 2,), -77.0, dtype=torch.float64, device="cuda")
        v = buf[shift:shift + n]
        v.copy_(torch.from_numpy(a))
        return buf, v

    bx, x = place(xh)
    by, y = place(yh)
    bz, z = place(xh)
    spk.vec_axpy(3.0, x, y)
    assert np.array_equal(y.cpu().numpy(), yh + 3 * xh)
    spk.vec_aypx(-2.0, x, y)
    want = xh - 2 * (yh + 3 * xh)
    assert np.array_equal(y.cpu().numpy(), want)
    D = spkgen.CSR(n, np.arange(n + 1, dtype=np.int32), np.arange(n, dtype=np.int32), dh)
    with mat_on_gpu(spk, D) as M:
        spk.pc_jacobi_apply(M, y, z)
    assert np.array_equal(z.cpu().numpy(), want / dh)
    for b in (bx, by, bz):
        h = b.cpu().numpy()
        assert h[:shift].tolist() == [-77.0] * shift and h[shift + n:].tolist() == [-77.0] * (2 - shift)
    res = torch.empty(2, dtype=torch.float64, device="cuda")
    spk.vec_dot(x, y, res)
    assert res[0].item() == float(np.dot(xh, want))
    spk.vec_dot2(x, y, x, res)
    assert res.tolist() == [float(np.dot(xh, want)), float(np.dot(xh, xh))]


@pytest.mark.parametrize("n", [(1 << 22) - 1, 1 << 22, (1 << 22) + 1, (1 << 23) + 5])
def test_dot_alone_and_with_another(n):
    """A single dot of a long vector loads one element ahead, two dots four:
    the lanes' sums and so the bits are the same."""
    spk = need_gpu()
    import torch

    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    x, y, w = (torch.randn(n, generator=g, device="cuda", dtype=torch.float64) for _ in range(3))
    one, two, norm = (torch.zeros(k, dtype=torch.float64, device="cuda") for k in (1, 2, 1))
    spk.vec_dot(x, y, one)
    spk.vec_dot2(x, y, w, two)
    assert one[0].item() == two[0].item()
    spk.vec_dot(x, x, one)
    spk.vec_nrm2(x, norm)
    assert norm[0].item() == np.sqrt(one[0].item())
    xi, yi = (v.mul(4).round() for v in (x, y))
    spk.vec_dot(xi, yi, one)
    assert one[0].item() == (xi.to(torch.int64) * yi.to(torch.int64)).sum().item()


@pytest.mark.parametrize("case", ["one_row", "one_tile", "two_tiles", "bins_1", "bins_2", "bins_2_full", "bins_3",
                                  "long_row", "longest_row", "empty_rows", "one_bin_used", "no_entries"])
def test_binned_products_of_few_rows(case, monkeypatch):
    """The binned kernels at their edges, on sizes that by themselves take the
    merge path over the slices."""
    monkeypatch.setenv("SPK_BINNED_ROWS", "1")
    test_binned_products(case)


@pytest.mark.parametrize("n", [(1 << 18) - 1, 1 << 18])
def test_sliced_or_binned(n):
    """The sliced family's merge path runs over bins from 2^18 rows on: exact
    on integers, and 20 bytes an entry instead of 12 and the slices' partials."""
    spk = need_gpu()
    A = _scattered(n, np.full(n, 16), 5)
    M = mat_on_gpu(spk, A, flags=spk.MAT_MIXED)
    spk.mat_set_kernel(M, spk.KERNEL_VECTOR, 8)
    before = M.info.device_bytes
    spk.mat_set_kernel(M, spk.KERNEL_SLICED, 2048)
    assert spk.KERNEL_NAMES[M.info.kernel] == "sliced" and M.info.lanes == 2048
    extra = (M.info.device_bytes - before) / A.nnz
    assert (24 <= extra < 25) if n >= 1 << 18 else (16 + 96 / 16 <= extra < 16 + 96 / 16 + 1), extra
    x = np.random.default_rng(1).integers(-50, 50, n).astype(np.float64)
    ref = oracle.spmv(A, x)
    y, y32 = to_dev(np.full(n, np.nan)), to_dev(np.full(n, np.nan, np.float32))
    spk.mat_mult(M, to_dev(x), y)
    spk.mat_mult_f32(M, to_dev(x.astype(np.float32)), y32)
    assert np.array_equal(y.cpu().numpy(), ref)
    assert np.array_equal(y32.cpu().numpy().astype(np.float64), ref)
    M.close()


@pytest.mark.parametrize("param", [0, 4, 2048])
def test_sliced_fp32_without_entries(param):
    """An empty matrix has an FP32 product in the sliced family too."""
    spk = need_gpu()
    M = mat_on_gpu(spk, spkgen.CSR(300, np.zeros(301, np.int32), np.zeros(0, np.int32), np.zeros(0)), flags=spk.MAT_MIXED)
    spk.mat_set_kernel(M, spk.KERNEL_SLICED, param)
    x, y = to_dev(np.ones(300, np.float32)), to_dev(np.full(300, np.nan, np.float32))
    spk.mat_mult_f32(M, x, y)
    assert np.array_equal(y.cpu().numpy(), np.zeros(300, np.float32))
    M.close()
