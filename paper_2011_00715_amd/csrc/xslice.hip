// Column-sliced CSR and its binned form: layout setup on the device (counts,
// one exclusive scan, scatter) and the two-pass SpMV launch.

#include "binned.hpp"
#include "scan.hpp"
#include "xslice.hpp"
#include "runtime.hpp"

#include <cstdlib>

namespace spk {

static int grid_rows(int64_t n)
{
    int64_t g = (n + kBlock - 1) / kBlock;
    if (g > kMaxBlocksSingle) g = kMaxBlocksSingle;
    return (int)(g < 1 ? 1 : g);
}

static __global__ void k_xs_f32(int64_t m, const double *__restrict__ a, float *__restrict__ b)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < m; i += (int64_t)gridDim.x * blockDim.x)
        b[i] = (float)a[i];
}

bool sliced_fits(const spk_mat *A) { return (int64_t)kSlices * A->n + 1 < 0x7fff0000LL && A->n > 0; }

int sliced_lanes(const spk_mat *A)
{
    const double mean = A->n ? (double)A->nnz / ((double)kSlices * A->n) : 0.0;
    int L = 1;
    while (L < mean && L < 64) L <<= 1;  // next power of two of the mean slice-row length,
    return L >= 4 ? L / 2 : 2;           // halved: short slice rows leave half the lanes idle otherwise
}

// The merge path over the stacked slices has int32 diagonals.
bool sliced_merge_fits(const spk_mat *A) { return (int64_t)kSlices * A->n + A->nnz < 0x7fff0000LL; }

// Rows too uneven for a fixed number of lanes per slice row.
bool sliced_skewed(const spk_mat *A)
{
    const double mean = A->n ? (double)A->nnz / A->n : 0.0;
    return A->stats.max_len > 8 * mean + 8;
}

static void free_sliced_merge(spk_mat *A)
{
    hipFree(A->xs_tile_row);
    hipFree(A->xs_tile_k);
    hipFree(A->xs_carry_row);
    hipFree(A->xs_carry_val);
    hipFree(A->xs_slice_tile);
    A->xs_tile_row = A->xs_tile_k = A->xs_carry_row = A->xs_slice_tile = nullptr;
    A->xs_carry_val = nullptr;
    if (A->xs_tiles) A->bytes -= 20 * ((int64_t)A->xs_tiles + 1);
    A->xs_tiles = 0;
}

// Merge-path partition of the stacked slices (8n rows, nnz entries) and each
// slice's tile range.
static int setup_sliced_merge(spk_mat *A, hipStream_t s)
{
    if (A->xs_tiles) return SPK_OK;
    if (!A->xs_ptr) { set_error("internal: no sliced layout"); return SPK_EINVAL; }
    const int n = A->n;
    const int64_t rows = (int64_t)kSlices * n;
    const int64_t items = rows + A->nnz;
    if (items >= 0x7fff0000LL) { set_error("merge path over the slices needs 8n + nnz < 2^31"); return SPK_EINVAL; }
    const int T = (int)((items + kMergeItems - 1) / kMergeItems);
    int32_t head[kSlices] = {};
    for (int q = 0; q < kSlices; ++q)
        SPK_HIP(hipMemcpyAsync(&head[q], A->xs_ptr + (size_t)q * n, sizeof(int32_t), hipMemcpyDeviceToHost, s));
    SPK_HIP(hipStreamSynchronize(s));
    int32_t st[kSlices + 1];
    int most = 0;
    for (int q = 0; q < kSlices; ++q) {
        const int64_t d = (int64_t)q * n + head[q];  // merge-path diagonal where slice q starts
        st[q] = (int32_t)((d + kMergeItems - 1) / kMergeItems);
    }
    st[kSlices] = T;
    for (int q = 0; q < kSlices; ++q) most = std::max(most, st[q + 1] - st[q]);
    hipError_t e = hipMalloc(&A->xs_tile_row, sizeof(int32_t) * ((size_t)T + 1));
    if (e == hipSuccess) e = hipMalloc(&A->xs_tile_k, sizeof(int32_t) * ((size_t)T + 1));
    if (e == hipSuccess) e = hipMalloc(&A->xs_carry_row, sizeof(int32_t) * (size_t)T);
    if (e == hipSuccess) e = hipMalloc(&A->xs_carry_val, sizeof(double) * (size_t)T);
    if (e == hipSuccess) e = hipMalloc(&A->xs_slice_tile, sizeof(int32_t) * (kSlices + 1));
    if (e == hipSuccess) e = hipMemcpyAsync(A->xs_slice_tile, st, sizeof(st), hipMemcpyHostToDevice, s);
    if (e != hipSuccess) {
        free_sliced_merge(A);
        return hip_fail(e, "sliced merge setup", __FILE__, __LINE__);
    }
    A->xs_tiles = T;
    A->xs_tile_grid = std::max(1, most) * kSlices;
    A->bytes += 20 * ((int64_t)T + 1);
    hipLaunchKernelGGL(k_merge_partition, dim3(ceil_div(T + 1, kBlock)), dim3(kBlock), 0, s, (int)rows,
                       (int)A->nnz, (const int32_t *)A->xs_ptr, T, kMergeItems, A->xs_tile_row, A->xs_tile_k);
    e = hipGetLastError();
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) {
        free_sliced_merge(A);
        return hip_fail(e, "sliced merge partition", __FILE__, __LINE__);
    }
    return SPK_OK;
}

static void free_binned(spk_mat *A)
{
    hipFree(A->bn_slab);
    hipFree(A->bn_val32);
    A->bytes -= A->bn_bytes;
    A->bn_slab = nullptr;
    A->bn_val32 = nullptr;
    A->bn_bytes = 0;
    A->bn_tiles = 0;
}

static void free_slices(spk_mat *A)
{
    free_sliced_merge(A);
    A->bytes -= A->xs_bytes;
    A->xs_bytes = 0;
    hipFree(A->xs_ptr);
    hipFree(A->xs_col);
    hipFree(A->xs_val);
    hipFree(A->xs_val32);
    hipFree(A->xs_part);
    A->xs_ptr = nullptr;
    A->xs_col = nullptr;
    A->xs_val = nullptr;
    A->xs_val32 = nullptr;
    A->xs_part = nullptr;
}

void free_sliced(spk_mat *A)
{
    free_binned(A);
    free_slices(A);
}

int ensure_sliced_f32(spk_mat *A, hipStream_t s)
{
    if (A->bn_slab && !A->bn_val32) {
        SPK_HIP(hipMalloc(&A->bn_val32, sizeof(float) * ((size_t)A->nnz + 2)));
        hipLaunchKernelGGL(k_xs_f32, dim3(grid_rows(A->nnz)), dim3(kBlock), 0, s, A->nnz, (const double *)A->bn_val,
                           A->bn_val32);
        A->bytes += 4 * (A->nnz + 2);
        A->bn_bytes += 4 * (A->nnz + 2);
        SPK_HIP(hipGetLastError());
    }
    if (!A->xs_ptr || A->xs_val32) return SPK_OK;
    SPK_HIP(hipMalloc(&A->xs_val32, sizeof(float) * (size_t)std::max<int64_t>(A->nnz, 1)));
    if (A->nnz > 0)
        hipLaunchKernelGGL(k_xs_f32, dim3(grid_rows(A->nnz)), dim3(kBlock), 0, s, A->nnz, (const double *)A->xs_val,
                           A->xs_val32);
    A->bytes += 4 * A->nnz;
    A->xs_bytes += 4 * A->nnz;
    SPK_HIP(hipGetLastError());
    return SPK_OK;
}

// From this many rows on x no longer lies in the L2s beside what streams through
// them, and the products by bin pay.  FP64 / FP32 over the slices and binned:
// 40^3 27-point 18.3 / 17.0 and 28.4 / 21.8 us, 61 x 47 x 53 7-point 22.1 / 17.6 and
// 26.2 / 20.7, 64^3 32.1 / 21.7 and 28.3 / 22.7, 80^3 51.9 / 34.5 and 36.8 / 29.0.  (The
// automatic choice takes the family from 2^19 rows on.)  SPK_BINNED_ROWS in the
// environment sets another line (testing).
constexpr int kBinRows = 1 << 18;

// The bins cover n and the merge path over the rows has int32 diagonals.
bool binned_fits(const spk_mat *A)
{
    const char *e = getenv("SPK_BINNED_ROWS");
    return A->n > 0 && A->n >= (e ? atoi(e) : kBinRows) && A->n <= kBinMax * kBinCols &&
           (int64_t)A->n + A->nnz < 0x7fff0000LL;
}

static int setup_binned(spk_mat *A, hipStream_t s)
{
    if (A->bn_slab) return SPK_OK;
    const int nb = ceil_div(A->n, kBinCols);
    const int T = ceil_div((int64_t)A->n + A->nnz, kBinItems);
    const size_t m = (size_t)A->nnz + 2, cells = (size_t)nb * T;
    // Blocks of the product pass: some of each bin's entries, about four times
    // as many blocks as there are CUs (each loads its bin's x again)
    const int64_t target = std::max<int64_t>(kBinCols, A->nnz / (4 * 256));
    const size_t most = (size_t)nb + (size_t)(A->nnz / target) + 1;
    size_t at = 0;
    auto take = [&](size_t bytes) {
        const size_t o = at;
        at += (bytes + 255) / 256 * 256;
        return o;
    };
    const size_t o_tr = take(4 * ((size_t)T + 1)), o_tk = take(4 * ((size_t)T + 1)), o_ts = take(4 * (cells + nb)),
                 o_pc = take(sizeof(int4) * most), o_col = take(2 * m), o_dst = take(2 * m), o_val = take(8 * m),
                 o_prod = take(8 * m), o_cr = take(4 * (size_t)T), o_cv = take(8 * (size_t)T);
    char *tmp = nullptr;  // cell counts, their scan, the scan's block sums
    const size_t t_cp = (4 * cells + 255) / 256 * 256, t_bs = t_cp + (4 * (cells + 1) + 255) / 256 * 256;
    hipError_t e = hipMalloc(&tmp, t_bs + sizeof(long long) * ((size_t)scan_blocks((int)cells) + 1));
    if (e == hipSuccess) e = hipMalloc(&A->bn_slab, at);
    std::vector<int32_t> first((size_t)nb + 1);
    std::vector<int4> piece;
    if (e == hipSuccess) {
        char *p = A->bn_slab;
        A->bn_bytes = (int64_t)at;
        A->bytes += A->bn_bytes;
        A->bn_tiles = T;
        A->bn_bins = nb;
        A->bn_tile_row = (int32_t *)(p + o_tr);
        A->bn_tile_k = (int32_t *)(p + o_tk);
        A->bn_start = (int32_t *)(p + o_ts);
        A->bn_piece = (int4 *)(p + o_pc);
        A->bn_col = (uint16_t *)(p + o_col);
        A->bn_dst = (uint16_t *)(p + o_dst);
        A->bn_val = (double *)(p + o_val);
        A->bn_prod = p + o_prod;
        A->bn_carry_row = (int32_t *)(p + o_cr);
        A->bn_carry_val = p + o_cv;
        int32_t *cnt = (int32_t *)tmp, *cp = (int32_t *)(tmp + t_cp);
        hipLaunchKernelGGL(k_merge_partition, dim3(ceil_div(T + 1, kBlock)), dim3(kBlock), 0, s, A->n, (int)A->nnz,
                           (const int32_t *)A->rowptr, T, kBinItems, A->bn_tile_row, A->bn_tile_k);
        hipLaunchKernelGGL(k_bin_count, dim3(T), dim3(kBinThreads), 0, s, nb, T, (const int32_t *)A->bn_tile_k,
                           (const int32_t *)A->col, cnt);
        e = scan_exclusive((int)cells, cnt, cp, (long long *)(tmp + t_bs), s);
        hipLaunchKernelGGL(k_bin_fill, dim3(T), dim3(kBinThreads), 0, s, nb, T, (const int32_t *)A->bn_tile_k,
                           (const int32_t *)A->col, (const double *)A->val, (const int32_t *)cp, A->bn_start, A->bn_col,
                           A->bn_val, A->bn_dst);
        if (e == hipSuccess) e = hipGetLastError();
        // the first tile's starts are the bins'
        if (e == hipSuccess)
            e = hipMemcpyAsync(first.data(), A->bn_start, sizeof(int32_t) * nb, hipMemcpyDeviceToHost, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
    }
    if (e == hipSuccess) {
        first[nb] = (int32_t)A->nnz;
        for (int c = 0; c < nb; ++c) {
            const int64_t b = first[c], cnt = first[c + 1] - b;
            const int64_t k = cnt / target + (cnt % target != 0);
            for (int64_t i = 0; i < k; ++i)
                piece.push_back(make_int4(c, (int)(b + cnt * i / k), (int)(b + cnt * (i + 1) / k), 0));
        }
        A->bn_pieces = (int)piece.size();
        if (!piece.empty())
            e = hipMemcpyAsync(A->bn_piece, piece.data(), sizeof(int4) * piece.size(), hipMemcpyHostToDevice, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
    }
    hipFree(tmp);
    if (e != hipSuccess) {
        free_binned(A);
        return hip_fail(e, "binned layout", __FILE__, __LINE__);
    }
    const int rc = A->val32 ? ensure_sliced_f32(A, s) : SPK_OK;
    if (rc != SPK_OK) free_binned(A);  // no half a copy beside what the caller takes instead
    return rc;
}

static int setup_slices(spk_mat *A, hipStream_t s)
{
    if (A->xs_ptr) return SPK_OK;
    if (!sliced_fits(A)) {
        set_error("the sliced layout needs 8 n + 1 < 2^31");
        return SPK_EINVAL;
    }
    const int n = A->n;
    const int rows = kSlices * n;  // rows of the stacked slices
    int32_t *cnt = nullptr;
    long long *bsum = nullptr;
    int rc = SPK_OK;
    auto fail = [&](hipError_t e, const char *what) {
        hipFree(cnt);
        hipFree(bsum);
        free_slices(A);
        return hip_fail(e, what, __FILE__, __LINE__);
    };
    hipError_t e = hipMalloc(&cnt, sizeof(int32_t) * (size_t)rows);
    if (e == hipSuccess) e = hipMalloc(&bsum, sizeof(long long) * ((size_t)scan_blocks(rows) + 1));
    if (e == hipSuccess) e = hipMalloc(&A->xs_ptr, sizeof(int32_t) * ((size_t)rows + 1));
    if (e == hipSuccess) e = hipMalloc(&A->xs_col, sizeof(int32_t) * (size_t)std::max<int64_t>(A->nnz, 1));
    if (e == hipSuccess) e = hipMalloc(&A->xs_val, sizeof(double) * (size_t)std::max<int64_t>(A->nnz, 1));
    if (e == hipSuccess) e = hipMalloc(&A->xs_part, sizeof(double) * (size_t)rows);
    if (e != hipSuccess) return fail(e, "hipMalloc");
    A->xs_bytes = 4 * ((int64_t)rows + 1) + 12 * A->nnz + 8 * (int64_t)rows;
    A->bytes += A->xs_bytes;
    hipLaunchKernelGGL(k_xs_count, dim3(grid_rows(n)), dim3(kBlock), 0, s, n, (const int32_t *)A->rowptr,
                       (const int32_t *)A->col, cnt);
    e = scan_exclusive(rows, cnt, A->xs_ptr, bsum, s);
    if (e != hipSuccess) return fail(e, "slice scan");
    hipLaunchKernelGGL(k_xs_fill, dim3(grid_rows(n)), dim3(kBlock), 0, s, n, (const int32_t *)A->rowptr,
                       (const int32_t *)A->col, (const double *)A->val, (const int32_t *)A->xs_ptr, A->xs_col,
                       A->xs_val);
    e = hipGetLastError();
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return fail(e, "slice fill");
    hipFree(cnt);
    hipFree(bsum);
    if (A->val32) rc = ensure_sliced_f32(A, s);
    if (rc != SPK_OK) free_slices(A);
    return rc;
}

// merge: rows of any lengths, binned where that fits (binned_fits), else and where there is
// no room for it the merge path over the slices; the other copy is given back.
// Power-law matrices, FP64 / FP32: 600 k rows 165 / 148 us over the slices, 139 /
// 99 binned; 2 M rows 516 / 475 and 456 / 311; 4 M rows (133 M entries, FP64)
// 1142 and 898.  Above kBinMax bins the segments get too short.
int setup_sliced(spk_mat *A, int merge, hipStream_t s)
{
    if (merge && binned_fits(A) && setup_binned(A, s) == SPK_OK) {
        free_slices(A);
        return SPK_OK;
    }
    int rc = setup_slices(A, s);
    if (rc == SPK_ENOMEM && A->bn_slab) {
        // the binned copy makes room, and comes back where that is not enough
        free_binned(A);
        rc = setup_slices(A, s);
        if (rc != SPK_OK) (void)setup_binned(A, s);
    }
    if (rc == SPK_OK && merge) rc = setup_sliced_merge(A, s);
    if (rc == SPK_OK) free_binned(A);
    return rc;
}

template <class V, int L>
static void launch_xs_l(const spk_mat *A, const V *xval, const V *x, V *part, hipStream_t s, const SysState *gst,
                        int gmode)
{
    constexpr int rpb = kBlock / L;
    int nb = ceil_div(ceil_div(A->n, rpb), 2);  // two row groups per lane group and block
    if (nb > kMaxBlocksSingle) nb = kMaxBlocksSingle;
    if (nb < 1) nb = 1;
    hipLaunchKernelGGL((k_spmv_xs<V, L>), dim3(nb * kSlices), dim3(kBlock), 0, s, A->n, (const int32_t *)A->xs_ptr,
                       (const int32_t *)A->xs_col, xval, x, part, gst, gmode);
}

template <class V>
int launch_sliced(const spk_mat *A, const V *x, V *y, hipStream_t s, const SysState *gst, int gmode)
{
    const bool f64 = std::is_same<V, double>::value;
    if (A->xs_merge && A->bn_slab) {
        const V *bval = f64 ? (const V *)A->bn_val : (const V *)A->bn_val32;
        if (!bval) { set_error("internal: no binned layout with FP32 values"); return SPK_EINVAL; }
        V *prod = (V *)A->bn_prod, *cv = (V *)A->bn_carry_val;
        if (A->bn_pieces)
            hipLaunchKernelGGL((k_bin_products<V>), dim3(A->bn_pieces), dim3(kBinProdThreads), 0, s, A->n,
                               (const int4 *)A->bn_piece, (const uint16_t *)A->bn_col, bval, x, prod, gst, gmode);
        hipLaunchKernelGGL((k_bin_sum<V>), dim3((A->bn_tiles + kXcd - 1) / kXcd * kXcd), dim3(kBinThreads), 0, s,
                           A->n, A->bn_bins, A->bn_tiles, (const int32_t *)A->rowptr, (const int32_t *)A->bn_tile_row,
                           (const int32_t *)A->bn_tile_k, (const int32_t *)A->bn_start, (const uint16_t *)A->bn_dst,
                           (const V *)prod, y, A->bn_carry_row, cv, gst, gmode);
        hipLaunchKernelGGL((k_merge_fixup<V>), dim3(ceil_div(A->bn_tiles, kBlock)), dim3(kBlock), 0, s, A->n,
                           A->bn_tiles, (const int32_t *)A->bn_carry_row, (const V *)cv, y, gst, gmode);
        SPK_HIP(hipGetLastError());
        return SPK_OK;
    }
    const V *xval = f64 ? (const V *)A->xs_val : (const V *)A->xs_val32;
    if (!A->xs_ptr || !xval) {
        set_error("internal: no sliced layout%s", f64 ? "" : " with FP32 values");
        return SPK_EINVAL;
    }
    V *part = (V *)A->xs_part;
    if (A->xs_merge) {
        if (!A->xs_tiles) { set_error("internal: no merge partition of the slices"); return SPK_EINVAL; }
        const int rows = kSlices * A->n;
        V *cv = (V *)A->xs_carry_val;
        hipLaunchKernelGGL((k_spmv_xs_merge<V>), dim3(A->xs_tile_grid), dim3(kBlock), 0, s, rows,
                           (const int32_t *)A->xs_ptr, (const int32_t *)A->xs_col, xval, x, part,
                           (const int32_t *)A->xs_tile_row, (const int32_t *)A->xs_tile_k, A->xs_carry_row, cv,
                           (const int32_t *)A->xs_slice_tile, gst, gmode);
        hipLaunchKernelGGL((k_merge_fixup<V>), dim3(ceil_div(A->xs_tiles, kBlock)), dim3(kBlock), 0, s, rows,
                           A->xs_tiles, (const int32_t *)A->xs_carry_row, (const V *)cv, part, gst, gmode);
    } else {
    switch (A->lanes) {
    case 1: launch_xs_l<V, 1>(A, xval, x, part, s, gst, gmode); break;
    case 2: launch_xs_l<V, 2>(A, xval, x, part, s, gst, gmode); break;
    case 4: launch_xs_l<V, 4>(A, xval, x, part, s, gst, gmode); break;
    case 8: launch_xs_l<V, 8>(A, xval, x, part, s, gst, gmode); break;
    case 16: launch_xs_l<V, 16>(A, xval, x, part, s, gst, gmode); break;
    case 32: launch_xs_l<V, 32>(A, xval, x, part, s, gst, gmode); break;
    default: launch_xs_l<V, 64>(A, xval, x, part, s, gst, gmode); break;
    }
    }
    hipLaunchKernelGGL((k_xs_reduce<V>), dim3(grid_rows(A->n)), dim3(kBlock), 0, s, A->n, (const V *)part, y, gst,
                       gmode);
    SPK_HIP(hipGetLastError());
    return SPK_OK;
}

template int launch_sliced<double>(const spk_mat *, const double *, double *, hipStream_t, const SysState *, int);
template int launch_sliced<float>(const spk_mat *, const float *, float *, hipStream_t, const SysState *, int);

}  // namespace spk
